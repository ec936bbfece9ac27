// y = L^-T L^-1 b for the factors the library makes itself (the right-to-left L^-T L^-1 of Section 2, the
// remark after Algorithm 1): two launches, one per triangle, each a chain of 128-row blocks that
// hand their part of the solution to the next ones through device memory.
//
// What bounds it: the chain. A solve in launches of two 64-row blocks (trsv.hip) pays 9.5 + 6.5 us per
// 128 rows whatever it reads; here a block costs one trip of 128 values between compute units and two
// 128 x 128 products from registers, about 2.1 us per triangle. One application of L^-T L^-1 at n = 256,
// 1024, 2048, 4096: 27, 122, 245, 520 us before, 17, 43, 75, 135 us now (175 us at 4096 when S has
// streamed through the caches since, so that L comes from HBM: each of the 32 workgroups then waits for
// its 128 KB panels); 128 vectors of 16 factors of n = 1024: 363 us before, 75 us now.
//
// The factor is kept mirrored: L below the diagonal, L^T above it (the Cholesky writes both). The
// forward sum over L_Jk z_k and the backward sum over L_kJ^T y_k then read the same way: rows of
// block k, columns of block J, 64 lanes along a row.
//
// D_J = L_JJ^-1 (128 x 128, row-major and transposed) is formed once per factor by tri_inv_kernel.
#include "dfisher_internal.h"

#include <algorithm>
#include <cstdlib>

namespace dfi {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int TB = 128;                  // block rows
constexpr int IB = 16;                   // sub-blocks of the inverse
constexpr int NI = TB / IB;
constexpr int LDL = TB + 2;              // padded row of the block in LDS (doubles)
constexpr int SPIN_MAX = 1 << 22;        // polls of a wait (seconds; a wait is microseconds)
constexpr int SPIN_BUSY = 64;            // of them without a pause
constexpr uint64_t UNSET = TRI_UNSET;    // what a value of z or y holds until it is stored

__device__ __forceinline__ f64x4 mfma(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Lane j's value of a double (j wave-uniform).
__device__ __forceinline__ double lane_read(double v, int j) {
  const uint64_t b = __double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, j);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), j);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// D_J of one block: X_jj = L_jj^-1 for the eight 16 x 16 diagonal sub-blocks (wave j, lane c < 16 column c,
// forward substitution), then column j of sub-blocks by wave j, X_ij = -X_ii sum_{j <= k < i} L_ik X_kj
// on the matrix cores: a product's result registers are the next product's B operand, so a column stays
// in registers. Rows and columns past n are the identity's. One workgroup of 8 waves per block, all
// blocks and factors in parallel; the first column's 140 products are the length of it. 14-17 us for any
// n, against 42 us for 64-row blocks by one lane per column.
__global__ void __launch_bounds__(512)
tri_inv_kernel(const double* __restrict__ L, int64_t n, double* __restrict__ Dinv, int64_t sL, int64_t sD,
               const TriJob* __restrict__ jobs, TriPrep prep) {
  __shared__ double Ls[TB * LDL];          // the block; its diagonal sub-blocks become X_jj
  if (jobs) {
    const TriJob& j = jobs[blockIdx.y];
    L = j.L;
    Dinv = j.Dinv;
    n = j.n;
  } else {
    L += (int64_t)blockIdx.y * sL;
    Dinv += (int64_t)blockIdx.y * sD;
  }
  const int64_t nblk = (n + TB - 1) / TB, J = blockIdx.x, r0 = J * TB;
  if (J >= nblk) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = (int)min<int64_t>(TB, n - r0);
  if (prep.z) {   // for the solve behind it
    if (tid < nb) {
      reinterpret_cast<uint64_t*>(prep.z)[r0 + tid] = UNSET;
      reinterpret_cast<uint64_t*>(prep.y)[r0 + tid] = UNSET;
    }
    if (J == 0 && tid < 2) prep.ticket[tid] = 0;
  }
  {   // four rows of 128 columns at a time, all loads in flight first (clamped into the block, not guarded:
      // a branch per load would wait for each)
    const int c = tid & (TB - 1), rr = __builtin_amdgcn_readfirstlane(tid >> 7);
    const uint32_t cc = (uint32_t)min(c, nb - 1);
    double v[TB / 4];
#pragma unroll
    for (int u = 0; u < TB / 4; ++u) v[u] = (L + (r0 + min(4 * u + rr, nb - 1)) * n + r0)[cc];
#pragma unroll
    for (int u = 0; u < TB / 4; ++u) {
      const int r = 4 * u + rr;
      Ls[r * LDL + c] = (r < nb && c <= r) ? v[u] : (r == c ? 1.0 : 0.0);
    }
  }
  __syncthreads();
  const int g = lane >> 4, l16 = lane & 15;
  {
    double x[IB];
    const double* B = Ls + (w * IB) * LDL + w * IB;
    const double rd = 1.0 / B[l16 * LDL + l16];
#pragma unroll
    for (int u = 0; u < IB; ++u) x[u] = (u == l16) ? 1.0 : 0.0;
#pragma unroll
    for (int t = 0; t < IB; ++t) {
      x[t] *= lane_read(rd, t);
#pragma unroll
      for (int u = t + 1; u < IB; ++u) x[u] = fma(-B[u * LDL + t], x[t], x[u]);
      asm volatile("" ::: "memory");   // one column's operands at a time: all of them do not fit the registers
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);   // the sub-block is read before it is overwritten (one wave)
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int u = 0; u < IB; ++u) Ls[(w * IB + u) * LDL + w * IB + l16] = x[u];   // (four lanes, one value)
  }
  __syncthreads();
  double* D = Dinv + J * TB * TB;
  double* Dt = Dinv + (nblk + J) * TB * TB;
  f64x4 X[NI];   // column w: lane 16 g + c, register q: X_iw[4 q + g][c]
  auto a_at = [&](int i, int k, int s) {   // A operand, step s: row l16, column 4 s + g of sub-block (i, k)
    return Ls[(i * IB + l16) * LDL + k * IB + 4 * s + g];
  };
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    X[i] = (f64x4){0.0, 0.0, 0.0, 0.0};
    if (i == w) {
#pragma unroll
      for (int q = 0; q < 4; ++q) X[i][q] = Ls[(w * IB + 4 * q + g) * LDL + w * IB + l16];
    } else if (i > w && i * IB < nb) {   // (rows past n: zero below the identity)
      f64x4 s = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int k = 0; k < i; ++k)
        if (k >= w)
#pragma unroll
          for (int t = 0; t < 4; ++t) s = mfma(a_at(i, k, t), X[k][t], s);
#pragma unroll
      for (int t = 0; t < 4; ++t) X[i] = mfma(-a_at(i, i, t), s[t], X[i]);
    }
    asm volatile("" ::: "memory");   // likewise one row's
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      (D + (i * IB + 4 * q) * TB + w * IB)[(uint32_t)(g * TB + l16)] = X[i][q];
      (Dt + w * IB * TB + i * IB + 4 * q)[(uint32_t)(l16 * TB + g)] = X[i][q];
    }
  }
}

__device__ __forceinline__ uint64_t load_agent(const double* p) {
  return __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Tickets to zero; z and y (n values of every vector, or of every job that has not stopped) unset.
__global__ void __launch_bounds__(256)
tri_prep_kernel(double* __restrict__ z, double* __restrict__ y, int64_t n, uint32_t* __restrict__ ticket,
                const TriJob* __restrict__ jobs) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0 && blockIdx.y == 0) ticket[0] = ticket[1] = 0;   // one per triangle
  if (jobs) {
    const TriJob& j = jobs[blockIdx.y];
    if (j.skip && *j.skip) return;
    z = j.z;
    y = j.y;
    n = j.n;
  }
  if (i < n) {
    reinterpret_cast<uint64_t*>(z)[i] = UNSET;
    reinterpret_cast<uint64_t*>(y)[i] = UNSET;
  }
}

// acc[h] += sum_c m[c][h] z[c] over 16 columns: the row's 16 z are in the 16 lanes of every lane row, and
// each product takes its own by a lane-row broadcast (v_fmac_f64 with row_newbcast), without an LDS read.
// (The s_nop covers a z written by the vector ALU just before: a broadcast reads it two states later.)
__device__ __forceinline__ void dot16(double& acc, double z, const double (&m)[16]) {
#define TRI_F(l, r) "v_fmac_f64_dpp %0, %1, %" #r " row_newbcast:" #l " row_mask:0xf bank_mask:0xf\n"
  asm("s_nop 1\n" TRI_F(0, 2) TRI_F(1, 3) TRI_F(2, 4) TRI_F(3, 5) TRI_F(4, 6) TRI_F(5, 7) TRI_F(6, 8) TRI_F(7, 9)
          TRI_F(8, 10) TRI_F(9, 11) TRI_F(10, 12) TRI_F(11, 13) TRI_F(12, 14) TRI_F(13, 15) TRI_F(14, 16) TRI_F(15, 17)
      : "+v"(acc)
      : "v"(z), "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "v"(m[4]), "v"(m[5]), "v"(m[6]), "v"(m[7]), "v"(m[8]),
        "v"(m[9]), "v"(m[10]), "v"(m[11]), "v"(m[12]), "v"(m[13]), "v"(m[14]), "v"(m[15]));
#undef TRI_F
}

// Sum of x over the four 16-lane rows, in every lane (fixed order: rows (0 + 1) + (2 + 3)).
__device__ __forceinline__ double sum_rows(double x) {
  auto other = [](double v, bool half) {   // the other lane row's value: rows 0 <-> 1, 2 <-> 3, or halves
    const uint64_t b = __double_as_longlong(v);
    uint32_t r[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t w = (uint32_t)(b >> (32 * h));
      // swap with itself: the two results hold the even and the odd rows (the lower and the upper half)
      const auto s = half ? __builtin_amdgcn_permlane32_swap(w, w, false, false)
                          : __builtin_amdgcn_permlane16_swap(w, w, false, false);
      const bool odd = half ? (threadIdx.x & 32) != 0 : (threadIdx.x & 16) != 0;
      r[h] = odd ? s[0] : s[1];
    }
    return __longlong_as_double((long long)(((uint64_t)r[1] << 32) | r[0]));
  };
  x += other(x, false);
  return x + other(x, true);
}

// One triangle of the solve. Task (block J, group of up to R vectors of one factor), 8 waves: wave g owns
// the columns 16 g .. 16 g + 15 of every other block, lane l the rows l and l + 64 of block J. As the
// earlier blocks' parts of the solution appear, each wave polls its own 16 values of a part (unset
// before the launch; lane l value l % 16) and adds
//     acc_i += sum_c M[k 128 + 16 g + c][J 128 + i] out_k[16 g + c]
// from registers, the panel's 32 values per lane loaded two or three blocks ahead, and the waves meet only at the
// block's end: every wave sums its 16 entries of in_J - acc from all waves' parts, multiplies them by
// its columns of D_J (D_J^T backward; loaded as one more panel), and out_J is the sum of the waves'
// products. Two barriers per block; all sums have a fixed order.
// A workgroup takes its task by ticket, blocks in the chain's order, so it waits for earlier tickets
// only: whatever part of the grid is resident, the oldest unfinished block can run. Waits are bounded
// all the same: past the bound a wave raises *gave_up, which ends every wait; the unset values it read
// (NaN) go into the result, and the host reports the word.
template <int R, bool BWD>
__global__ void __launch_bounds__(512)
tri_kernel(const double* __restrict__ M, int64_t n, const double* __restrict__ Dinv, const double* __restrict__ in,
           double* __restrict__ out, uint32_t* __restrict__ ticket, int64_t sL, int64_t sD, int64_t nper,
           int64_t gpf, int64_t ngroup, const TriJob* __restrict__ jobs, int spin_max) {
  constexpr int NW = 8, C = TB / NW;
  __shared__ double part[2][R][NW][TB];
  __shared__ uint32_t my;
  const int tid = threadIdx.x;
  uint32_t* gave_up = ticket + 2;
  if (tid == 0) my = __hip_atomic_fetch_add(ticket + (BWD ? 1 : 0), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const uint32_t tk = __builtin_amdgcn_readfirstlane(my);
  const int64_t step = tk / (uint32_t)ngroup, grp = tk % (uint32_t)ngroup;
  int nv = 1;
  if (jobs) {
    const TriJob& j = jobs[grp];
    if (j.skip && *j.skip) return;
    M = j.L;
    Dinv = j.Dinv;
    n = j.n;
    in = BWD ? j.z : j.b;
    out = BWD ? j.y : j.z;
  } else {
    const int64_t f = grp / gpf, v0 = (grp - f * gpf) * R;
    nv = (int)min<int64_t>(R, nper - v0);
    M += f * sL;
    Dinv += f * sD;
    in += (f * nper + v0) * n;
    out += (f * nper + v0) * n;
  }
  const int64_t nblk = (n + TB - 1) / TB;
  if (step >= nblk) return;
  const int64_t J = BWD ? nblk - 1 - step : step;
  const int cnt = (int)step;                 // blocks before this one in the chain
  const int lane = tid & 63, l16 = lane & 15;
  const int g = __builtin_amdgcn_readfirstlane(tid >> 6);
  // (32-bit lane offsets from wave-uniform rows: no address registers per load)
  const uint32_t row0 = (uint32_t)min<int64_t>(J * TB + lane, n - 1);
  const uint32_t row1 = (uint32_t)min<int64_t>(J * TB + 64 + lane, n - 1);
  constexpr int NBUF = R == 1 ? 3 : 2;       // panels in registers
  double m[NBUF][2][C], acc[R][2];
  // panel s: the block's rows 16 g .. of M, columns of block J; panel cnt: D_J's
  auto load = [&](double (&p)[2][C], int s) {
    if (s > cnt) return;
    const int64_t k0 = (BWD ? nblk - 1 - s : (int64_t)s) * TB + g * C;
    const bool isd = s == cnt;
    const double* base = isd ? Dinv + ((BWD ? J : nblk + J) * TB + g * C) * TB : M + min<int64_t>(k0, n - 1) * n;
    const int64_t stride = isd ? TB : n;
    const int last = isd ? C - 1 : (int)max<int64_t>(0, min<int64_t>(C - 1, n - 1 - k0));   // rows past n: row n - 1
    const uint32_t o0 = isd ? (uint32_t)lane : row0, o1 = isd ? (uint32_t)lane + 64 : row1;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const double* r = base + min(c, last) * stride;
      p[0][c] = r[o0];
      p[1][c] = r[o1];
    }
  };
#pragma unroll
  for (int s = 0; s < NBUF; ++s) load(m[s], s);
  const int64_t at_in = J * TB + g * C + l16;   // this lane's entry of in_J
  double rhs[R];
#pragma unroll
  for (int v = 0; v < R; ++v) {
    rhs[v] = (v < nv && at_in < n) ? in[v * n + at_in] : 0.0;
    acc[v][0] = acc[v][1] = 0.0;
  }
  auto take = [&](double (&p)[2][C], int s) {
    const int64_t at = (BWD ? nblk - 1 - s : (int64_t)s) * TB + g * C + l16;
    uint64_t b[R];
    for (int spins = 0;; ++spins) {
      bool ok = true;
#pragma unroll
      for (int v = 0; v < R; ++v) {
        b[v] = (v < nv && at < n) ? load_agent(out + v * n + at) : 0;
        ok = ok && b[v] != UNSET;
      }
      if (__ballot(ok) == ~0ull) break;
      if (spins >= spin_max) {
        if (lane == 0) __hip_atomic_store(gave_up, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
      if (spins >= SPIN_BUSY) {
        if ((spins & 255) == 0 && __hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) break;
        __builtin_amdgcn_s_sleep(1);
      }
    }
#pragma unroll
    for (int v = 0; v < R; ++v) {
      if (R > 1 && v >= nv) break;
      const double z = __longlong_as_double((long long)b[v]);
      dot16(acc[v][0], z, p[0]);
      dot16(acc[v][1], z, p[1]);
    }
    load(p, s + NBUF);
  };
  for (int s = 0; s < cnt; s += NBUF)
#pragma unroll
    for (int e = 0; e < NBUF; ++e)
      if (s + e < cnt) take(m[e], s + e);
#pragma unroll
  for (int v = 0; v < R; ++v) {
    part[0][v][g][lane] = acc[v][0];
    part[0][v][g][lane + 64] = acc[v][1];
  }
  __syncthreads();
  const int q = lane >> 4;
  auto finish = [&](double (&p)[2][C]) {
#pragma unroll
    for (int v = 0; v < R; ++v) {
      if (R > 1 && v >= nv) break;
      const double s = sum_rows(part[0][v][2 * q][g * C + l16] + part[0][v][2 * q + 1][g * C + l16]);
      const double r = at_in < n ? rhs[v] - s : 0.0;
      double x0 = 0.0, x1 = 0.0;
      dot16(x0, r, p[0]);
      dot16(x1, r, p[1]);
      part[1][v][g][lane] = x0;
      part[1][v][g][lane + 64] = x1;
    }
  };
#pragma unroll
  for (int e = 0; e < NBUF; ++e)
    if (cnt % NBUF == e) finish(m[e]);
  __syncthreads();
  for (int e = tid; e < R * TB; e += 512) {
    const int v = e / TB, i = e % TB;
    const double (*p)[TB] = part[1][v];
    const double x = ((p[0][i] + p[1][i]) + (p[2][i] + p[3][i])) + ((p[4][i] + p[5][i]) + (p[6][i] + p[7][i]));
    if (v < nv && J * TB + i < n)
      __hip_atomic_store(out + v * n + J * TB + i, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// n <= 128: both triangles of one vector in one workgroup (no chain, nothing to prepare).
__global__ void __launch_bounds__(512)
tri_small_kernel(int64_t n, const double* __restrict__ Dinv, const double* __restrict__ b, double* __restrict__ z,
                 double* __restrict__ y, int64_t sD, int64_t nper) {
  constexpr int G = 4, U = TB / G;
  __shared__ double part[G][TB];
  __shared__ double rs[TB];
  const int64_t j = blockIdx.x;
  Dinv += (j / nper) * sD;
  const int tid = threadIdx.x, i = tid & (TB - 1);
  const int g = __builtin_amdgcn_readfirstlane(tid >> 7);
  double df[U], db[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    df[u] = Dinv[TB * TB + (g * U + u) * TB + i];
    db[u] = Dinv[(g * U + u) * TB + i];
  }
  if (tid < TB) rs[i] = i < n ? b[j * n + i] : 0.0;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u) s = fma(df[u], rs[g * U + u], s);
  part[g][i] = s;
  __syncthreads();
  if (tid < TB) {
    const double v = part[0][i] + part[1][i] + part[2][i] + part[3][i];
    rs[i] = v;
    if (i < n) z[j * n + i] = v;
  }
  __syncthreads();
  s = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u) s = fma(db[u], rs[g * U + u], s);
  part[g][i] = s;
  __syncthreads();
  if (tid < TB && i < n) y[j * n + i] = part[0][i] + part[1][i] + part[2][i] + part[3][i];
}

// Upper triangle := transpose of the lower one (for a factor that was made in place). 64 x 64 tiles
// through LDS; tile pair (I, J), I >= J, of matrix blockIdx.y.
__global__ void __launch_bounds__(256)
mirror_kernel(double* __restrict__ A, int64_t n, int64_t sA, const FactorJob* __restrict__ jobs) {
  __shared__ double t[64][65];
  if (jobs) {
    A = jobs[blockIdx.y].A;
    n = jobs[blockIdx.y].n;
  } else {
    A += (int64_t)blockIdx.y * sA;
  }
  const int64_t nb = (n + 63) / 64, x = blockIdx.x;
  int64_t I = (int64_t)((sqrt(8.0 * (double)x + 1.0) - 1.0) * 0.5);
  while ((I + 1) * (I + 2) / 2 <= x) ++I;
  while (I * (I + 1) / 2 > x) --I;
  const int64_t J = x - I * (I + 1) / 2;
  if (I >= nb) return;
  const int c = threadIdx.x & 63, r0 = threadIdx.x >> 6;
  for (int r = r0; r < 64; r += 4) {
    const int64_t row = I * 64 + r, col = J * 64 + c;
    t[r][c] = (row < n && col < n && col <= row) ? A[row * n + col] : 0.0;
  }
  __syncthreads();
  for (int r = r0; r < 64; r += 4) {
    const int64_t row = J * 64 + r, col = I * 64 + c;
    if (row < n && col < n && row < col) A[row * n + col] = t[c][r];
  }
}

}  // namespace

size_t tri_dinv_bytes(int64_t n) { return 2 * (size_t)((n + TB - 1) / TB) * TB * TB * sizeof(double); }

hipError_t tri_inv_batched(const double* L, int64_t sL, int64_t n, int64_t nfac, double* Dinv, hipStream_t st,
                           const TriPrep& prep) {
  if (n < 1 || nfac < 1 || nfac > 65535 || (prep.z && nfac != 1)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(tri_inv_kernel, dim3((unsigned)((n + TB - 1) / TB), (unsigned)nfac), dim3(512), 0, st, L, n, Dinv,
                     sL, (int64_t)(tri_dinv_bytes(n) / sizeof(double)), (const TriJob*)nullptr, prep);
  return hipGetLastError();
}

hipError_t tri_inv_grouped(const TriJob* jobs_dev, int64_t njobs, int64_t nmax, hipStream_t st) {
  if (nmax < 1 || njobs < 1 || njobs > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL(tri_inv_kernel, dim3((unsigned)((nmax + TB - 1) / TB), (unsigned)njobs), dim3(512), 0, st,
                     (const double*)nullptr, (int64_t)0, (double*)nullptr, (int64_t)0, (int64_t)0, jobs_dev, TriPrep{});
  return hipGetLastError();
}

// DFISHER_TRI_SPIN overrides the bound on a wait's polls (0: no value that is not there at the first look is waited for).
static int spin_max() {
  const char* e = std::getenv("DFISHER_TRI_SPIN");
  return e ? std::max(0, std::min(SPIN_MAX, std::atoi(e))) : SPIN_MAX;
}

// Several vectors of one factor share a workgroup's reads of the factor, four at a time.
hipError_t tri_solve_batched(const double* L, int64_t sL, const double* Dinv, int64_t n, int64_t nvec, int64_t nper,
                             const double* b, double* z, double* y, uint32_t* ticket, hipStream_t st, bool ready) {
  if (n < 1 || nvec < 1 || nvec > 65535 || nper < 1 || nvec % nper != 0) return hipErrorInvalidValue;
  const int64_t sD = (int64_t)(tri_dinv_bytes(n) / sizeof(double));
  if (n <= TB) {
    hipLaunchKernelGGL(tri_small_kernel, dim3((unsigned)nvec), dim3(512), 0, st, n, Dinv, b, z, y, sD, nper);
    return hipGetLastError();
  }
  const int64_t nblk = (n + TB - 1) / TB, nfac = nvec / nper;
  const int64_t R = nper == 1 ? 1 : 4, gpf = (nper + R - 1) / R, ng = nfac * gpf, tot = n * nvec;
  if (nblk * ng > 0x7FFFFFFF) return hipErrorInvalidValue;
  if (!ready)
    hipLaunchKernelGGL(tri_prep_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, z, y, tot, ticket,
                       (const TriJob*)nullptr);
  const dim3 grid((unsigned)(nblk * ng));
  const TriJob* nj = nullptr;
  const int spin = spin_max();
  for (int t = 0; t < 2; ++t) {
    const double* in = t ? z : b;
    double* out = t ? y : z;
    if (R == 1 && t == 0) hipLaunchKernelGGL((tri_kernel<1, false>), grid, dim3(512), 0, st, L, n, Dinv, in, out, ticket, sL, sD, nper, gpf, ng, nj, spin);
    if (R == 1 && t == 1) hipLaunchKernelGGL((tri_kernel<1, true>), grid, dim3(512), 0, st, L, n, Dinv, in, out, ticket, sL, sD, nper, gpf, ng, nj, spin);
    if (R == 4 && t == 0) hipLaunchKernelGGL((tri_kernel<4, false>), grid, dim3(512), 0, st, L, n, Dinv, in, out, ticket, sL, sD, nper, gpf, ng, nj, spin);
    if (R == 4 && t == 1) hipLaunchKernelGGL((tri_kernel<4, true>), grid, dim3(512), 0, st, L, n, Dinv, in, out, ticket, sL, sD, nper, gpf, ng, nj, spin);
  }
  return hipGetLastError();
}

hipError_t tri_solve_grouped(const TriJob* jobs_dev, int64_t njobs, int64_t nmax, uint32_t* ticket, hipStream_t st) {
  if (nmax < 1 || njobs < 1 || njobs > 65535) return hipErrorInvalidValue;
  const int64_t nblk = (nmax + TB - 1) / TB;
  if (nblk * njobs > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(tri_prep_kernel, dim3((unsigned)((nmax + 255) / 256), (unsigned)njobs), dim3(256), 0, st,
                     (double*)nullptr, (double*)nullptr, (int64_t)0, ticket, jobs_dev);
  const dim3 grid((unsigned)(nblk * njobs));
  const double* nd = nullptr;
  const int spin = spin_max();
  hipLaunchKernelGGL((tri_kernel<1, false>), grid, dim3(512), 0, st, nd, (int64_t)0, nd, nd, (double*)nullptr, ticket,
                     (int64_t)0, (int64_t)0, (int64_t)1, (int64_t)1, njobs, jobs_dev, spin);
  hipLaunchKernelGGL((tri_kernel<1, true>), grid, dim3(512), 0, st, nd, (int64_t)0, nd, nd, (double*)nullptr, ticket,
                     (int64_t)0, (int64_t)0, (int64_t)1, (int64_t)1, njobs, jobs_dev, spin);
  return hipGetLastError();
}

hipError_t tri_mirror_batched(double* A, int64_t n, int64_t nbatch, int64_t sA, hipStream_t st) {
  const int64_t nb = (n + 63) / 64;
  hipLaunchKernelGGL(mirror_kernel, dim3((unsigned)(nb * (nb + 1) / 2), (unsigned)nbatch), dim3(256), 0, st, A, n, sA,
                     (const FactorJob*)nullptr);
  return hipGetLastError();
}

hipError_t tri_mirror_grouped(const FactorJob* jobs_dev, int64_t njobs, int64_t nmax, hipStream_t st) {
  const int64_t nb = (nmax + 63) / 64;
  hipLaunchKernelGGL(mirror_kernel, dim3((unsigned)(nb * (nb + 1) / 2), (unsigned)njobs), dim3(256), 0, st,
                     (double*)nullptr, (int64_t)0, (int64_t)0, jobs_dev);
  return hipGetLastError();
}

}  // namespace dfi
