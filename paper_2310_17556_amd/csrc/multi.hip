// Multi-vector streaming passes over S for many right-hand sides and damping values that share
// one S: the batched form of the right-to-left evaluation x = (v - S^T L^-T L^-1 S v) / lambda
// (Section 2), where one HBM pass over S serves up to MV = 16 vectors instead of one.
//
// Row pass  B_c = S V_c for c < nv on the FP64 matrix cores (rowpass_multi_tm_kernel). A wave
//           owns 16 rows and a group of columns; a step's share of the vectors is staged in LDS as
//           FP64. Vectors are FP32 (separate arrays, the caller's right-hand sides) or FP64
//           interleaved T[k * MV + c] (the column pass output), up to four groups of MV at a time.
//           FP64 partials per (column group, vector, row) are added in fixed order by a second
//           kernel, which can also form refinement residuals r = b - lambda y - S t.
// Column pass t_c = S^T y_c for c < nc on the FP64 matrix cores. A wave owns 64 consecutive
//           columns and walks all rows, 4 at a time per product, with the y_c copied out
//           interleaved by row first. Output either T[k * MV + c] (FP64) or
//           x_c = (v_c - t_c) / lambda_c (FP32 or FP64), each column with its own v, x, lambda.
// Products of FP32 and FP64 values are formed and accumulated in FP64.
#include "dfisher_internal.h"

#include <algorithm>
#include <type_traits>

namespace dfi {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int MV = MULTI_VECS;   // 16
typedef __attribute__((address_space(3))) void lds_void;
constexpr int RM_STEP = 256;     // columns per wave step (4 per lane)

__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// one load of its own alignment only: rows of any stride and offset
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ void load_s4(const float* __restrict__ p, int64_t col, int64_t c1, f32x4& out) {
  if (col + 4 <= c1) {
    out = *reinterpret_cast<const f32x4u*>(p);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = (col + e < c1) ? p[e] : 0.f;
  }
}

// Row pass B_c = S V_c for c < nv, the vectors either FP64 interleaved, T[k * MV + c] (the
// refinement's S t_c, from the column pass), or FP32 arrays vs.f[c] (the caller's right-hand
// sides). Grid: x = blocks of RT_ROWS rows, y = column groups of cg columns; part[(g * MV + c) * n
// + i] = sum over group g of S_ik V_c[k]. The workgroup's RT_WAVES waves (32 rows) share each
// 256-column step of the vectors through LDS, widened to FP64 (32 KB, double-buffered), so the
// vectors are read once per 32 rows of S instead of once per wave. In LDS each lane's 4 columns
// x 16 vectors (512 bytes) are padded by 16 bytes, so the 16-byte fragment reads of 16
// consecutive lanes cover all banks. Four rows per wave: the 4 x 16 FP64 accumulators take 128
// registers per lane. The next step's rows of S and share of the vectors are loaded while the
// current step's products run. This form takes over when 16 row strides do not fit a 32-bit buffer offset.
constexpr int RT_WAVES = 8;
constexpr int RT_RPW = 4;                    // rows per wave
constexpr int RT_ROWS = RT_WAVES * RT_RPW;   // 32 rows per workgroup
constexpr int RT_GROUP = 4 * MV + 2;         // doubles per lane group (4 columns x MV vectors + pad)
constexpr int RT_PIECES = 256 * MV / (2 * 64 * RT_WAVES);   // 16-byte pieces of T per thread and step

template <bool FP32V>
__global__ void __launch_bounds__(64 * RT_WAVES)
rowpass_multi_t_kernel(const float* __restrict__ S, int64_t n, int64_t m, int64_t lds, const double* __restrict__ T,
                       MultiVecs vs, int nv, int64_t cg, double* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) double tl[2][64 * RT_GROUP];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int64_t row0 = (int64_t)blockIdx.x * RT_ROWS + wave * RT_RPW;
  const int64_t g = blockIdx.y;
  const int64_t c0 = g * cg;
  const int64_t c1 = min(m, c0 + cg);
  // waves whose rows lie past n still load their share of T and meet the barriers
  const int nr = (int)max<int64_t>(0, min<int64_t>(RT_RPW, n - row0));

  double acc[RT_RPW][MV];
#pragma unroll
  for (int r = 0; r < RT_RPW; ++r)
#pragma unroll
    for (int c = 0; c < MV; ++c) acc[r][c] = 0.0;

  // This thread's share of one step of the vectors, loaded into registers: FP32V, vector tid / 32
  // and 8 consecutive columns (two 16-byte loads, zero past c1 and for vectors c >= nv); else
  // RT_PIECES 16-byte pieces of T[cs .. cs + 256) x MV (zero past c1).
  static_assert(!FP32V || 64 * RT_WAVES == 32 * MV, "one vector per 32 threads");
  struct VecShare {
    f32x4 f[2];
    f64x2 t[RT_PIECES];
  };
  auto load_vecs = [&](int64_t cs, VecShare& vsh) {
    if constexpr (FP32V) {
      const int c = tid >> 5;
      const int cl0 = (tid & 31) * 8;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int cl = cl0 + 4 * h;
        vsh.f[h] = (f32x4){0.f, 0.f, 0.f, 0.f};
        if (c < nv) load_s4(vs.f[c] + cs + cl, cs + cl, c1, vsh.f[h]);
      }
    } else {
#pragma unroll
      for (int h = 0; h < RT_PIECES; ++h) {
        const int idx = 2 * (h * 64 * RT_WAVES + tid);   // double index in the step: column idx / MV, vector idx % MV
        vsh.t[h] = (f64x2){0.0, 0.0};
        if (cs + idx / MV < c1) vsh.t[h] = *reinterpret_cast<const f64x2*>(T + cs * MV + idx);
      }
    }
  };
  // ... and stored to LDS, widened to FP64, in the layout the products read
  auto store_vecs = [&](const VecShare& vsh, double* tb) {
    if constexpr (FP32V) {
      const int c = tid >> 5;
      const int cl0 = (tid & 31) * 8;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) tb[((cl0 + 4 * h) >> 2) * RT_GROUP + e * MV + c] = (double)vsh.f[h][e];
    } else {
#pragma unroll
      for (int h = 0; h < RT_PIECES; ++h) {
        const int idx = 2 * (h * 64 * RT_WAVES + tid);
        const int cl = idx / MV;
        *reinterpret_cast<f64x2*>(&tb[(cl >> 2) * RT_GROUP + (cl & 3) * MV + (idx % MV)]) = vsh.t[h];
      }
    }
  };
  auto load_rows = [&](int64_t cs, f32x4* sv) {
    const int64_t col = cs + 4 * lane;
#pragma unroll
    for (int r = 0; r < RT_RPW; ++r) {
      sv[r] = (f32x4){0.f, 0.f, 0.f, 0.f};
      if (r < nr) load_s4(S + (row0 + r) * lds + col, col, c1, sv[r]);
    }
  };
  // Software pipeline: step cs + 256's rows of S and share of the vectors are loaded into
  // registers while step cs's products run, so each step's loads have a whole step to arrive.
  VecShare vn;
  f32x4 sn[RT_RPW];
  if (c0 < c1) {
    load_vecs(c0, vn);
    load_rows(c0, sn);
  }
  int buf = 0;
  for (int64_t cs = c0; cs < c1; cs += RM_STEP, buf ^= 1) {
    store_vecs(vn, tl[buf]);
    __syncthreads();   // the other buffer is rewritten only after the next step's barrier
    f32x4 sv[RT_RPW];
#pragma unroll
    for (int r = 0; r < RT_RPW; ++r) sv[r] = sn[r];
    if (cs + RM_STEP < c1) {
      load_vecs(cs + RM_STEP, vn);
      load_rows(cs + RM_STEP, sn);
    }
    const double* tg = &tl[buf][lane * RT_GROUP];
    // one column at a time: its MV vector entries are live only while its products are formed
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      double vv[MV];
#pragma unroll
      for (int c = 0; c < MV; c += 2) {
        const f64x2 t2 = *reinterpret_cast<const f64x2*>(tg + e * MV + c);
        vv[c] = t2[0];
        vv[c + 1] = t2[1];
      }
#pragma unroll
      for (int r = 0; r < RT_RPW; ++r) {
        const double sd = (double)sv[r][e];
#pragma unroll
        for (int c = 0; c < MV; ++c) acc[r][c] = fma(sd, vv[c], acc[r][c]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int r = 0; r < RT_RPW; ++r) {
    if (r >= nr) continue;
#pragma unroll
    for (int c = 0; c < MV; ++c) {
      const double t = wave_sum(acc[r][c]);
      if (lane == 0 && c < nv) part[(g * MV + c) * n + row0 + r] = t;
    }
  }
}

// The row pass on the FP64 matrix cores. A wave owns 16 rows; a workgroup of RowShape::WAVES waves
// walks its column group STEP columns at a time, with that step of the vectors staged in LDS
// (double-buffered; of 4 columns k .. k + 3 with k / 4 = w, column k + e's 16 vectors lie in the quarter (e + w) % 4 of
// their 512 bytes, so that the 4 columns 4 apart that a product reads lie in different quarters: no bank conflicts). Per step each lane = 16 kr + q loads
// row r0 + q, columns 16 u + 4 kr .. + 3 for u < STEP / 16 (16 bytes each), and product (u, j) takes
// element j of load u as its A operand (row q, column 16 u + 4 kr + j) and
// T[16 u + 4 kr + j][q] from LDS as its B operand: D(16 rows x 16 vectors) +=
// S(16 x 4) T(4 x 16) with v_mfma_f64_16x16x4f64. Lane l then holds D[row kr + 4 r][vector q] in
// register r, the partial this wave stores for the group. Rows past n and columns past c1 read
// as zero. S of the next step is loaded while this step's products run.
//
// NG groups of up to MV vectors share every load and conversion of S. With one group the pass is bound by
// reading S, with four by the products (64 cycles each): over 2048 x 200000 1 group takes 317 us (5.2 TB/s; 394 when the
// step's vectors went through registers and its loads were waited for at once), FP32 vectors 319 (530 on the vector unit);
// over 1024 x 250000 4 groups take 538 us (61 of 78 TFLOP/s), where two passes of 2 groups took 380 each.
// A step is 128 columns; with three or four groups 8 waves share its 64 vectors in LDS (128 KB, one
// workgroup a compute unit, two waves a SIMD).
__device__ __forceinline__ int rg_slot(int col, int c) { return (col >> 2) * (4 * MV) + (((col + (col >> 2)) & 3) * MV) + c; }
template <int NG>
struct RowShape {
  static constexpr int WAVES = NG <= 2 ? 4 : 8;
  static constexpr int ROWS = 16 * WAVES;
  static constexpr int STEP = 128;                    // columns per step
};
struct GroupPtrs {
  const double* T[MULTI_GROUPS];
  double* part[MULTI_GROUPS];
  int nv[MULTI_GROUPS];
};

template <int NG, bool FP32V>
__global__ void __launch_bounds__(64 * RowShape<NG>::WAVES, 2)
rowpass_multi_tm_kernel(const float* __restrict__ S, int64_t n, int64_t m, int64_t lds, GroupPtrs gp, MultiVecs vs,
                        int64_t cg) {
  static_assert(!FP32V || NG == 1, "FP32 vectors come one group at a time");
  constexpr int W = RowShape<NG>::WAVES;
  constexpr int STEP = RowShape<NG>::STEP;
  constexpr int BUF = STEP * MV;                        // doubles per LDS buffer and group
  constexpr int PIECES = STEP * MV / 2 / (64 * W);      // 16-byte pieces of T per thread, step, group
  constexpr int NU = STEP / 16;                         // 16-byte loads of S per lane and step
  // two objects, named by constants: the compiler then knows which one the loads in flight go to
  __shared__ __attribute__((aligned(16))) double tl0[NG][BUF];
  __shared__ __attribute__((aligned(16))) double tl1[NG][BUF];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane & 15, kr = lane >> 4;
  // the row blocks of a column group run on one XCD (workgroup w on XCD w % 8) at about the same time: its L2 serves
  // their reads of the vectors
  const int64_t rb = (n + RowShape<NG>::ROWS - 1) / RowShape<NG>::ROWS;
  const int64_t l = blockIdx.x >> 3;
  const int64_t g = l / rb * 8 + (blockIdx.x & 7);
  const int64_t rbase = l % rb * RowShape<NG>::ROWS + wave * 16;
  const int64_t c0 = g * cg;
  const int64_t c1 = min(m, c0 + cg);
  if (c0 >= m) return;
  auto buffer = [&](auto bc) __attribute__((always_inline)) -> double (&)[NG][BUF] {
    if constexpr (decltype(bc)::value == 0) return tl0;
    else return tl1;
  };
  // FP64 vectors go from memory to LDS directly: wave instruction i carries the 128 bytes of each of columns 8 i .. + 7 of
  // the step, lane l the column of its quarter (see rg_slot). The buffer ends with the column group: zeros behind it.
  const __amdgpu_buffer_rsrc_t rt[4] = {
      __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(gp.T[0] + c0 * MV), 0, (int)((c1 - c0) * MV * 8), 0x00020000),
      __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(gp.T[1] + c0 * MV), 0, (int)((c1 - c0) * MV * 8), 0x00020000),
      __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(gp.T[2] + c0 * MV), 0, (int)((c1 - c0) * MV * 8), 0x00020000),
      __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(gp.T[3] + c0 * MV), 0, (int)((c1 - c0) * MV * 8), 0x00020000)};
  static_assert(W % 2 == 0, "the lanes' columns are the same for every instruction of a wave");
  const int w0 = 2 * wave + (lane >> 5);
  const uint32_t toff = (uint32_t)((4 * w0 + (((lane >> 3) - w0) & 3)) * (MV * 8) + (lane & 7) * 16);
  // FP32 vectors (waves whose rows lie past n stage their share too): a thread's two 4-column pieces of one vector
  static_assert(!FP32V || (STEP * MV == 8 * 64 * W), "8 entries a thread");
  f32x4 sh[2];
  auto load_t = [&](auto bc, int64_t cs) __attribute__((always_inline)) {
    if constexpr (FP32V) {
      const int c = tid & (MV - 1);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int64_t col = cs + 4 * (tid / MV + (4 * W) * h);
        sh[h] = (f32x4){0.f, 0.f, 0.f, 0.f};
        if (c < gp.nv[0]) load_s4(vs.f[c] + col, col, c1, sh[h]);
      }
    } else {
      const uint32_t o = toff + (uint32_t)(cs - c0) * (MV * 8);
#pragma unroll
      for (int gg = 0; gg < NG; ++gg)
#pragma unroll
        for (int h = 0; h < PIECES; ++h)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rt[gg], (lds_void*)(&buffer(bc)[gg][(wave + W * h) * 8 * MV]), 16,
                                                   (int)(o + W * h * 8 * MV * 8), 0, 0, 0);
    }
  };
  auto store_t = [&](auto bc) __attribute__((always_inline)) {
    if constexpr (FP32V) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          buffer(bc)[0][rg_slot(4 * (tid / MV + (4 * W) * h) + e, tid & (MV - 1))] = (double)sh[h][e];
    }
  };
  // The wave's 16 rows of S as one buffer from a wave-uniform base (row rbase, column c0) with a
  // 32-bit lane offset (the launcher checks 16 lds * 4 < 2^31): the records end with S, so lanes
  // of rows past n read zeros, and a wave with no rows below n has no records and touches no memory.
  const int rin = (int)max<int64_t>(0, min<int64_t>(16, n - rbase));
  const float* sbase = S + (rin > 0 ? rbase : 0) * lds + c0;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(sbase), 0, row_records(rin, (int)lds, (int)(m - c0)), 0x00020000);
  const uint32_t qoff = (uint32_t)((int64_t)q * lds * 4);
  // NA independent accumulators per group (product j of each load into accumulator j % NA), added
  // in a fixed order at the end: a single chain of dependent products per group would, with few groups,
  // leave the matrix cores waiting on each product's result
  constexpr int NA = NG <= 2 ? 2 : 1;
  f64x4 acc[NG][NA];
#pragma unroll
  for (int gg = 0; gg < NG; ++gg)
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[gg][a] = (f64x4){0.0, 0.0, 0.0, 0.0};
  int slot[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) slot[j] = rg_slot(4 * kr + j, q);
  auto load_s = [&](int64_t cs, f32x4* sv) {
    const int kc = (int)(cs - c0);
#pragma unroll
    for (int u = 0; u < NU; ++u)
      sv[u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                            rs, (int)(qoff + 4u * (uint32_t)(kc + 16 * u + 4 * kr)), 0, 0));
  };
  // A step's products, S in sv and the vectors in a buffer. LDS operands are read one load of S ahead of their products.
  auto products = [&](auto bc, const f32x4* sv) __attribute__((always_inline)) {
    double b[2][4][NG];
    auto read_b = [&](int u) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int gg = 0; gg < NG; ++gg) b[u & 1][j][gg] = buffer(bc)[gg][4 * u * (4 * MV) + slot[j]];   // column 16 u + 4 kr + j
    };
    read_b(0);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      if (u + 1 < NU) read_b(u + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double a = (double)sv[u][j];
#pragma unroll
        for (int gg = 0; gg < NG; ++gg)
          acc[gg][j % NA] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b[u & 1][j][gg], acc[gg][j % NA], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);   // widen load u's values only where its products use them
    }
  };
  // The loads of vectors into LDS have landed: all but the loads of S issued behind them (kept there by the fence in load).
  // (vmcnt(NU), the other counters alone.)
  auto landed = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!FP32V) __builtin_amdgcn_s_waitcnt((NU & 15) | ((NU >> 4) << 14) | (7 << 4) | (15 << 8));
    asm volatile("" ::: "memory");
  };
  auto load = [&](auto bc, int64_t cs, f32x4* sv) __attribute__((always_inline)) {
    load_t(bc, cs);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    load_s(cs, sv);
    __builtin_amdgcn_sched_barrier(0);
  };
  // A step with another behind it, whose S goes to nx and whose vectors go to the other buffer meanwhile. Two register sets
  // in turn and no branch: with one set and a copy, or loads under a condition, the compiler waits for the loads as soon
  // as they are issued, a whole memory latency a step.
  auto step = [&](auto bc, int64_t cs, const f32x4* sv, f32x4* nx) __attribute__((always_inline)) {
    using Other = std::integral_constant<int, 1 - decltype(bc)::value>;
    load(Other{}, cs + STEP, nx);
    products(bc, sv);
    store_t(Other{});   // last read before the previous barrier
    landed();
    __syncthreads();
  };
  // the last step: columns past c1 count as zero
  auto last = [&](auto bc, int64_t cs, f32x4* sv) __attribute__((always_inline)) {
    const int lim = (int)(c1 - cs);
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) sv[u][e] = (16 * u + 4 * kr + e < lim) ? sv[u][e] : 0.f;
    products(bc, sv);
  };
  {
    using B0 = std::integral_constant<int, 0>;
    using B1 = std::integral_constant<int, 1>;
    f32x4 s0[NU], s1[NU];
    load(B0{}, c0, s0);
    store_t(B0{});
    landed();
    __syncthreads();
    int64_t cs = c0;
    for (; cs + 2 * STEP < c1; cs += 2 * STEP) {
      step(B0{}, cs, s0, s1);
      step(B1{}, cs + STEP, s1, s0);
    }
    if (cs + STEP < c1) {
      step(B0{}, cs, s0, s1);
      last(B1{}, cs + STEP, s1);
    } else {
      last(B0{}, cs, s0);
    }
  }
#pragma unroll
  for (int gg = 0; gg < NG; ++gg) {
    if (q >= gp.nv[gg]) continue;
    double* part = gp.part[gg];
    f64x4 tot = acc[gg][0];
#pragma unroll
    for (int a = 1; a < NA; ++a) tot += acc[gg][a];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t rr = rbase + kr + 4 * r;
      if (rr < n) part[(g * MV + q) * n + rr] = tot[r];
    }
  }
}

// out.b[c][i] = sum_g part[(g * MV + c) * n + i]; with out.r0[c] set:
// out.b[c][i] = (r0_c[i] - lam_c y_c[i]) - sum_g part[...] (refinement residual).
// (blockIdx.z: the group)
struct GroupOuts {
  const double* part[MULTI_GROUPS];
  int nv[MULTI_GROUPS];
  MultiOut out[MULTI_GROUPS];
};
__global__ void rowpass_multi_reduce_kernel(int64_t n, int64_t ngroups, GroupOuts go) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int c = blockIdx.y, z = blockIdx.z;
  if (i >= n || c >= go.nv[z]) return;
  const double* part = go.part[z];
  const MultiOut& out = go.out[z];
  double s = 0.0;
  int64_t g = 0;
  for (; g + 8 <= ngroups; g += 8) {   // eight loads at a time, added in order
    double p[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) p[k] = part[((g + k) * MV + c) * n + i];
#pragma unroll
    for (int k = 0; k < 8; ++k) s += p[k];
  }
  for (; g < ngroups; ++g) s += part[(g * MV + c) * n + i];
  const double* r0 = out.r0[c];
  out.b[c][i] = r0 ? (r0[i] - out.lam[c] * out.y[c][i]) - s : s;
}

// Yi[(i ng + g) MV + c] = cols.g[g].y[c][i] for i < n, c < MV, g < ng: the y vectors interleaved by row.
struct GroupCols {
  MultiCols g[MULTI_GROUPS];
  int nc[MULTI_GROUPS];
};
__global__ void interleave_y_kernel(GroupCols cols, int64_t n, int ng, double* __restrict__ Yi) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = idx / (ng * MV);
  const int c = (int)(idx % (ng * MV));
  if (i < n) Yi[idx] = cols.g[c / MV].y[c % MV][i];
}

// The column pass on the FP64 matrix cores: per wave 64 consecutive columns, D_j(16 vectors x 16
// columns) += Y(4 rows x 16 vectors)^T S(4 rows x 16 columns) with v_mfma_f64_16x16x4f64. Lane l
// = 16 kr + q loads row i + kr, columns col .. col + 3 (col = c0 + 4 q) of S with one 16-byte load
// and supplies element j to product j (columns col + j: D_j covers columns c0 + 4 n + j); its A
// operand is Yi[((i + kr) NG + g) MV + q], one 8-byte load a group. Lane l holds D_j[vector kr + 4 r][n = q] in
// register r. Each product adds 4 rows (its k = 4) in FP64; rows past n and columns past m read
// as zero. NG groups share every load and conversion of S; an iteration takes 16 rows, whose loads went out under the
// products before. As for the row pass, one group is bound by reading S and four by the products: T out, 2048 x 200000
// 342 us for 1 group (383 with guarded loads), 1024 x 250000 550 us for 4 (two passes of 2: 360 each); x out 528 (443 each).
constexpr int CF_WAVES = 4;
constexpr int CF_COLS = 64;    // columns per wave
constexpr int CF_GROUPS = 4;   // 4-row groups per loop step
static_assert(MV == 16, "one MFMA dimension holds the vectors");

struct GroupT {
  double* T[MULTI_GROUPS];
};

template <int MODE, int NG>
__global__ void __launch_bounds__(64 * CF_WAVES, NG >= 3 ? 2 : NG == 2 ? 3 : 4)
colpass_multi_mfma_kernel(const float* __restrict__ S, int64_t n, int64_t m, int64_t lds, GroupCols cols,
                          const double* __restrict__ Yi, GroupT tt, const int* __restrict__ skip) {
  if (skip && *skip) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t own = ((int64_t)blockIdx.x * CF_WAVES + wave) * CF_COLS;   // first column this wave stores
  if (own >= m) return;   // the whole wave
  // the last wave takes the last 64 columns (a partial one would go through guarded loads: 330 us at the end of a 540 us pass)
  const int64_t c0 = m >= CF_COLS ? min(own, m - CF_COLS) : 0;
  const int q = lane & 15, kr = lane >> 4;
  const int64_t col = c0 + 4 * q;
  f64x4 acc[NG][4];
#pragma unroll
  for (int gg = 0; gg < NG; ++gg)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[gg][j] = (f64x4){0.0, 0.0, 0.0, 0.0};
  struct Rows {
    f32x4 s[CF_GROUPS];
    double y[NG][CF_GROUPS];
  };
  constexpr int ROWS = 4 * CF_GROUPS;
  auto products = [&](const Rows& a) __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < CF_GROUPS; ++g)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double b = (double)a.s[g][j];
#pragma unroll
        for (int gg = 0; gg < NG; ++gg) acc[gg][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y[gg][g], b, acc[gg][j], 0, 0, 0);
      }
  };
  int64_t i = 0;
  if (m >= CF_COLS && n >= ROWS) {   // 16 whole rows of 64 columns at a time: loads without a test
    const float* sp = S + kr * lds + col;
    const double* yp = Yi + kr * (MV * NG) + q;
    auto load = [&](Rows& a) __attribute__((always_inline)) {
#pragma unroll
      for (int g = 0; g < CF_GROUPS; ++g) {
        a.s[g] = *reinterpret_cast<const f32x4u*>(sp + 4 * g * lds);
#pragma unroll
        for (int gg = 0; gg < NG; ++gg) a.y[gg][g] = yp[(4 * g * NG + gg) * MV];
      }
    };
    const int64_t full = n / ROWS * ROWS;
    int64_t at = 0;   // rows the next load takes (at the end the last ones again, unused)
    auto next = [&](Rows& a) __attribute__((always_inline)) {
      load(a);
      const int64_t step = at + ROWS < full ? ROWS : 0;
      at += step;
      sp += step * lds;
      yp += step * (NG * MV);
    };
    Rows r0, r1;   // in turn: no copies
    next(r0);
    for (; i + 2 * ROWS <= full; i += 2 * ROWS) {
      next(r1);
      products(r0);
      __builtin_amdgcn_sched_barrier(0);
      next(r0);
      products(r1);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (i < full) products(r0);
    i = full;
  }
  for (; i < n; i += ROWS) {   // the last n % 16 rows, or all of them where m < 64
    Rows a;
#pragma unroll
    for (int g = 0; g < CF_GROUPS; ++g) {
      const int64_t row = i + 4 * g + kr;
      a.s[g] = (f32x4){0.f, 0.f, 0.f, 0.f};
      if (row < n) load_s4(S + row * lds + col, col, m, a.s[g]);
#pragma unroll
      for (int gg = 0; gg < NG; ++gg) a.y[gg][g] = row < n ? Yi[(row * NG + gg) * MV + q] : 0.0;
    }
    products(a);
  }
  if constexpr (MODE == 2) {
#pragma unroll
    for (int gg = 0; gg < NG; ++gg) {
      double* T = tt.T[gg];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (col + j >= m || col + j < own) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) T[(col + j) * MV + kr + 4 * r] = acc[gg][j][r];
      }
    }
  } else {
    // a lane has four columns of the vectors kr + 4 r: their pointers from LDS, one load and one store of four columns
    __shared__ const float* vp[NG * MV];
    __shared__ void* xp[NG * MV];
    __shared__ double lam[NG * MV];
    if (lane < NG * MV) {   // every wave writes the same (a wave past m has returned: no barrier)
      vp[lane] = cols.g[lane / MV].v[lane % MV];
      xp[lane] = cols.g[lane / MV].x[lane % MV];
      lam[lane] = cols.g[lane / MV].lam[lane % MV];
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int gg = 0; gg < NG; ++gg)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = kr + 4 * r;
        if (c >= cols.nc[gg]) continue;
        const float* v = vp[gg * MV + c];
        void* x = xp[gg * MV + c];
        const double l = lam[gg * MV + c];
        f32x4 vv;
        load_s4(v + col, col, m, vv);
        double xs[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) xs[j] = ((double)vv[j] - acc[gg][j][r]) / l;
        if constexpr (MODE == 0) {
          float* xf = static_cast<float*>(x) + col;
          if (col + 4 <= m && col >= own) *reinterpret_cast<f32x4u*>(xf) = (f32x4){(float)xs[0], (float)xs[1], (float)xs[2], (float)xs[3]};
          else
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (col + j < m && col + j >= own) xf[j] = (float)xs[j];
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (col + j < m && col + j >= own) static_cast<double*>(x)[col + j] = xs[j];
        }
      }
  }
}

__global__ void axpy_many_kernel(double* __restrict__ y, const double* __restrict__ d, int64_t len) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < len) y[i] += d[i];
}

}  // namespace

RowMultiPlan rowmulti_plan(int64_t n, int64_t m, int64_t lds) {
  RowMultiPlan p{};
  p.n = n;
  p.m = m;
  p.lds = lds;
  const int64_t rowblocks = (n + RT_ROWS - 1) / RT_ROWS;
  const int64_t target = std::max<int64_t>(1, 2048 / rowblocks);       // ~2048 workgroups
  const int64_t maxg = (m + 2047) / 2048;                                // >= 2048 columns per group
  p.nchunk = std::max<int64_t>(1, std::min(target, maxg));
  int64_t cg = (m + p.nchunk - 1) / p.nchunk;
  cg = (cg + RM_STEP - 1) / RM_STEP * RM_STEP;
  p.chunk = cg;
  p.nchunk = (m + cg - 1) / cg;
  p.part_bytes = (size_t)p.nchunk * MV * (size_t)n * sizeof(double);
  return p;
}

RowMultiPlan rowmulti_groups(const RowMultiPlan& p, int ng) {
  RowMultiPlan r = p;
  if (ng < 3 || 16 * p.lds * 4 >= ((int64_t)1 << 31)) return r;
  // one workgroup a compute unit: as many column groups as just fill whole rounds of 256, of p's at most
  const int64_t rb = (p.n + RowShape<4>::ROWS - 1) / RowShape<4>::ROWS;
  const int64_t rounds = rb * p.nchunk / 256;
  if (rounds < 1) return r;
  const int64_t want = 256 * rounds / rb;
  constexpr int64_t step = RowShape<4>::STEP;
  r.chunk = ((p.m + want - 1) / want + step - 1) / step * step;
  r.nchunk = (p.m + r.chunk - 1) / r.chunk;
  return r;
}

namespace {
template <int NG, bool FP32V>
void tm_launch(const RowMultiPlan& p, const float* S, const GroupPtrs& gp, const MultiVecs& vs, hipStream_t st) {
  constexpr int rows = RowShape<NG>::ROWS;
  hipLaunchKernelGGL((rowpass_multi_tm_kernel<NG, FP32V>), dim3((unsigned)((p.n + rows - 1) / rows * ((p.nchunk + 7) / 8 * 8))),
                     dim3(4 * rows), 0, st, S, p.n, p.m, p.lds, gp, vs, p.chunk);
}

template <int MODE>
void col_launch(const float* S, int64_t n, int64_t m, int64_t lds, const GroupCols& gc, int ng, const double* Yi,
                const GroupT& tt, hipStream_t st, const int* skip) {
  const dim3 grid((unsigned)((m + CF_WAVES * CF_COLS - 1) / (CF_WAVES * CF_COLS)));
  const dim3 block(64 * CF_WAVES);
  switch (ng) {
    case 1: hipLaunchKernelGGL((colpass_multi_mfma_kernel<MODE, 1>), grid, block, 0, st, S, n, m, lds, gc, Yi, tt, skip); break;
    case 2: hipLaunchKernelGGL((colpass_multi_mfma_kernel<MODE, 2>), grid, block, 0, st, S, n, m, lds, gc, Yi, tt, skip); break;
    case 3: hipLaunchKernelGGL((colpass_multi_mfma_kernel<MODE, 3>), grid, block, 0, st, S, n, m, lds, gc, Yi, tt, skip); break;
    default: hipLaunchKernelGGL((colpass_multi_mfma_kernel<MODE, 4>), grid, block, 0, st, S, n, m, lds, gc, Yi, tt, skip); break;
  }
}

bool counts_ok(const int* c, int ng) {
  if (ng < 1 || ng > MULTI_GROUPS) return false;
  for (int g = 0; g < ng; ++g)
    if (c[g] < 1 || c[g] > MV) return false;
  return true;
}
}  // namespace

hipError_t rowpass_multi_launch(const RowMultiPlan& p, const float* S, const MultiVecs& vs, int nv, double* part,
                                hipStream_t st) {
  if (nv < 1 || nv > MV) return hipErrorInvalidValue;
  if (16 * p.lds * 4 < ((int64_t)1 << 31) && p.chunk < ((int64_t)1 << 24)) {
    GroupPtrs gp{};
    gp.part[0] = part;
    gp.nv[0] = nv;
    tm_launch<1, true>(p, S, gp, vs, st);
  } else {
    hipLaunchKernelGGL(rowpass_multi_t_kernel<true>, dim3((unsigned)((p.n + RT_ROWS - 1) / RT_ROWS), (unsigned)p.nchunk),
                       dim3(64 * RT_WAVES), 0, st, S, p.n, p.m, p.lds, (const double*)nullptr, vs, nv, p.chunk, part);
  }
  return hipGetLastError();
}

hipError_t rowpass_multi_groups(const RowMultiPlan& p, const float* S, const double* const* T, const int* nv, int ng,
                                double* const* part, hipStream_t st) {
  if (!counts_ok(nv, ng)) return hipErrorInvalidValue;
  const MultiVecs none{};
  if (16 * p.lds * 4 >= ((int64_t)1 << 31) || p.chunk >= ((int64_t)1 << 24)) {   // a pass per group
    for (int g = 0; g < ng; ++g)
      hipLaunchKernelGGL(rowpass_multi_t_kernel<false>, dim3((unsigned)((p.n + RT_ROWS - 1) / RT_ROWS), (unsigned)p.nchunk),
                         dim3(64 * RT_WAVES), 0, st, S, p.n, p.m, p.lds, T[g], none, nv[g], p.chunk, part[g]);
    return hipGetLastError();
  }
  GroupPtrs gp{};
  for (int g = 0; g < ng; ++g) {
    gp.T[g] = T[g];
    gp.part[g] = part[g];
    gp.nv[g] = nv[g];
  }
  switch (ng) {
    case 1: tm_launch<1, false>(p, S, gp, none, st); break;
    case 2: tm_launch<2, false>(p, S, gp, none, st); break;
    case 3: tm_launch<3, false>(p, S, gp, none, st); break;
    default: tm_launch<4, false>(p, S, gp, none, st); break;
  }
  return hipGetLastError();
}

hipError_t rowpass_multi_reduce(const RowMultiPlan& p, const double* const* part, const int* nv, int ng,
                                const MultiOut* out, hipStream_t st) {
  if (!counts_ok(nv, ng)) return hipErrorInvalidValue;
  GroupOuts go{};
  int most = 0;
  for (int g = 0; g < ng; ++g) {
    go.part[g] = part[g];
    go.nv[g] = nv[g];
    go.out[g] = out[g];
    most = std::max(most, nv[g]);
  }
  hipLaunchKernelGGL(rowpass_multi_reduce_kernel, dim3((unsigned)((p.n + 255) / 256), (unsigned)most, (unsigned)ng),
                     dim3(256), 0, st, p.n, p.nchunk, go);
  return hipGetLastError();
}

hipError_t colpass_multi_groups(const float* S, int64_t n, int64_t m, int64_t lds, const MultiCols* mc, const int* nc,
                                int ng, int mode, double* const* T, double* Yi, hipStream_t st, const int* skip) {
  if (!counts_ok(nc, ng) || !Yi) return hipErrorInvalidValue;
  GroupCols gc{};
  GroupT tt{};
  for (int g = 0; g < ng; ++g) {
    gc.g[g] = mc[g];
    gc.nc[g] = nc[g];
    if (mode == 2) {
      if (!T[g]) return hipErrorInvalidValue;
      tt.T[g] = T[g];
    }
  }
  hipLaunchKernelGGL(interleave_y_kernel, dim3((unsigned)((n * MV * ng + 255) / 256)), dim3(256), 0, st, gc, n, ng, Yi);
  switch (mode) {
    case 0: col_launch<0>(S, n, m, lds, gc, ng, Yi, tt, st, skip); break;
    case 1: col_launch<1>(S, n, m, lds, gc, ng, Yi, tt, st, skip); break;
    case 2: col_launch<2>(S, n, m, lds, gc, ng, Yi, tt, st, skip); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t axpy_many(double* y, const double* d, int64_t len, hipStream_t st) {
  hipLaunchKernelGGL(axpy_many_kernel, dim3((unsigned)((len + 255) / 256)), dim3(256), 0, st, y, d, len);
  return hipGetLastError();
}

}  // namespace dfi
