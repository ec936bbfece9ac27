// FP64 Cholesky W = L L^T (Algorithm 1 step 2) in one launch: a task per 64 x 64 tile of the lower
// triangle, ordered by data flags in device memory instead of by launches.
//
// What bounds it: for n <= 2048 the chain over the block columns (factor a diagonal block, solve the
// block below it, update the next diagonal block), not its n^3 / 3 products. The launch-per-step form
// (potrf.hip) pays 34 us per 64 columns for that chain: two launches with their gaps (8 us), a 20 us
// diagonal factor on the vector ALU and a panel solve that waits for all of it. Here the chain stays
// inside one workgroup per block column and everything else runs ahead of it on other compute units.
// A block column takes 11 us: 0.8 us for the last panel to reach the next task, 0.6 us for its solve and
// update, 4 x 1.1 us of factor16, 4 x 0.7 us between them, the rest the wait for the previous block
// column's strips. dfisher_potrf, n = 256, 1024, 2048, 4096: 155, 548, 1106, 2444 us before, 78, 209,
// 400, 1030 us now (45 us of each are the call's wait and its small launches); at
// n = 4096 the products run at 23 TFLOP/s of the 72 that a large FP64 product reaches.
//
// Task of an off-diagonal tile (I, J), four waves of 16 rows each, nothing shared between them
// (left-looking: the tile is read once and written once):
//     T = A_IJ - sum_{k < J} L_Ik L_Jk^T,   L_IJ = T L_JJ^-T
// Task of block column J's diagonal: the same for tile (J, J - 1), then
//     T = A_JJ - sum_{k < J - 1} L_Jk L_Jk^T - L_{J,J-1} L_{J,J-1}^T,   L_JJ = chol(T),
// so that from one diagonal factor to the next only one flag crosses compute units.
//
// Every product is v_mfma_f64_16x16x4 on fragments straight from device memory: a finished tile is
// stored packed (32 KB) in the instruction's operand order, rows l % 16 and k = l / 16 of lane l, two
// steps of 4 columns per 16-byte load. A and B operands have the same order, so one copy serves
// both. The sums are kept transposed (T^T): their register layout is the B operand's, and the
// panel solve X_p^T = D_p T_p^T, T_q^T -= L_qp X_p^T runs from registers with no LDS transposition.
//
// Flags: ready[I * nb + J], one byte per 16-row strip (for a diagonal tile: per 16-column panel). A
// wave stores its strip with agent-scope write-through stores, waits for them, then stores its byte;
// a reader polls the bytes with agent-scope loads before it loads the strip. The strip's lines are
// whole 128-byte lines that nobody has read before in this launch, so its plain loads cannot hit a
// stale line of its own L2 (caches are invalidated at the start of a launch). A workgroup takes its
// task by a ticket, in an order in which every task depends on earlier tickets only: whatever part
// of the grid is resident, the oldest unfinished task can always run. Waits are bounded all the same:
// past the bound a wave raises ticket[1], which ends every wait, and the matrix's status reads -1.
#include "dfisher_internal.h"

#include <algorithm>

namespace dfi {
namespace {

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int NB = 64;              // tile edge
constexpr int TD = NB * NB;         // doubles of a packed tile
constexpr uint32_t FULL = 0x01010101u;
constexpr int SPIN_MAX = 1 << 22;   // polls of a wait (seconds; a wait is microseconds)
// What a diagonal tile's last panel holds until it is stored: a signalling NaN, which no arithmetic gives.
constexpr uint64_t UNSET = 0x7FF4D15EA5ED0001ull;
constexpr int LAST_AT = 3840;       // doubles of a packed tile before that panel's 256
constexpr int LDD = 17;             // padded row of a 16 x 16 block in LDS (doubles)
constexpr int AUX_SC1 = 16;         // cache policy of a buffer store: agent scope, write through

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

__device__ __forceinline__ uint32_t load_agent(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Fragment pair (row block rb, columns 8 kp .. 8 kp + 7) of a packed tile: lane l holds rows
// 16 rb + l % 16, columns 8 kp + l / 16 and 8 kp + 4 + l / 16.
__device__ __forceinline__ int frag_at(int rb, int kp, int lane) { return ((rb * 8 + kp) * 64 + lane) * 2; }
__device__ __forceinline__ f64x2 frag_load(const double* tile, int rb, int kp, int lane) {
  return *reinterpret_cast<const f64x2*>(tile + frag_at(rb, kp, lane));
}
__device__ __forceinline__ void frag_store(double* tile, int rb, int kp, int lane, f64x2 v) {
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(tile, 0, TD * 8, 0x00020000);
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs, frag_at(rb, kp, lane) * 8, 0, AUX_SC1);
}

// This wave's earlier stores have reached memory; then its byte of the flag word.
__device__ __forceinline__ void publish(uint32_t* word, int byte, int lane) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (lane == 0)
    __hip_atomic_store(reinterpret_cast<uint8_t*>(word) + byte, (uint8_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One more poll of a wait: false once the wait has to end (bound reached, or another wave gave up).
__device__ __forceinline__ bool keep_waiting(int& spins, uint32_t* ticket, int lane) {
  if (++spins > SPIN_MAX) {
    if (lane == 0) __hip_atomic_store(ticket + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return false;
  }
  if ((spins & 255) == 0 && load_agent(ticket + 1) != 0) return false;
  __builtin_amdgcn_s_sleep(1);
  return true;
}

// Waits until tiles k0 of both rows are finished; returns how many consecutive k from k0 (< kend)
// are (lane l looks at k0 + l, so a late task learns of up to 64 finished tiles in one poll). 0: gave up.
__device__ __forceinline__ int wait_tiles(const uint32_t* rowI, const uint32_t* rowJ, int k0, int kend,
                                          uint32_t* ticket, int lane) {
  const int k = k0 + lane;
  int spins = 0;
  for (;;) {
    bool ok = false;
    if (k < kend) {
      const uint32_t a = load_agent(rowI + k), b = load_agent(rowJ + k);
      ok = a == FULL && b == FULL;
    }
    const uint64_t mask = __ballot(ok);
    if (mask & 1) {
      asm volatile("" ::: "memory");   // the tiles' loads stay behind the poll
      return mask == ~0ull ? 64 : __builtin_ctzll(~mask);
    }
    if (!keep_waiting(spins, ticket, lane)) return 0;
  }
}

// Waits for panel p of a diagonal tile; `seen` keeps the flag word of the last poll, so panels that were
// finished by then are not polled for again.
__device__ __forceinline__ bool wait_panel(uint32_t& seen, const uint32_t* word, int p, uint32_t* ticket, int lane) {
  int spins = 0;
  while (((seen >> (8 * p)) & 0xFFu) == 0) {
    seen = __builtin_amdgcn_readfirstlane(load_agent(word));
    if (((seen >> (8 * p)) & 0xFFu) == 0 && !keep_waiting(spins, ticket, lane)) return false;
  }
  asm volatile("" ::: "memory");
  return true;
}

// The last panel of a diagonal tile (D_3), the one every next diagonal factor waits for: its values are
// polled themselves, which saves the wait for the stores before a flag and the load after it (0.9 us of
// a step). On a wait that gave up f is whatever was read last.
__device__ __forceinline__ bool wait_last(f64x2 (&f)[2], const double* tile, uint32_t* ticket, int lane) {
  const uint64_t* src = reinterpret_cast<const uint64_t*>(tile + LAST_AT) + 2 * lane;
  int spins = 0;
  for (;;) {
    uint64_t v[4];
#pragma unroll
    for (int h = 0; h < 4; ++h)
      v[h] = __hip_atomic_load(src + 128 * (h >> 1) + (h & 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool ok = v[0] != UNSET && v[1] != UNSET && v[2] != UNSET && v[3] != UNSET;
#pragma unroll
    for (int h = 0; h < 4; ++h) f[h >> 1][h & 1] = __longlong_as_double((long long)v[h]);
    if (__ballot(ok) == ~0ull) return true;
    if (!keep_waiting(spins, ticket, lane)) return false;
  }
}

// acc[p] += L_J[16 p ..][k] L_I[16 w ..][k]^T, p < NP, over cnt packed tiles from tj (row J) and ti (row I):
// per 8 columns five 16-byte loads and eight products, three groups of loads in flight ahead of the
// products (one takes 512 cycles of the matrix core). The last loads repeat the last group.
template <int NP>
__device__ __forceinline__ void accumulate(f64x4 (&acc)[4], const double* tj, const double* ti, int cnt, int w, int lane) {
  const int groups = cnt * 8;
  if (groups == 0) return;
  f64x2 a[4][NP], b[4];
  auto load = [&](int slot, int g) {
    g = min(g, groups - 1);
    const double* aj = tj + (int64_t)(g >> 3) * TD;
    const double* bi = ti + (int64_t)(g >> 3) * TD;
#pragma unroll
    for (int p = 0; p < NP; ++p) a[slot][p] = frag_load(aj, p, g & 7, lane);
    b[slot] = frag_load(bi, w, g & 7, lane);
  };
  load(0, 0);
  load(1, 1);
  load(2, 2);
  for (int g0 = 0; g0 < groups; g0 += 4) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      load((s + 3) & 3, g0 + s + 3);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int p = 0; p < NP; ++p) acc[p] = mfma(a[s][p][h], b[s][h], acc[p]);
    }
  }
}

// x's four 16-lane rows, each broadcast to all four: y[g] in lane l = x in lane 16 g + l % 16.
__device__ __forceinline__ void gather_rows(double x, double (&y)[4]) {
  const uint64_t b = __double_as_longlong(x);
  uint32_t o[4][2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t v = (uint32_t)(b >> (32 * h));
    const auto s = __builtin_amdgcn_permlane16_swap(v, v, false, false);          // rows 0 0 2 2 | 1 1 3 3
    const auto even = __builtin_amdgcn_permlane32_swap(s[0], s[0], false, false);   // 0 0 0 0 | 2 2 2 2
    const auto odd = __builtin_amdgcn_permlane32_swap(s[1], s[1], false, false);
    o[0][h] = even[0];
    o[1][h] = odd[0];
    o[2][h] = even[1];
    o[3][h] = odd[1];
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) y[g] = __longlong_as_double((long long)(((uint64_t)o[g][1] << 32) | o[g][0]));
}

// A diagonal entry of W below this may leave a pivot whose reciprocal overflows (2^-1024): factor16 then gets the block with
// every row and column scaled by a power of two (scale16), which is exact and taken off its results again. The entries are
// looked at before a task's waits, so that the chain of pivots carries nothing of it.
constexpr double SMALL_DIAG = 0x1p-900;
__device__ __forceinline__ int row_exponent(const f64x4& t, int lane) {   // half of T[r][r]'s, 0 unless it is > 0
  const int r = lane & 15;
  double d = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double v = __shfl(t[q], 16 * (r & 3) + r, 64);
    if ((r >> 2) == q) d = v;
  }
  return d > 0.0 && d < __builtin_inf() ? __builtin_amdgcn_frexp_exp(d) >> 1 : 0;
}
__device__ __forceinline__ void scale16(f64x4& t, int k, int lane) {   // k: the row's exponent
#pragma unroll
  for (int q = 0; q < 4; ++q) t[q] = __builtin_ldexp(t[q], -k - __shfl(k, 4 * q + (lane >> 4), 64));
}

// 1 / d and 1 / sqrt(d) of a normal d > 0: the hardware estimate (relative error e of about 2^-23) and
// one third-order step, error e^3.
__device__ __forceinline__ double recip(double d) {
  const double y = __builtin_amdgcn_rcp(d);
  const double e = fma(-d, y, 1.0);
  return fma(y * e, 1.0 + e, y);
}
__device__ __forceinline__ double recip_sqrt(double d) {
  const double y = __builtin_amdgcn_rsq(d);
  const double e = fma(-d * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// 1-based index of the first of 16 pivots (lane 16 g, register q: pivot 4 q + g) that is not > 0, 0 if none.
__device__ __forceinline__ int piv_bad(const double (&piv)[4]) {
  int bad = 0;
#pragma unroll
  for (int q = 3; q >= 0; --q) {
    const uint64_t m = __ballot(!(piv[q] > 0.0));
    if (m) bad = 4 * q + (int)(__builtin_ctzll(m) >> 4) + 1;
  }
  return bad;
}

// One wave's factor of a 16 x 16 block: T = L L^T and D = L^-1. t: T in the sums' layout (lane 16 g + r,
// register q: T[r][4 q + g]; entries above the diagonal are never used). l: L in the same layout
// (garbage above the diagonal). d[q] in lane 16 g + r: D[4 q + g][r]. piv[q] in lane 16 g + r: the
// pivot of column 4 q + g.
// Bound by the chain of 16 pivots. Four columns at a time: the 4 x 4 pivot block is read into every
// lane, which eliminates it redundantly (a pivot costs its reciprocal, a product and a difference,
// 53 cycles; the square roots stay off the chain) and with it its own row's four columns; the columns
// after them lose W diag(1 / d) W^T in one matrix instruction of depth 4. An identity block below T
// goes through the same steps and ends as D^T. About 1.9k cycles, against 5-7k for column by column
// with each multiplier read across lanes.
__device__ __forceinline__ void factor16(f64x4 t, f64x4& l, f64x4& d, double (&piv)[4], int lane) {
  const int g = lane >> 4, r = lane & 15;
  f64x4 e;
#pragma unroll
  for (int q = 0; q < 4; ++q) e[q] = (r == 4 * q + g) ? 1.0 : 0.0;
  auto pick = [&](double a, double b, double c, double f) {   // entry g of four
    const double lo = (g & 1) ? b : a, hi = (g & 1) ? f : c;
    return (g & 2) ? hi : lo;
  };
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    double p[4][4], m[4][4], rd[4], y[4], z[4];   // pivot block, unit multipliers, reciprocals, the rows
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = j; i < 4; ++i) p[i][j] = lane_read(t[q], 16 * j + 4 * q + i);
    gather_rows(t[q], y);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      rd[j] = recip(p[j][j]);
#pragma unroll
      for (int i = j + 1; i < 4; ++i) {
        m[i][j] = p[i][j] * rd[j];
#pragma unroll
        for (int c = j + 1; c <= i; ++c) p[i][c] = fma(-m[i][j], p[c][j], p[i][c]);
      }
#pragma unroll
      for (int i = j + 1; i < 4; ++i) y[i] = fma(-m[i][j], y[j], y[i]);
    }
    const double wy = pick(y[0], y[1], y[2], y[3]);
    const double a = -wy * pick(rd[0], rd[1], rd[2], rd[3]);
    if (q < 3) t = mfma(a, wy, t);
    __builtin_amdgcn_sched_barrier(0);   // the rest runs while the matrix core is busy
    gather_rows(e[q], z);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = j + 1; i < 4; ++i) z[i] = fma(-m[i][j], z[j], z[i]);
    const double wz = pick(z[0], z[1], z[2], z[3]);
    if (q < 3) e = mfma(a, wz, e);
    piv[q] = pick(p[0][0], p[1][1], p[2][2], p[3][3]);
    const double ws = recip_sqrt(piv[q]);
    l[q] = wy * ws;
    d[q] = wz * ws;
  }
}

// -W_IJ (with add on the diagonal) of this wave's strip (rows 64 I + 16 w ..), transposed sums' layout: lane l, register q of
// block p holds row l % 16, column 16 p + l / 16 + 4 q. Rows past n are zero; on the diagonal tile the
// strict upper triangle is zero and rows past n are the identity's.
__device__ __forceinline__ void load_strip(f64x4 (&acc)[4], const double* W, double add, int64_t n, int I, int J, int w,
                                           int lane) {
  const int64_t row = (int64_t)I * NB + 16 * w + (lane & 15);
  const double* ar = W + (row < n ? row : n - 1) * n;
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t col = (int64_t)J * NB + 16 * p + (lane >> 4) + 4 * q;
      const double v = ar[col < n ? col : n - 1] + (row == col ? add : 0.0);
      acc[p][q] = (row >= n) ? (row == col ? -1.0 : 0.0) : (col > row ? 0.0 : -v);
    }
}

// X L_JJ^T = T by panels, X_p^T = D_p T_p^T, then T_q^T -= L_qp X_p^T for the later ones, from the packed
// diagonal tile (D_p on its diagonal) whose panels are flagged one by one (the last is its own flag).
// done(p, -X_p^T) follows each
// panel; T[p] is X_p^T by then. When the first three panels are there at the first poll (a late task)
// their loads go out together. Returns false when a wait gave up.
template <class Done>
__device__ __forceinline__ bool solve_strip(f64x4 (&T)[4], const double* tile, const uint32_t* word, uint32_t* ticket,
                                            int lane, Done done) {
  f64x2 f[4][4][2];   // [p][q][h]
  uint32_t seen = 0;
  bool ok = wait_panel(seen, word, 0, ticket, lane);
  auto load = [&](int p) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q >= p)
#pragma unroll
        for (int h = 0; h < 2; ++h) f[p][q][h] = frag_load(tile, q, 2 * p + h, lane);
  };
  const bool late = (seen & 0x010101u) == 0x010101u;
  load(0);
  if (late) {
    load(1);
    load(2);
  }
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    if (p == 3) {
      if (ok) ok = wait_last(f[3][3], tile, ticket, lane);
    } else if (p > 0 && !late) {
      if (ok) ok = wait_panel(seen, word, p, ticket, lane);
      load(p);
    }
    f64x4 x = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int h = 0; h < 4; ++h) x = mfma(f[p][p][h >> 1][h & 1], T[p][h], x);
    const f64x4 xn = -x;
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
      for (int q = 1; q < 4; ++q)
        if (q > p) T[q] = mfma(f[p][q][h >> 1][h & 1], xn[h], T[q]);
    T[p] = x;
    done(p, xn);
  }
  return ok;
}

// The finished strip of an off-diagonal tile into the row-major factor, and mirrored above the diagonal
// (the triangular solves read both).
__device__ __forceinline__ void store_strip(const f64x4 (&T)[4], double* A, int64_t n, int I, int J, int w, int lane) {
  const int64_t row = (int64_t)I * NB + 16 * w + (lane & 15);
  if (row >= n) return;
  double* ar = A + row * n + (int64_t)J * NB + (lane >> 4);
  double* at = A + ((int64_t)J * NB + (lane >> 4)) * n + row;
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      ar[16 * p + 4 * q] = T[p][q];
      at[(int64_t)(16 * p + 4 * q) * n] = T[p][q];
    }
}

struct CholLds {
  double x[TD];   // L_{J,J-1} in fragment order
  double l[TD];   // the blocks of L_JJ below its 16 x 16 diagonal blocks in fragment order
  double d[4][16 * LDD];   // D_p, row-major
  int have_x[4];      // strip w of x is there
  int have_l[4][4];   // block (q, p) of l is there
  int have_bad[4];    // wave w has looked at its pivots
  int bad;        // 1-based column of the block's first pivot that is not > 0, 0 if none
};

__device__ __forceinline__ f64x2 lds_frag(const double* f, int rb, int kp, int lane) {
  return *reinterpret_cast<const f64x2*>(f + frag_at(rb, kp, lane));
}

// A block of the sums' layout (X^T of a 16-row strip) into the strip's fragments of panel p.
__device__ __forceinline__ void put_frags(double* f, int rb, int p, int lane, const f64x4& x) {
#pragma unroll
  for (int h = 0; h < 2; ++h) *reinterpret_cast<f64x2*>(f + frag_at(rb, 2 * p + h, lane)) = (f64x2){x[2 * h], x[2 * h + 1]};
}

// t -= L_rb,p X^T (K = 16): xn = -X^T in the sums' layout, L_rb,p from LDS.
__device__ __forceinline__ void sub_product(f64x4& t, const double* f, int rb, int p, int lane, const f64x4& xn) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const f64x2 a = lds_frag(f, rb, 2 * p + h, lane);
    t = mfma(a[0], xn[2 * h], t);
    t = mfma(a[1], xn[2 * h + 1], t);
  }
}

// A wait ended without its tile: the matrix's status says so.
__device__ __forceinline__ void gave_up(int64_t* info, int32_t* flag, int lane) {
  if (lane == 0) {
    __hip_atomic_store(info, (int64_t)-1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Between the waves of a diagonal task: LDS words instead of barriers, so that only the waves that need
// a block wait for it. (A wave's LDS operations are done in order: the word after its data.)
__device__ __forceinline__ void have(int* word) {
  asm volatile("" ::: "memory");
  __hip_atomic_store(word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void await(int* word) {   // every wave of the task reaches its have()s
  while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) == 0) {
  }
  asm volatile("" ::: "memory");
}

// The diagonal task of block column J (see the head of this file). Wave w holds its 16 rows' blocks
// 0 .. w in registers. Panel p of the factor: wave p factors its diagonal block (factor16) and puts
// D_p = L_pp^-1 in LDS; the later waves form X_wp^T = D_p T_wp^T, subtract X_wp X_wp^T from their own
// diagonal block (both operands are the same registers) and, as the other waves' X appear in LDS, the
// products with those from their other blocks. The chain from wave p to wave p + 1 is thus one LDS
// round trip and eight products; everything else is kept behind it, the stores and flags above all. A panel is published as soon as it is finished, so
// the tasks that wait for it solve their panels 0 .. 2 while the later ones are still being factored.
__device__ void diag_task(double* A, const double* W, double add, int64_t n, int J, int nb, double* pack, uint32_t* ready, int64_t* info, int32_t* flag,
                          uint32_t* ticket, CholLds& sm, int w, int lane) {
  const double* rowJ = pack + (int64_t)J * (J + 1) / 2 * TD;
  uint32_t* fJ = ready + (int64_t)J * nb;
  double* tileJ = const_cast<double*>(rowJ) + (int64_t)J * TD;
  if (threadIdx.x < 4) sm.have_x[threadIdx.x] = sm.have_bad[threadIdx.x] = 0;
  if (threadIdx.x < 16) sm.have_l[threadIdx.x >> 2][threadIdx.x & 3] = 0;
  f64x4 t1[4], t2[4];
  load_strip(t2, W, add, n, J, J, w, lane);
  const int64_t own = min<int64_t>((int64_t)J * NB + 16 * w + (lane & 15), n - 1);
  const double own_diag = W[own * n + own] + add;
  __builtin_amdgcn_s_setprio(3);   // ahead of the tile task that shares the compute unit's matrix cores
  __syncthreads();
  bool small = false;
  if (J == 0) small = __ballot(own_diag > 0.0 && own_diag < SMALL_DIAG) != 0;
  if (J > 0) {
    bool ok = true;
    const double* rowP = pack + (int64_t)(J - 1) * J / 2 * TD;
    const uint32_t* fP = ready + (int64_t)(J - 1) * nb;
    double* tileX = const_cast<double*>(rowJ) + (int64_t)(J - 1) * TD;
    load_strip(t1, W, 0.0, n, J, J - 1, w, lane);
    for (int k = 0; k < J - 1;) {
      const int cnt = wait_tiles(fJ, fP, k, J - 1, ticket, lane);
      if (cnt == 0) {
        ok = false;
        break;
      }
      const double* tp = rowP + (int64_t)k * TD;
      const double* tj = rowJ + (int64_t)k * TD;
      accumulate<4>(t1, tp, tj, cnt, w, lane);
      k += cnt;
      if (w == 0) accumulate<1>(t2, tj, tj, cnt, w, lane);   // the blocks of the lower triangle
      else if (w == 1) accumulate<2>(t2, tj, tj, cnt, w, lane);
      else if (w == 2) accumulate<3>(t2, tj, tj, cnt, w, lane);
      else accumulate<4>(t2, tj, tj, k == J - 1 ? cnt - 1 : cnt, w, lane);   // its last tile below
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) t1[p] = -t1[p];
    small = __ballot(own_diag > 0.0 && own_diag < SMALL_DIAG) != 0;
    // own rows of L_{J,J-1}, panel by panel
    const bool solved = solve_strip(t1, rowP + (int64_t)(J - 1) * TD, fP + (J - 1), ticket, lane,
                                    [&](int p, const f64x4& xn) {
      put_frags(sm.x, w, p, lane, t1[p]);
      if (w == 1 || w == 2)
#pragma unroll
        for (int h = 0; h < 2; ++h) frag_store(tileX, w, 2 * p + h, lane, (f64x2){t1[p][2 * h], t1[p][2 * h + 1]});
#pragma unroll
      for (int q = 0; q < 4; ++q)   // (t2 still has the other sign)
        if (q == w)
#pragma unroll
          for (int h = 0; h < 4; ++h) t2[q] = mfma(t1[p][h], t1[p][h], t2[q]);
    });
    have(&sm.have_x[w]);
    if (!ok || !solved) gave_up(info, flag, lane);
    // Wave 2 has the fewest sums left before its turn: it stores the strips of wave 0, which goes on with
    // the factor, and of wave 3, whose last sums come only now (before, they would hold up the strips
    // that the next block column waits for).
    if (w == 2) {
#pragma unroll
      for (int q = 0; q < 4; q += 3) {
        await(&sm.have_x[q]);
#pragma unroll
        for (int h = 0; h < 8; ++h) frag_store(tileX, q, h, lane, lds_frag(sm.x, q, h, lane));
      }
      publish(fJ + (J - 1), 2, lane);
      publish(fJ + (J - 1), 0, lane);
      publish(fJ + (J - 1), 3, lane);
    }
    if (w == 3 && ok && J > 1) {
      const double* tj = rowJ + (int64_t)(J - 2) * TD;
      accumulate<4>(t2, tj, tj, 1, w, lane);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q)
      if (q < w) {
        await(&sm.have_x[q]);
#pragma unroll
        for (int p = 0; p < 4; ++p) sub_product(t2[q], sm.x, q, p, lane, t1[p]);
      }
    if (w == 1) publish(fJ + (J - 1), 1, lane);
  }
#pragma unroll
  for (int p = 0; p < 4; ++p) t2[p] = -t2[p];
  // a block of the sums' layout (rows 16 w .., columns 16 p ..) of the row-major factor
  auto store_block = [&](int p, const f64x4& x) {
    const int64_t row = (int64_t)J * NB + 16 * w + (lane & 15);
    if (row >= n) return;
    double* ar = A + row * n + (int64_t)J * NB + 16 * p + (lane >> 4);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (p < w || (lane >> 4) + 4 * q <= (lane & 15)) ar[4 * q] = x[q];
  };
  f64x4 td = t2[0];   // this wave's diagonal block
  if (w == 1) td = t2[1];
  if (w == 2) td = t2[2];
  if (w == 3) td = t2[3];
  // L_wp for the panels before this wave's, then its own
  f64x4 xl = td;   // X_{w,w-1}, stored after the factor
#pragma unroll 1
  for (int p = 0; p < w; ++p) {
    f64x4 tp = t2[0];
    if (p == 1) tp = t2[1];
    if (p == 2) tp = t2[2];
    await(&sm.have_l[p][p]);
    f64x4 x = (f64x4){0.0, 0.0, 0.0, 0.0};
    const double* dp = &sm.d[p][(lane & 15) * LDD + (lane >> 4)];
#pragma unroll
    for (int h = 0; h < 4; ++h) x = mfma(dp[4 * h], tp[h], x);
    const f64x4 xn = -x;
#pragma unroll
    for (int h = 0; h < 4; ++h) td = mfma(x[h], xn[h], td);
    put_frags(sm.l, w, p, lane, x);
    have(&sm.have_l[w][p]);
    if (p + 1 == w) {
      xl = x;
    } else {
#pragma unroll
      for (int q = 1; q < 3; ++q)
        if (q > p && q < w) {
          await(&sm.have_l[q][p]);
          sub_product(t2[q], sm.l, q, p, lane, xn);
        }
      store_block(p, x);
    }
  }
  f64x4 lw, dw;
  double piv[4];
  int k = 0;
  if (small) {
    k = row_exponent(td, lane);
    scale16(td, k, lane);
  }
  factor16(td, lw, dw, piv, lane);
  if (small)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      lw[q] = __builtin_ldexp(lw[q], k);
      dw[q] = __builtin_ldexp(dw[q], -k);
    }
#pragma unroll
  for (int q = 0; q < 4; ++q) sm.d[w][((lane >> 4) + 4 * q) * LDD + (lane & 15)] = dw[q];
  have(&sm.have_l[w][w]);
  // The first breakdown of the matrix is reported; what follows runs on garbage. (sm.bad goes from wave
  // to wave with the factor, the status from block column to block column with the last panel.)
  const int bad = piv_bad(piv);
  if (w == 0) {
    if (lane == 0) sm.bad = bad;
    have(&sm.have_bad[0]);
  } else {
    await(&sm.have_bad[w - 1]);
    if (lane == 0 && bad != 0 && sm.bad == 0) sm.bad = 16 * w + bad;
    have(&sm.have_bad[w]);
  }
  if (w == 3) {
    if (__builtin_amdgcn_readfirstlane(sm.bad) != 0) {
      if (lane == 0 && load_agent(reinterpret_cast<uint32_t*>(flag)) == 0) {
        __hip_atomic_store(info, (int64_t)J * NB + sm.bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
  }
  const double* dp = &sm.d[w][(lane & 15) * LDD + (lane >> 4)];
#pragma unroll
  for (int h = 0; h < 2; ++h) frag_store(tileJ, w, 2 * w + h, lane, (f64x2){dp[8 * h], dp[8 * h + 4]});
#pragma unroll
  for (int q = 1; q < 4; ++q)
    if (q > w) {
      await(&sm.have_l[q][w]);
#pragma unroll
      for (int h = 0; h < 2; ++h) frag_store(tileJ, q, 2 * w + h, lane, lds_frag(sm.l, q, 2 * w + h, lane));
    }
  if (w < 3) publish(fJ + J, w, lane);
  store_block(w, lw);
  if (w > 0) store_block(w - 1, xl);
  if (J > 0) store_strip(t1, A, n, J, J - 1, w, lane);
}

// The off-diagonal task of tile (I, J), I >= J + 2.
__device__ void tile_task(double* A, const double* W, int64_t n, int I, int J, int nb, double* pack, uint32_t* ready, int64_t* info,
                          int32_t* flag, uint32_t* ticket, int w, int lane) {
  const double* rowI = pack + (int64_t)I * (I + 1) / 2 * TD;
  const double* rowJ = pack + (int64_t)J * (J + 1) / 2 * TD;
  uint32_t* fI = ready + (int64_t)I * nb;
  const uint32_t* fJ = ready + (int64_t)J * nb;
  f64x4 t[4];
  load_strip(t, W, 0.0, n, I, J, w, lane);
  for (int k = 0; k < J;) {
    const int cnt = wait_tiles(fI, fJ, k, J, ticket, lane);
    if (cnt == 0) return gave_up(info, flag, lane);
    accumulate<4>(t, rowJ + (int64_t)k * TD, rowI + (int64_t)k * TD, cnt, w, lane);
    k += cnt;
  }
#pragma unroll
  for (int p = 0; p < 4; ++p) t[p] = -t[p];
  double* tile = const_cast<double*>(rowI) + (int64_t)J * TD;
  if (!solve_strip(t, rowJ + (int64_t)J * TD, fJ + J, ticket, lane, [&](int p, const f64x4&) {
#pragma unroll
        for (int h = 0; h < 2; ++h) frag_store(tile, w, 2 * p + h, lane, (f64x2){t[p][2 * h], t[p][2 * h + 1]});
      }))
    return gave_up(info, flag, lane);
  publish(fI + J, w, lane);
  store_strip(t, A, n, I, J, w, lane);
}

// Tasks of one matrix of nb block rows, in ticket order: diagonal 0, then for c = 1 .. nb - 1
// diagonal c (with tile (c, c - 1)) followed by the tiles (c + 1 .. nb - 1, c - 1).
__host__ __device__ inline int64_t chol_tasks(int64_t nb) { return 1 + nb * (nb - 1) / 2; }

// nbatch matrices (matrix b at A + b sA, pack + b sP, ready + b sR; with src.W all read src.W, its diagonal shifted by
// each matrix's own term, and A is only written): ticket t is task t / nbatch of
// matrix t % nbatch. With jobs / tasks: ticket t is entry t of the task table. 256 threads; two
// workgroups per compute unit (74 KB of its 160 KB of LDS each, at most 256 registers).
__global__ void __launch_bounds__(256, 2)
chol_kernel(double* A, int64_t n, int64_t sA, double* pack, int64_t sP, uint32_t* ready, int64_t sR, int64_t* info,
            int32_t* flag, uint32_t* ticket, int nbatch, const FactorJob* __restrict__ jobs,
            const FactorTask* __restrict__ tasks, CholSource src) {
  __shared__ CholLds sm;
  __shared__ uint32_t my;
  if (threadIdx.x == 0) my = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const uint32_t tk = __builtin_amdgcn_readfirstlane(my);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int c, i, nb;
  const double* W = src.W;
  double add = 0.0;
  if (tasks) {
    const FactorTask t = tasks[tk];
    const FactorJob& j = jobs[t.job];
    A = j.A;
    n = j.n;
    info = j.info;
    flag = j.flag;
    pack = j.pack;
    ready = j.ready;
    nb = (int)((n + NB - 1) / NB);
    c = t.c;
    i = t.i;
  } else {
    const int b = (int)(tk % (uint32_t)nbatch);
    const int s = (int)(tk / (uint32_t)nbatch);
    A += b * sA;
    if (W) add = src.lam[b] + (src.scale != 0.0 ? src.scale * src.dmax[0] : 0.0);
    pack += b * sP;
    ready += b * sR;
    info += b;
    flag += b;
    nb = (int)((n + NB - 1) / NB);
    c = i = 0;
    if (s > 0) {   // column group c has nb - c tasks: counted from the end, groups of 1, 2, 3, ...
      const int total = nb * (nb - 1) / 2;
      const int rem = total - s;
      int j = (int)((sqrt(8.0 * (double)rem + 1.0) - 1.0) * 0.5);
      while ((j + 1) * (j + 2) / 2 <= rem) ++j;
      while (j * (j + 1) / 2 > rem) --j;
      c = nb - 1 - j;
      i = (s - 1) - (total - (j + 1) * (j + 2) / 2);
    }
  }
  c = __builtin_amdgcn_readfirstlane(c);
  i = __builtin_amdgcn_readfirstlane(i);
  if (!W) W = A;
  if (i == 0) diag_task(A, W, add, n, c, nb, pack, ready, info, flag, ticket, sm, w, lane);
  else tile_task(A, W, n, c + i, c - 1, nb, pack, ready, info, flag, ticket, w, lane);
}

// Statuses, flags and the ticket start at zero, the diagonal tiles' last panels unset. Grid (x, y): y = matrix.
__global__ void chol_clear_kernel(int64_t n, double* pack, int64_t sP, uint32_t* ready, int64_t sR, int64_t* info,
                                  int32_t* flag, uint32_t* ticket, const FactorJob* __restrict__ jobs) {
  const int64_t b = blockIdx.y;
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (jobs) {
    n = jobs[b].n;
    pack = jobs[b].pack;
    ready = jobs[b].ready;
    info = jobs[b].info;
    flag = jobs[b].flag;
  } else {
    pack += b * sP;
    ready += b * sR;
    info += b;
    flag += b;
  }
  const int64_t nb = (n + NB - 1) / NB;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = x; e < nb * nb; e += step) ready[e] = 0;
  for (int64_t e = x; e < nb * (TD - LAST_AT); e += step) {   // the last panels of the diagonal tiles
    const int64_t j = e / (TD - LAST_AT);
    reinterpret_cast<uint64_t*>(pack)[((j + 1) * (j + 2) / 2 - 1) * TD + LAST_AT + e % (TD - LAST_AT)] = UNSET;
  }
  if (x == 0) {
    *info = 0;
    *flag = 0;
    if (b == 0) ticket[0] = ticket[1] = 0;
  }
}

size_t ready_bytes(int64_t nb) { return ((size_t)(nb * nb) * 4 + 255) / 256 * 256; }

}  // namespace

size_t chol_pack_bytes(int64_t n) {
  const int64_t nb = (n + NB - 1) / NB;
  return (size_t)(nb * (nb + 1) / 2) * TD * sizeof(double) + ready_bytes(nb);
}

int64_t chol_task_count(int64_t n) { return chol_tasks((n + NB - 1) / NB); }

uint32_t* chol_ready_at(double* pack, int64_t n) {
  const int64_t nb = (n + NB - 1) / NB;
  return reinterpret_cast<uint32_t*>(pack + nb * (nb + 1) / 2 * TD);
}

hipError_t chol_launch_batched(double* A, int64_t n, int64_t nbatch, int64_t sA, int64_t* info_dev, int32_t* flag_dev,
                               double* pack, uint32_t* ticket, hipStream_t st, const CholSource& src) {
  if (src.W && nbatch > CHOL_LAMS) return hipErrorInvalidValue;
  const int64_t nb = (n + NB - 1) / NB;
  const int64_t wgs = chol_tasks(nb) * nbatch;
  if (n < 1 || nbatch < 1 || nbatch > 65535 || wgs > 0x7FFFFFFF) return hipErrorInvalidValue;
  const int64_t sP = (int64_t)(chol_pack_bytes(n) / sizeof(double));
  uint32_t* ready = chol_ready_at(pack, n);
  const FactorJob* nj = nullptr;
  hipLaunchKernelGGL(chol_clear_kernel, dim3((unsigned)std::min<int64_t>(32, nb), (unsigned)nbatch), dim3(256), 0, st,
                     n, pack, sP, ready, 2 * sP, info_dev, flag_dev, ticket, nj);
  hipLaunchKernelGGL(chol_kernel, dim3((unsigned)wgs), dim3(256), 0, st, A, n, sA, pack, sP, ready, 2 * sP, info_dev,
                     flag_dev, ticket, (int)nbatch, nj, (const FactorTask*)nullptr, src);
  return hipGetLastError();
}

hipError_t chol_launch_grouped(const FactorJob* jobs_dev, int64_t njobs, int64_t nmax, const FactorTask* tasks_dev,
                               int64_t ntasks, uint32_t* ticket, hipStream_t st) {
  if (njobs < 1 || njobs > 65535 || ntasks < 1 || ntasks > 0x7FFFFFFF) return hipErrorInvalidValue;
  const int64_t nb = (nmax + NB - 1) / NB;
  hipLaunchKernelGGL(chol_clear_kernel, dim3((unsigned)std::min<int64_t>(32, nb), (unsigned)njobs), dim3(256), 0, st,
                     (int64_t)0, (double*)nullptr, (int64_t)0, (uint32_t*)nullptr, (int64_t)0, (int64_t*)nullptr,
                     (int32_t*)nullptr, ticket, jobs_dev);
  hipLaunchKernelGGL(chol_kernel, dim3((unsigned)ntasks), dim3(256), 0, st, (double*)nullptr, (int64_t)0, (int64_t)0,
                     (double*)nullptr, (int64_t)0, (uint32_t*)nullptr, (int64_t)0, (int64_t*)nullptr,
                     (int32_t*)nullptr, ticket, 1, jobs_dev, tasks_dev, CholSource{});
  return hipGetLastError();
}

}  // namespace dfi
