// Gram W = S S^T + lambda I_n on the CDNA4 matrix cores (Algorithm 1 step 1; the O(n^2 m)
// term that dominates the cost of the method, Section 2).
//
// Work decomposition
//   * Only lower-triangle 256 x 256 tiles of W are computed (W is symmetric).
//   * The contraction dimension (m, the parameters) is split into k-slices. A work item is
//     (tile, slice); it accumulates S_I S_J^T over its slice in FP32 matrix-core accumulators
//     and stores the FP32 partial tile. gram_reduce then adds the slices in FP64 in a fixed
//     order (deterministic, and the FP32 error stays that of one slice).
//   * XCD-aware mapping: workgroups are dealt round-robin to the 8 XCDs, so workgroup w runs on
//     XCD w % 8. Each XCD gets its own run of work items in slice order, and consecutive workgroups
//     on an XCD take different tiles of the same slice: tiles that run together read the same
//     columns of S, which then come from that XCD's L2 instead of HBM.
//   * Each workgroup has 8 waves in a 2 x 4 layout; a wave owns a 128 x 64 sub-tile as
//     4 x 2 blocks of 32 x 32 MFMA accumulators (128 FP32 accumulators per lane).
//   * Per k-step, 32 columns of the row panels S_I and S_J are loaded from global memory into
//     registers (prefetched one step ahead) and written to LDS; for split-BF16 they are split
//     into hi/lo bf16 on the way. Diagonal tiles load one panel and use it twice.
//
// k-ordering inside a step: an MFMA consumes k-values that depend on the lane half h = lane/32.
// Both operands use the same assignment (half h takes columns 16h .. 16h+15 of the step), so
// every product S_ik S_jk is formed exactly once and the sum over k is unchanged.
#include "dfisher_internal.h"

#include <algorithm>
#include <type_traits>
#include <vector>

namespace dfi {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

constexpr int T = GRAM_TILE;      // 256
constexpr int KS = GRAM_KSTEP;    // 32
constexpr int WM = 2, WN = 4;             // wave grid inside the tile
constexpr int NTHR = 64 * WM * WN;        // 512
constexpr int BMW = T / WM, BNW = T / WN; // 128 x 64 per wave
constexpr int IM = BMW / 32, IN = BNW / 32;
constexpr int LOADS = T * KS / 4 / NTHR;  // float4 loads per thread per panel = 4
constexpr int ROWS_PER_LOAD = NTHR / (KS / 4);  // 64

// LDS row strides (elements). +16 bytes of padding per row keeps the 16-byte fragment reads
// of 16 consecutive rows on distinct bank groups.
constexpr int F32_STRIDE = KS + 4;    // 36 floats = 144 B
constexpr int BF_STRIDE = KS + 8;     // 40 bf16   = 80 B

__device__ __forceinline__ void tri_index(int64_t t, int64_t& ti, int64_t& tj) {
  // t -> (ti, tj), ti >= tj, t = ti (ti + 1) / 2 + tj
  int64_t r = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
  while ((r + 1) * (r + 2) / 2 <= t) ++r;
  while (r * (r + 1) / 2 > t) --r;
  ti = r;
  tj = t - r * (r + 1) / 2;
}

// A value the whole wave agrees on, moved to scalar registers. 64-bit division and the square
// root in tri_index expand to vector code, and without this everything derived from their
// results (column ranges, step counts, load addresses) would be computed per lane in the loops.
__device__ __forceinline__ int64_t uni64(int64_t x) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)x >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// The (slice, tile) work item of workgroup w: items in slice order, an eighth of them per XCD. False for
// the few workgroups past the last item (the count need not be a multiple of 8).
__host__ __device__ __forceinline__ int64_t items_per_xcd(int64_t ntri, int64_t nslice) { return (ntri * nslice + 7) >> 3; }
__device__ __forceinline__ bool work_item(int64_t w, int64_t ntri, int64_t nslice, int64_t& slice, int64_t& tile) {
  const int64_t per = items_per_xcd(ntri, nslice), local = w >> 3;
  const int64_t item = (w & 7) * per + local;
  if (local >= per || item >= ntri * nslice) return false;
  slice = uni64(item / ntri);
  tile = item - slice * ntri;
  return true;
}

// Whether the reduction reads anything of the 32 x 32 block at (row, col) of a tile (rows and columns of
// W below n, lower triangle): the others are not stored.
__device__ __forceinline__ bool block_used(bool diag, int64_t rowA, int64_t rowB, int row, int col, int64_t n) {
  return rowA + row < n && rowB + col < n && !(diag && col > row);
}

// Global -> register staging for one 256-row panel and one k-step.
// Thread t loads rows (t / 8) + 64 i, columns 4 (t % 8) .. +3 of the step.
template <bool VEC>
__device__ __forceinline__ void load_panel(const float* __restrict__ S, int64_t lds, int64_t n,
                                           int64_t row0, int64_t kcol, int64_t kend, f32x4 (&r)[LOADS]) {
  const int t = threadIdx.x;
  const int c = 4 * (t & 7);
  const int64_t col = kcol + c;
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int64_t row = row0 + (t >> 3) + ROWS_PER_LOAD * i;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (row < n) {
      const float* p = S + row * lds + col;
      if (VEC && col + 4 <= kend) {
        v = *reinterpret_cast<const f32x4*>(p);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (col + e < kend) v[e] = p[e];
      }
    }
    r[i] = v;
  }
}

template <int PREC>
struct Lds;

// FP32 operands: one panel of T rows x KS columns per operand.
template <>
struct Lds<0> {
  float a[T * F32_STRIDE];
  float b[T * F32_STRIDE];
};
// split-BF16 operands: hi and lo panels per operand.
template <>
struct Lds<1> {
  __bf16 ahi[T * BF_STRIDE];
  __bf16 alo[T * BF_STRIDE];
  __bf16 bhi[T * BF_STRIDE];
  __bf16 blo[T * BF_STRIDE];
};

__device__ __forceinline__ void store_f32(float* panel, const f32x4 (&r)[LOADS]) {
  const int t = threadIdx.x;
  const int c = 4 * (t & 7);
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int row = (t >> 3) + ROWS_PER_LOAD * i;
    *reinterpret_cast<f32x4*>(panel + row * F32_STRIDE + c) = r[i];
  }
}

__device__ __forceinline__ void store_bf16(__bf16* hi, __bf16* lo, const f32x4 (&r)[LOADS]) {
  const int t = threadIdx.x;
  const int c = 4 * (t & 7);
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int row = (t >> 3) + ROWS_PER_LOAD * i;
    bf16x4 h, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float a = r[i][e];
      const __bf16 hb = (__bf16)a;               // round to nearest even
      h[e] = hb;
      l[e] = (__bf16)(a - (float)hb);            // a - hi is exact in FP32
    }
    *reinterpret_cast<bf16x4*>(hi + row * BF_STRIDE + c) = h;
    *reinterpret_cast<bf16x4*>(lo + row * BF_STRIDE + c) = l;
  }
}

// Flip the sign bits of eight bf16 values when mask = 0x80008000 (identity for mask = 0).
__device__ __forceinline__ bf16x8 flip_sign(bf16x8 v, uint32_t mask) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 u = __builtin_bit_cast(u32x4, v);
  u ^= mask;
  return __builtin_bit_cast(bf16x8, u);
}

template <int PREC, bool VEC>
__global__ void __launch_bounds__(NTHR, 1)
gram_kernel(const float* __restrict__ S, int64_t n, int64_t lds, int64_t m, int64_t ntri,
            int64_t nslice, int64_t kslice, float* __restrict__ part) {
  __shared__ Lds<PREC> sm;

  int64_t slice, tile;
  if (!work_item(blockIdx.x, ntri, nslice, slice, tile)) return;
  // Alternating slice sign: on odd k-slices the A operand is negated and the stored partial tile negated back. The bf16
  // matrix-core accumulation shows a small sign-independent bias (low-order bits of the aligned addends are dropped toward
  // minus infinity); it is the same for +A and -A, so it cancels between even and odd slices instead of adding up
  // coherently over all entries (which would shift W along directions where many entries add, such as the all-ones
  // direction of a column-centered S).
  const float sgn = (slice & 1) ? -1.f : 1.f;
  const uint32_t bflip = (slice & 1) ? 0x80008000u : 0u;

  int64_t ti, tj;
  tri_index(tile, ti, tj);
  const bool diag = (ti == tj);
  const int64_t rowA = ti * T, rowB = tj * T;
  const int64_t k0 = slice * kslice;
  const int64_t kend = min(m, k0 + kslice);

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wr = wave / WN, wc = wave % WN;
  const int half = lane >> 5;
  const int l32 = lane & 31;
  // In a diagonal tile, wave sub-tiles that lie wholly above the diagonal idle.
  const bool active = !(diag && wc * BNW >= (wr + 1) * BMW);

  f32x16 acc[IM][IN];
#pragma unroll
  for (int i = 0; i < IM; ++i)
#pragma unroll
    for (int j = 0; j < IN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  const int64_t nsteps = (kend > k0) ? (kend - k0 + KS - 1) / KS : 0;
  f32x4 ra[LOADS], rb[LOADS];
  if (nsteps > 0) {
    load_panel<VEC>(S, lds, n, rowA, k0, kend, ra);
    if (!diag) load_panel<VEC>(S, lds, n, rowB, k0, kend, rb);
  }

  for (int64_t s = 0; s < nsteps; ++s) {
    __syncthreads();  // previous step's fragment reads are done
    if constexpr (PREC == 0) {
      store_f32(sm.a, ra);
      if (!diag) store_f32(sm.b, rb);
    } else {
      store_bf16(sm.ahi, sm.alo, ra);
      if (!diag) store_bf16(sm.bhi, sm.blo, rb);
    }
    __syncthreads();
    if (s + 1 < nsteps) {  // prefetch the next step while this one computes
      const int64_t kc = k0 + (s + 1) * KS;
      load_panel<VEC>(S, lds, n, rowA, kc, kend, ra);
      if (!diag) load_panel<VEC>(S, lds, n, rowB, kc, kend, rb);
    }
    if (!active) continue;

    if constexpr (PREC == 0) {
      const float* pa = sm.a;
      const float* pb = diag ? sm.a : sm.b;
#pragma unroll
      for (int kk = 0; kk < 16; kk += 8) {
        f32x4 fa[IM][2], fb[IN][2];
#pragma unroll
        for (int i = 0; i < IM; ++i) {
          const float* ra_ = pa + (wr * BMW + i * 32 + l32) * F32_STRIDE + half * 16 + kk;
          fa[i][0] = *reinterpret_cast<const f32x4*>(ra_);
          fa[i][1] = *reinterpret_cast<const f32x4*>(ra_ + 4);
        }
#pragma unroll
        for (int j = 0; j < IN; ++j) {
          const float* rb_ = pb + (wc * BNW + j * 32 + l32) * F32_STRIDE + half * 16 + kk;
          fb[j][0] = *reinterpret_cast<const f32x4*>(rb_);
          fb[j][1] = *reinterpret_cast<const f32x4*>(rb_ + 4);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
          for (int i = 0; i < IM; ++i)
#pragma unroll
            for (int j = 0; j < IN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(sgn * fa[i][e >> 2][e & 3], fb[j][e >> 2][e & 3],
                                                               acc[i][j], 0, 0, 0);
      }
    } else {
      const __bf16* ph = sm.ahi;
      const __bf16* pl = sm.alo;
      const __bf16* qh = diag ? sm.ahi : sm.bhi;
      const __bf16* ql = diag ? sm.alo : sm.blo;
#pragma unroll
      for (int kk = 0; kk < 16; kk += 8) {
        bf16x8 ah[IM], al[IM], bh[IN], bl[IN];
#pragma unroll
        for (int i = 0; i < IM; ++i) {
          const int oa = (wr * BMW + i * 32 + l32) * BF_STRIDE + half * 16 + kk;
          ah[i] = flip_sign(*reinterpret_cast<const bf16x8*>(ph + oa), bflip);
          al[i] = flip_sign(*reinterpret_cast<const bf16x8*>(pl + oa), bflip);
        }
#pragma unroll
        for (int j = 0; j < IN; ++j) {
          const int ob = (wc * BNW + j * 32 + l32) * BF_STRIDE + half * 16 + kk;
          bh[j] = *reinterpret_cast<const bf16x8*>(qh + ob);
          bl[j] = *reinterpret_cast<const bf16x8*>(ql + ob);
        }
#pragma unroll
        for (int i = 0; i < IM; ++i)
#pragma unroll
          for (int j = 0; j < IN; ++j) {
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[i], bh[j], acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bl[j], acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bh[j], acc[i][j], 0, 0, 0);
          }
      }
    }
  }

  // Store the FP32 partial tile (row-major T x T). 32x32 accumulator layout: lane l, register
  // r holds row 8 (r / 4) + 4 (l / 32) + (r % 4), column l % 32.
  float* out = part + (slice * ntri + tile) * (int64_t)(T * T);
#pragma unroll
  for (int i = 0; i < IM; ++i)
#pragma unroll
    for (int j = 0; j < IN; ++j)
      if (block_used(diag, rowA, rowB, wr * BMW + i * 32, wc * BNW + j * 32, n))
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = wr * BMW + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
        const int col = wc * BNW + j * 32 + l32;
        out[row * T + col] = sgn * acc[i][j][r];
      }
}

// ---------------------------------------------------------------------------------------------
// Gram kernel v2 (FP32): asynchronous direct-to-LDS loads into a two-stage ring.
//
//   * Each k-step stages the FP32 columns [k, k+32) of the two 256-row panels (of a diagonal tile's one panel: 64 columns)
//     with buffer loads to LDS: every wave instruction moves 8 rows x 128 B straight from global
//     memory to LDS (no register staging). Row r's eight 16-byte chunks are stored XOR-swizzled
//     (LDS chunk p holds column chunk p ^ (r & 7)) so that fragment reads of 8 consecutive rows
//     hit distinct banks.
//   * Two LDS stages: the loads for step s+1 are in flight while step s is multiplied; one
//     barrier per step.
//   * 4 waves in a 2 x 2 layout, each owning a 128 x 128 sub-tile (4 x 4 blocks of 32 x 32
//     accumulators), or the 36 blocks of a diagonal tile's lower triangle, 9 per wave.
//   * Rows beyond n and column chunks past a slice end lie outside the loads' buffers. The kernel
//     covers columns [0, m4) with m4 = m rounded down to a multiple of 4; the FP64 reduction adds
//     the products of the last m - m4 (< 4) columns.
//   * Bound by the FP32 matrix rate, 64 cycles a product and SIMD. A 32-column step of 256 products takes 6.96 us where
//     they alone need 6.83, a diagonal one of 64 columns and 288 products 7.89 (7.68). With 16 products' worth of idle
//     diagonal blocks, sign multiplications of A between the products (they change nothing: these sums round
//     symmetrically) and the loads' addresses in vector registers these took 7.97 and 15.9. Gram of 1024 x 10^6: 7.4 ms
//     (10.44 before), 256 x 10^5: 77 us (129), 2048 x 2 10^5: 5.7 ms (7.4).
// vmcnt(N) with the other counters left alone (gfx9 encoding: vmcnt bits [3:0] and [15:14]).
#define DFI_WAIT_VM(N) __builtin_amdgcn_s_waitcnt(((N) & 15) | (((N) >> 4) << 14) | (7 << 4) | (15 << 8))
// lgkmcnt(0) with the other counters left alone (lgkmcnt bits [11:8]).
#define DFI_WAIT_LGKM0() __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4))

namespace v2 {

constexpr int NW = 4;
constexpr int NT = 64 * NW;
constexpr int WT = 128;                 // wave sub-tile edge
constexpr int NB = WT / 32;             // 4 blocks per edge
constexpr int PANEL = T * KS;           // floats per panel per stage (32 KB)

typedef __attribute__((address_space(3))) void lds_void;

struct alignas(16) Stage {
  float a[PANEL];
  float b[PANEL];
};

// f(0) .. f(N - 1), the index a compile-time constant from the start: with a loop, unrolled only after the compiler has taken
// the register arrays apart, LDS reads are split into words and lose their width and the name of their stage.
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// Work items of this kernel: the off-diagonal tiles of every slice first, then the diagonal ones, each kind in eight equal
// parts by XCD. The short items come last and fill the end of the launch: 1024 x 10^6 (6 + 4 tiles) 8.4 -> 7.4 ms.
__host__ __device__ __forceinline__ int64_t v2_per_xcd(int64_t tiles, int64_t nslice) { return (tiles * nslice + 7) >> 3; }
__device__ __forceinline__ bool v2_item(int64_t w, int64_t ntile, int64_t nslice, int64_t& slice, int64_t& ti, int64_t& tj) {
  const int64_t noff = ntile * (ntile - 1) / 2, per = v2_per_xcd(noff, nslice);
  int64_t local = w >> 3;
  if (local < per) {
    const int64_t item = (w & 7) * per + local;
    if (item >= noff * nslice) return false;
    slice = uni64(item / noff);
    tri_index(item - slice * noff, ti, tj);
    ++ti;
    return true;
  }
  local -= per;
  const int64_t perd = v2_per_xcd(ntile, nslice), item = (w & 7) * perd + local;
  if (local >= perd || item >= ntile * nslice) return false;
  slice = uni64(item / ntile);
  ti = tj = item - slice * ntile;
  return true;
}

// A diagonal tile's lower triangle has 36 of the 64 blocks of 32 x 32, as 36 unordered pairs of its 8 block rows. Wave w
// takes 9 pairs that need each block row once: with F[t] the operand of block row (w + t) & 7, the pairs F[0] x F[0, 7, 6, 5],
// F[4] x F[4, 3, 2, 1] and F[4] x F[0] (differences 0 .. 3 from rows w and w + 4, and the one pair of w at difference 4).
// F[0]'s products that wrap around lie above the diagonal and are stored transposed.
constexpr int NDIAG = 9;
constexpr int DIAG_A[NDIAG] = {0, 0, 0, 0, 4, 4, 4, 4, 4};
constexpr int DIAG_B[NDIAG] = {0, 7, 6, 5, 4, 3, 2, 1, 0};

// W: bytes a lane loads, 16 (16-byte aligned rows) or 4 (any rows).
template <int W>
__device__ __forceinline__ void gram_v2_body(const float* __restrict__ S, int64_t n, int64_t lds, int64_t m, int64_t ntile,
                                             int64_t nslice, int64_t kslice, float* __restrict__ part) {
  __shared__ Stage st0;
  __shared__ Stage st1;

  int64_t slice, ti, tj;
  if (!v2_item(blockIdx.x, ntile, nslice, slice, ti, tj)) return;
  ti = uni64(ti);
  tj = uni64(tj);
  const int64_t ntri = ntile * (ntile + 1) / 2, tile = ti * (ti + 1) / 2 + tj;
  const bool diag = (ti == tj);
  const int64_t rowA = ti * T, rowB = tj * T;
  const int64_t k0 = uni64(slice * kslice);
  // W = 16: columns [m rounded down to 4, m) go to the reduction
  const int64_t kend = min(W == 16 ? m & ~(int64_t)3 : m, k0 + kslice);
  // a step is KS columns of both panels, or 2 KS columns of a diagonal tile's one panel: the same 16 loads a wave
  const int64_t span = diag ? 2 * KS : KS;
  const int64_t nsteps = (kend > k0) ? (kend - k0 + span - 1) / span : 0;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5;
  const int l32 = lane & 31;
  float* out = part + (slice * ntri + tile) * (int64_t)(T * T);

  // Loads: piece i of a panel carries rows 8 (wave + 4 i) .. + 7 of 32 columns; lane l of its one 16-byte load row l / 8 and
  // the column chunk (l % 8) ^ (row & 7), of its four 4-byte loads j row 2 j + l / 32 and the column that belongs to word
  // l % 32 of the swizzled row. A load's buffer begins at the first of its rows (64-bit scalar arithmetic) and ends behind the
  // last row of S, and a lane whose columns lie past the slice's end (for W = 16 a multiple of 4: a chunk is wholly inside or
  // wholly past it) gets an offset outside every buffer: out of range reads nothing and gives zeros. Needs 8 lds * 4 < 2^32.
  constexpr int NL = 16 / W;             // loads a piece
  constexpr int RL = 8 / NL;             // rows a load
  const uint32_t rowbytes = (uint32_t)lds * 4;
  uint32_t voff[NL];
  int coff[NL];                          // the lanes' (first) columns in a step
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const int r = RL * j + lane / (64 / RL);
    coff[j] = W == 16 ? 4 * ((lane & 7) ^ r) : 4 * (((lane & 31) >> 2) ^ r) + (lane & 3);
    voff[j] = (uint32_t)(lane / (64 / RL)) * rowbytes + 4 * coff[j];
  }
  const int64_t limA = kend - k0, limB = diag ? limA - KS : limA;
  const float* const baseA = S + (rowA + 8 * wave) * lds + k0;
  const float* const baseB = S + (rowB + 8 * wave) * lds + (diag ? k0 + KS : k0);
  const int leftA = (int)min(n - rowA, (int64_t)T) - 8 * wave, leftB = (int)min(n - rowB, (int64_t)T) - 8 * wave;
  // Stage k, a compile-time constant: every LDS access then names its stage object, and the compiler's tracking of the
  // direct-to-LDS loads can tell the stages apart.
  auto stage = [&](auto k) __attribute__((always_inline)) -> Stage& {
    if constexpr (decltype(k)::value == 0) return st0;
    else return st1;
  };
  constexpr uint32_t OUT = 0xfffffff0u;
  // Where the next load of a panel begins: first row and the rows left of S from there (<= 0 behind its end), and the lanes'
  // offsets. The fences keep the scalar arithmetic of one load next to it, instead of 16 addresses in registers.
  struct Cursor {
    const float* p;
    int left;
    int word;   // of the wave's next 8 rows in a panel
    uint32_t v[NL];
  };
  auto cursor = [&](int64_t off, bool second) __attribute__((always_inline)) {
    Cursor c;
    c.p = (second ? baseB : baseA) + off;
    c.left = second ? leftB : leftA;
    c.word = 8 * wave * KS;
#pragma unroll
    for (int j = 0; j < NL; ++j) c.v[j] = off + coff[j] < (second ? limB : limA) ? voff[j] : OUT;
    asm volatile("" : "+s"(c.p), "+s"(c.left), "+s"(c.word));
    return c;
  };
  // the panel's next piece, at its cursor, which moves on
  auto issue = [&](float* panel, Cursor& c) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      int rows = max(c.left, 0);
      asm volatile("" : "+s"(rows));
      rows = min(rows, RL);
      const __amdgpu_buffer_rsrc_t rs =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(c.p), 0, (int)((uint32_t)rows * rowbytes), 0x00020000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)(panel + c.word), W, c.v[j], 0, 0, 0);
      const int step = j + 1 < NL ? RL : 8 * NW - RL * j;   // rows to the next load
      c.p += step * lds;
      c.left -= step;
      c.word += step * KS;
      asm volatile("" : "+s"(c.p), "+s"(c.left), "+s"(c.word));
    }
  };
  static_assert(T / 8 / NW == 8, "16 pieces of both panels: four in each of four groups");
  using K0 = std::integral_constant<int, 0>;
  using K1 = std::integral_constant<int, 1>;
  // LDS word of row l32, chunk u (0 .. 3) of this lane's half of the 32 columns
  int lo[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) lo[u] = l32 * KS + 4 * ((half * 4 + u) ^ (l32 & 7));

  if (nsteps > 0) {
    Cursor ca = cursor(0, false), cb = cursor(0, true);
#pragma unroll
    for (int i = 0; i < T / 8 / NW; ++i) {
      issue(st0.a, ca);
      issue(st0.b, cb);
    }
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("s_barrier" ::: "memory");
  }

  // Both loops: a step in groups of products whose operands were read one group ahead; the last group reads the next
  // step's first operands, after the wait for that step's loads (issued a step ago) and the barrier that also frees this
  // step's stage, which the next step refills. The FP32 matrix instruction occupies the vector unit: a vector instruction
  // between two products that depends on nothing in flight still costs tens of cycles, so the loops hold none but the
  // addresses of the loads' lanes, once a step: LDS addresses are kept in registers for both stages, the loads' bases and
  // bounds are scalar, and the LDS reads take the rest as immediate offsets.
  if (diag) {
    f32x16 acc[NDIAG];
#pragma unroll
    for (int j = 0; j < NDIAG; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;
    // byte offsets of this lane's chunk u of block rows w + t: t = 0 .. 4 from ad[.][0], t = 5 .. 7 (may wrap) of their own
    int ad[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      ad[u][0] = 4 * (lo[u] + wave * 32 * KS);
#pragma unroll
      for (int t = 5; t < 8; ++t) ad[u][t - 4] = 4 * (lo[u] + ((wave + t) & 7) * 32 * KS);
#pragma unroll
      for (int t = 0; t < 4; ++t) asm volatile("" : "+v"(ad[u][t]));
    }
    constexpr int NG = 8;   // groups: chunk g & 3 of panel g >> 2
    f32x4 f[2][8];
    auto read_f = [&](const Stage& st, auto gc) __attribute__((always_inline)) {
      constexpr int g = decltype(gc)::value;
      const char* p = reinterpret_cast<const char*>(g < 4 ? st.a : st.b);
      static_for<8>([&](auto tc) __attribute__((always_inline)) {
        constexpr int t = decltype(tc)::value;
        constexpr int r = t < 5 ? 0 : t - 4, o = t < 5 ? t * 32 * KS * 4 : 0;
        f[g & 1][t] = *reinterpret_cast<const f32x4*>(p + ad[g & 3][r] + o);
      });
    };
    auto body = [&](auto k, int64_t s) __attribute__((always_inline)) {
      constexpr int K = decltype(k)::value;
      const int64_t off = (s + 1) * span;
      Cursor ca = cursor(off, false), cb = cursor(off, true);
      static_for<NG>([&](auto gc) __attribute__((always_inline)) {
        constexpr int g = decltype(gc)::value;
        DFI_WAIT_LGKM0();
        if constexpr (g + 1 < NG) {
          read_f(stage(k), std::integral_constant<int, g + 1>{});
        } else {
          __builtin_amdgcn_s_waitcnt(0);
          asm volatile("s_barrier" ::: "memory");
          read_f(stage(std::integral_constant<int, 1 - K>{}), K0{});
        }
        __builtin_amdgcn_sched_barrier(0);
        static_for<4>([&](auto ec) __attribute__((always_inline)) {
          constexpr int e = decltype(ec)::value;
          static_for<NDIAG>([&](auto jc) __attribute__((always_inline)) {
            constexpr int j = decltype(jc)::value;
            acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(f[g & 1][DIAG_A[j]][e], f[g & 1][DIAG_B[j]][e], acc[j], 0, 0, 0);
          });
          if constexpr (g < 4) {
            __builtin_amdgcn_sched_barrier(0);
            Stage& nx = stage(std::integral_constant<int, 1 - K>{});
            if constexpr (e & 1) issue(nx.b, cb);
            else issue(nx.a, ca);
            __builtin_amdgcn_sched_barrier(0);
          }
        });
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    if (nsteps > 0) {
      read_f(st0, K0{});
      int64_t s = 0;
      for (; s + 1 < nsteps; s += 2) {
        body(K0{}, s);
        body(K1{}, s + 1);
      }
      if (s < nsteps) body(K0{}, s);
    }
    __builtin_amdgcn_s_waitcnt(0);   // no load into LDS outlives the workgroup
#pragma unroll
    for (int j = 0; j < NDIAG; ++j) {
      const int rb = (wave + DIAG_A[j]) & 7, cb = (wave + DIAG_B[j]) & 7;
      if (!block_used(true, rowA, rowB, max(rb, cb) * 32, min(rb, cb) * 32, n)) continue;
      if (cb <= rb) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          out[(rb * 32 + 8 * (r >> 2) + 4 * half + (r & 3)) * T + cb * 32 + l32] = acc[j][r];
      } else {
#pragma unroll
        for (int r = 0; r < 16; r += 4)
          *reinterpret_cast<f32x4*>(&out[(cb * 32 + l32) * T + rb * 32 + 2 * r + 4 * half]) =
              f32x4{acc[j][r], acc[j][r + 1], acc[j][r + 2], acc[j][r + 3]};
      }
    }
    return;
  }

  const int wr = wave >> 1, wc = wave & 1;
  f32x16 acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // Groups of 8 columns of each half and one A block row (32 products); the four B blocks of the second 8 columns are read
  // during the first four groups.
  constexpr int NG = 2 * NB;
  int aa[4], ab[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    aa[u] = 4 * (lo[u] + wr * WT * KS);
    ab[u] = 4 * (lo[u] + wc * WT * KS);
    asm volatile("" : "+v"(aa[u]), "+v"(ab[u]));
  }
  f32x8 fa[2], fb[2][NB];
  auto read8 = [&](const float* p, int o0, int o1) __attribute__((always_inline)) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(reinterpret_cast<const char*>(p) + o0);
    const f32x4 y = *reinterpret_cast<const f32x4*>(reinterpret_cast<const char*>(p) + o1);
    return f32x8{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
  };
  auto read_a = [&](const Stage& st, int g, int d) __attribute__((always_inline)) {
    const int o = 32 * (g % NB) * KS * 4;
    fa[d] = read8(st.a, aa[2 * (g / NB)] + o, aa[2 * (g / NB) + 1] + o);
  };
  auto read_b = [&](const Stage& st, int h, int j) __attribute__((always_inline)) {
    fb[h][j] = read8(st.b, ab[2 * h] + 32 * j * KS * 4, ab[2 * h + 1] + 32 * j * KS * 4);
  };
  auto head = [&](const Stage& st) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NB; ++j) read_b(st, 0, j);
    read_a(st, 0, 0);
  };
  auto body = [&](auto k, int64_t s) __attribute__((always_inline)) {
    constexpr int K = decltype(k)::value;
    const int64_t off = (s + 1) * span;
    Cursor ca = cursor(off, false), cb = cursor(off, true);
    static_for<NG>([&](auto gc) __attribute__((always_inline)) {
      constexpr int g = decltype(gc)::value;
      DFI_WAIT_LGKM0();
      if constexpr (g + 1 < NG) {
        read_a(stage(k), g + 1, (g + 1) & 1);
        if constexpr (g < NB) read_b(stage(k), 1, g);
      } else {
        __builtin_amdgcn_s_waitcnt(0);
        asm volatile("s_barrier" ::: "memory");
        head(stage(std::integral_constant<int, 1 - K>{}));
      }
      __builtin_amdgcn_sched_barrier(0);
      static_for<8>([&](auto ec) __attribute__((always_inline)) {
        constexpr int e = decltype(ec)::value;
        static_for<NB>([&](auto jc) __attribute__((always_inline)) {
          constexpr int j = decltype(jc)::value;
          acc[g % NB][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[g & 1][e], fb[g / NB][j][e], acc[g % NB][j], 0, 0, 0);
        });
        if constexpr (g < 4 && (e & 1)) {
          __builtin_amdgcn_sched_barrier(0);
          Stage& nx = stage(std::integral_constant<int, 1 - K>{});
          if constexpr (e & 2) issue(nx.b, cb);
          else issue(nx.a, ca);
          __builtin_amdgcn_sched_barrier(0);
        }
      });
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  if (nsteps > 0) {
    head(st0);
    for (int64_t s = 0; s < nsteps; s += 2) {   // (an odd count ends with a step of zeros: the body alone once more spills)
      body(K0{}, s);
      body(K1{}, s + 1);
    }
  }
  __builtin_amdgcn_s_waitcnt(0);

#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
      if (block_used(false, rowA, rowB, wr * WT + i * 32, wc * WT + j * 32, n))
#pragma unroll
        for (int r = 0; r < 16; ++r)
          out[(wr * WT + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3)) * T + wc * WT + j * 32 + l32] = acc[i][j][r];
}

__global__ void __launch_bounds__(NT, 1)
gram_kernel_v2(const float* __restrict__ S, int64_t n, int64_t lds, int64_t m, int64_t ntile, int64_t nslice,
               int64_t kslice, float* __restrict__ part) {
  gram_v2_body<16>(S, n, lds, m, ntile, nslice, kslice, part);
}

__global__ void __launch_bounds__(NT, 1)
gram_kernel_v2_words(const float* __restrict__ S, int64_t n, int64_t lds, int64_t m, int64_t ntile, int64_t nslice,
                     int64_t kslice, float* __restrict__ part) {
  gram_v2_body<4>(S, n, lds, m, ntile, nslice, kslice, part);
}

}  // namespace v2

// ---------------------------------------------------------------------------------------------
// Gram kernel v3: scaled FP8. The operands are the block-scaled E4M3 codes written by the row
// pass in its column-blocked layout: 64-column blocks (one k-step), each holding all n rows
// contiguously (code (i, k) at q[((k / 64) n + i) 64 + k % 64]; the four E8M0 scale bytes of row
// i and 128-column block k / 128 form one aligned 4-byte word at sc[((k / 128) n + i) 4]). A
// k-step of a 256-row panel is then 16 KB of dense contiguous memory: whole cache lines, few
// pages, half the memory requests of 64-byte pieces of longer rows.
//   * k-step = 64 columns (two scale blocks). Codes move direct-to-LDS: each wave instruction
//     carries 16 rows x 64 B; row r's four 16-byte chunks are XOR-swizzled by (r >> 2) & 3 so the
//     fragment reads of 16 consecutive rows hit distinct banks. Scale bytes move direct-to-LDS as
//     one 4-byte word per row (four blocks, 128 columns; the step uses two of them), since the LDS
//     side of these loads advances 4 bytes per lane.
//   * Four LDS stages: the direct-to-LDS loads run up to four steps ahead of the matrix cores.
//     Every wave issues the same number of loads per step (diagonal tiles load their B panel as
//     well), so waiting for a stage is a vmcnt wait on the count of loads issued after it, plus
//     one barrier per step. Inside a step each A fragment is read one MFMA group ahead of its use;
//     the step's barrier sits before its last group, so the next step's B fragments and first A
//     fragment are read while that group's products run.
//   * v_mfma_scale_f32_32x32x64_f8f6f4: lane l supplies row (l % 32), 16 codes from scale block 0
//     and 16 from block 1 of the step (bytes [16h, 16h+16) and [32+16h, 32+16h+16) for h = l/32),
//     and the E8M0 scale of block h of its row. A and B use the same byte arrangement, so every
//     product pairs one column with itself.
//   * The slices cover all of [0, ldq): past m the row pass wrote zero codes, so every k-step is
//     whole and nothing is masked; the reduction adds no tail columns for this kernel.
//   * No alternating slice sign: the accumulation bias it cancels for bf16 (about 1e-6 relative)
//     is far below the E4M3 rounding of the operands.
namespace v3 {

constexpr int NW = 4;
constexpr int NT = 64 * NW;
constexpr int WT = 128;
constexpr int NB = WT / 32;
constexpr int KS8 = 64;                  // codes (bytes) per row per step
constexpr int PANEL = T * KS8;           // 16 KB
constexpr int NS = 4;                    // LDS stages
constexpr int LOADS_PER_STEP = 2 * (T / 16 / NW) + 2;   // codes A, B + scales A, B (per wave)

typedef __attribute__((address_space(3))) void lds_void;
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

struct Stage {
  uint8_t a[PANEL];
  uint8_t b[PANEL];
  uint8_t sa[4 * T];   // scale word of row r at [4r, 4r + 4): blocks 4w .. 4w + 3, w = kcol / 128
  uint8_t sb[4 * T];
};

// Loop-invariant per-lane byte offsets, inside one column block, of what this lane moves for a
// 256-row panel: code chunks (wave instruction i carries rows 16 g .. 16 g + 15, g = wave + 4 i;
// lane l fills LDS row 16 g + l / 4, chunk slot l % 4, with column chunk (l % 4) ^ ((row >> 2) & 3))
// and the scale word of row 64 wave + lane. Rows past n are clamped to n - 1 (their products are
// never stored).
struct PanelOffs {
  uint32_t code[T / 16 / NW];
  uint32_t scale;
};

__device__ __forceinline__ void panel_offsets(int64_t n, int64_t row0, PanelOffs& po) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < T / 16 / NW; ++i) {
    const int g = wave + NW * i;
    const int r = 16 * g + (lane >> 2);
    const int c = (lane & 3) ^ ((r >> 2) & 3);
    const int64_t R = min(row0 + r, n - 1);
    po.code[i] = (uint32_t)((R << 6) + 16 * c);
  }
  po.scale = (uint32_t)(min(row0 + 64 * wave + lane, n - 1) << 2);
}

// The step at column kcol (a multiple of 64): 64 code bytes of each of the panel's rows and the
// rows' scale words, direct to LDS. Every step lies inside [0, ldq), where the row pass wrote
// zero codes past m, so there is nothing to mask. issue_codes moves the rows of wave instruction
// i (16 rows x 64 B), issue_scales the scale words; a whole panel is i = 0 .. T / 16 / NW - 1
// plus the scales.
__device__ __forceinline__ void issue_codes(const uint8_t* q, int64_t n, int64_t kcol, const PanelOffs& po,
                                            uint8_t* panel, int i) {
  const int g = (int)(threadIdx.x >> 6) + NW * i;
  const uint8_t* qb = q + ((kcol >> 6) * n << 6);   // row 0 of this step's block, uniform
  __builtin_amdgcn_global_load_lds((const void*)(qb + po.code[i]), (lds_void*)(panel + 16 * g * KS8), 16, 0, 0);
}
__device__ __forceinline__ void issue_scales(const uint8_t* sc, int64_t n, int64_t kcol, const PanelOffs& po,
                                             uint8_t* sdst) {
  const int wave = threadIdx.x >> 6;
  const uint8_t* sb = sc + ((kcol >> 7) * n << 2);
  __builtin_amdgcn_global_load_lds((const void*)(sb + po.scale), (lds_void*)(sdst + 256 * wave), 4, 0, 0);
}

// Fragment of row r: chunks h and 2 + h (swizzled) -> 32 codes.
__device__ __forceinline__ i32x8 read_frag(const uint8_t* panel, int r, int h) {
  const int sw = (r >> 2) & 3;
  const i32x4 x0 = *reinterpret_cast<const i32x4*>(panel + r * KS8 + 16 * (h ^ sw));
  const i32x4 x1 = *reinterpret_cast<const i32x4*>(panel + r * KS8 + 16 * ((2 + h) ^ sw));
  i32x8 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = x0[e];
    v[4 + e] = x1[e];
  }
  return v;
}

// The work item of workgroup w (the kernel body; the grouped form below runs it for one problem's
// share of a launch over many problems).
__device__ __forceinline__ void gram_fp8_body(const uint8_t* __restrict__ q, const uint8_t* __restrict__ sc, int64_t n,
                                              int64_t kcap, int64_t ntri, int64_t nslice, int64_t kslice,
                                              float* __restrict__ part, int64_t w) {
  __shared__ Stage stg0, stg1, stg2, stg3;

  int64_t slice, tile;
  if (!work_item(w, ntri, nslice, slice, tile)) return;

  int64_t ti, tj;
  tri_index(tile, ti, tj);
  ti = uni64(ti);
  tj = uni64(tj);
  const bool diag = (ti == tj);
  const int64_t rowA = ti * T, rowB = tj * T;
  const int64_t k0 = uni64(slice * kslice);
  const int64_t kend = min(kcap, k0 + kslice);
  const int64_t nsteps = uni64((kend > k0) ? (kend - k0) / KS8 : 0);   // both multiples of 64

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wr = wave >> 1, wc = wave & 1;
  const int half = lane >> 5;
  const int l32 = lane & 31;

  f32x16 acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // Stage k of the ring, k a compile-time constant: the step loop is unrolled by NS so that every
  // LDS access names its stage object. The compiler's tracking of direct-to-LDS loads can then
  // tell the stages apart; with a stage picked at run time it cannot, and it inserts a wait for
  // every load in flight (the three steps ahead included) before the first operand read of a step.
  auto stage = [&](auto k) -> Stage& {
    constexpr int K = decltype(k)::value;
    if constexpr (K == 0) return stg0;
    else if constexpr (K == 1) return stg1;
    else if constexpr (K == 2) return stg2;
    else return stg3;
  };
  PanelOffs offA, offB;
  panel_offsets(n, rowA, offA);
  panel_offsets(n, rowB, offB);
  // Refill stage k with `step` (k = step mod NS). Steps past the slice's end load the slice's
  // last step again (never read as operands): every step then issues the same loads and waits
  // for the same count, with no branch in the loop.
  // Piece p (0 .. NB - 1) of the refill: code instruction p of both panels, and with the last
  // piece both panels' scale words. Diagonal tiles load their B panel too: uniform load counts.
  static_assert(T / 16 / NW == NB, "one refill piece per product of a group");
  auto issue_piece = [&](auto k, int64_t step, int p) {
    Stage& sp = stage(k);
    const int64_t kc = k0 + min(step, nsteps - 1) * KS8;
    issue_codes(q, n, kc, offA, sp.a, p);
    issue_codes(q, n, kc, offB, sp.b, p);
    if (p == NB - 1) {
      issue_scales(sc, n, kc, offA, sp.sa);
      issue_scales(sc, n, kc, offB, sp.sb);
    }
  };
  auto issue_step = [&](auto k, int64_t step) {
#pragma unroll
    for (int p = 0; p < NB; ++p) issue_piece(k, step, p);
  };
  // this wave's operands of one step, read from LDS into registers
  // head of a step: the four B fragments with their scales and the first A fragment
  struct Head {
    i32x8 fb[NB];
    int sbv[NB];
    i32x8 fa0;
    int sa0;
  };
  // Per-lane LDS byte offsets inside a stage. Fragment i of the wave's A rows is row
  // wr WT + 32 i + l32; its swizzle (row >> 2) & 3 depends on l32 only, so fragment i sits at the
  // fragment-0 offsets + 32 i KS8 and its scale byte at + 128 i.
  struct LaneOffs {
    int a0, a1, b0, b1, sa, sb;
  };
  LaneOffs lo0;
  {
    const int sw = (l32 >> 2) & 3;
    const int ra = wr * WT + l32, rb = wc * WT + l32;
    lo0.a0 = ra * KS8 + 16 * (half ^ sw);
    lo0.a1 = ra * KS8 + 16 * ((2 + half) ^ sw);
    lo0.b0 = rb * KS8 + 16 * (half ^ sw);
    lo0.b1 = rb * KS8 + 16 * ((2 + half) ^ sw);
    lo0.sa = 4 * ra + half;
    lo0.sb = 4 * rb + half;
  }
  auto frag = [](const uint8_t* p0, const uint8_t* p1) {
    const i32x4 x0 = *reinterpret_cast<const i32x4*>(p0);
    const i32x4 x1 = *reinterpret_cast<const i32x4*>(p1);
    i32x8 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = x0[e];
      v[4 + e] = x1[e];
    }
    return v;
  };
  auto load_head = [&](auto k, int64_t step, Head& h, const LaneOffs& lo) {
    const Stage& cu = stage(k);
    const int sbyte = (int)(((k0 + step * KS8) >> 5) & 3);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      h.fb[j] = frag(cu.b + lo.b0 + 32 * KS8 * j, cu.b + lo.b1 + 32 * KS8 * j);
      h.sbv[j] = cu.sb[lo.sb + 128 * j + sbyte];
    }
    h.fa0 = frag(cu.a + lo.a0, cu.a + lo.a1);
    h.sa0 = cu.sa[lo.sa + sbyte];
  };
  // Step s (in stage k) from head h (already in registers): A fragments 1..3 are read one group
  // ahead; after the third group every LDS read of step s is done, so the wave waits for step
  // s + 1's loads (two steps' loads issued later may stay in flight), meets the others at the
  // barrier, reads step s + 1's head into hn and refills stage k with step s + NS while the last
  // group of matrix-core products runs. The step has no branch: the scheduling fences below only
  // hold inside one basic block, and with branches in the step the compiler sinks its products
  // below the waits and the barrier, leaving the matrix cores idle through them. At the last step
  // the head read is of a stage that holds no later step; it is never used. The lane offsets are
  // made opaque once per step, so that the compiler forms each address next to its read instead
  // of keeping every stage's addresses live (which spills).
  auto body = [&](auto k, int64_t s, Head& h, Head& hn) {
    constexpr int K = decltype(k)::value;
    const Stage& cu = stage(k);
    LaneOffs lo = lo0;
    asm volatile("" : "+v"(lo.a0), "+v"(lo.a1), "+v"(lo.b0), "+v"(lo.b1), "+v"(lo.sa), "+v"(lo.sb));
    const int sbyte = (int)(((k0 + s * KS8) >> 5) & 3);
    i32x8 fa[2];
    int sav[2];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      // Group i's operands were requested a whole group earlier and have arrived; waiting for
      // them here, before fragment i + 1 is requested, keeps the wait off the newer reads.
      DFI_WAIT_LGKM0();
      if (i + 1 < NB) {
        fa[(i + 1) & 1] = frag(cu.a + lo.a0 + 32 * KS8 * (i + 1), cu.a + lo.a1 + 32 * KS8 * (i + 1));
        sav[(i + 1) & 1] = cu.sa[lo.sa + 128 * (i + 1) + sbyte];
      }
      if (i == NB - 1) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        DFI_WAIT_VM(2 * LOADS_PER_STEP);
        asm volatile("s_barrier" ::: "memory");
        load_head(std::integral_constant<int, (K + 1) % NS>{}, s + 1, hn, lo);
      }
      __builtin_amdgcn_sched_barrier(0);
      const i32x8 a = (i == 0) ? h.fa0 : fa[i & 1];
      const int sa = (i == 0) ? h.sa0 : sav[i & 1];
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, h.fb[j], acc[i][j], 0, 0, 0, sa, 0, h.sbv[j]);
        if (i == NB - 1) {
          // the refill of stage k goes out in pieces between the last group's products, whose
          // execution hides the issue of its loads and their address arithmetic
          __builtin_amdgcn_sched_barrier(0);
          issue_piece(k, s + NS, j);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using K0 = std::integral_constant<int, 0>;
  using K1 = std::integral_constant<int, 1>;
  using K2 = std::integral_constant<int, 2>;
  using K3 = std::integral_constant<int, 3>;
  static_assert(NS == 4, "the step loop is unrolled by the stage count");
  Head h0, h1;
  if (nsteps > 0) {
    issue_step(K0{}, 0);
    issue_step(K1{}, 1);
    issue_step(K2{}, 2);
    issue_step(K3{}, 3);
    DFI_WAIT_VM(3 * LOADS_PER_STEP);
    asm volatile("s_barrier" ::: "memory");
    load_head(K0{}, 0, h0, lo0);
    int64_t s = 0;
    // The loop starts on a multiple of 8 bytes: 44 of its 64 products (16 bytes each) then do too, 4 bytes off only 20.
    // Where it happened to lie decided over 5 %: n = 4096, m = 4M 33.2 ms 4 bytes off, 31.1 here (1M: 7.8, 7.7).
    // (Every product aligned, with a no-op before each group where needed: 32.3.)
    for (; s + 3 < nsteps; s += 4) {
      asm volatile(".p2align 3");
      __builtin_amdgcn_sched_barrier(0);
      body(K0{}, s, h0, h1);
      body(K1{}, s + 1, h1, h0);
      body(K2{}, s + 2, h0, h1);
      body(K3{}, s + 3, h1, h0);
    }
    if (s < nsteps) body(K0{}, s, h0, h1);
    if (s + 1 < nsteps) body(K1{}, s + 1, h1, h0);
    if (s + 2 < nsteps) body(K2{}, s + 2, h0, h1);
    DFI_WAIT_VM(0);   // the trailing refills land in LDS before the workgroup ends
  }

  float* out = part + (slice * ntri + tile) * (int64_t)(T * T);
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
      if (block_used(diag, rowA, rowB, wr * WT + i * 32, wc * WT + j * 32, n))
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = wr * WT + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
        const int col = wc * WT + j * 32 + l32;
        out[row * T + col] = acc[i][j][r];
      }
}

__global__ void __launch_bounds__(NT, 1)
gram_kernel_fp8(const uint8_t* __restrict__ q, const uint8_t* __restrict__ sc, int64_t n, int64_t kcap,
                int64_t ntri, int64_t nslice, int64_t kslice, float* __restrict__ part) {
  gram_fp8_body(q, sc, n, kcap, ntri, nslice, kslice, part, blockIdx.x);
}

// Many problems' scaled-FP8 Grams in one launch: job j owns workgroups [wg0_j, wg0_j + ntri_j
// nslice_j) and runs its (tile, slice) work items exactly as its own launch would (wg0_j a
// multiple of 8, so each work item keeps its XCD), writing its own partial tiles. The jobs are
// ordered by the work of one item (slice length), largest first, so the dispatcher hands the
// largest items out first and the small ones fill the end of the launch. A workgroup finds its job
// by bisection (uniform, scalar loads).
__global__ void __launch_bounds__(NT, 1)
gram_kernel_fp8_grouped(const GramJob* __restrict__ jobs, int njobs) {
  const int64_t w = blockIdx.x;
  int lo = 0, hi = njobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs[mid].wg0 <= w) lo = mid;
    else hi = mid - 1;
  }
  lo = __builtin_amdgcn_readfirstlane(lo);
  const GramJob& j = jobs[lo];
  const int64_t wl = w - j.wg0;
  if (wl < 0 || wl >= j.ntri * j.nslice) return;
  gram_fp8_body(j.q, j.sc, j.n, j.kcap, j.ntri, j.nslice, j.kslice, j.part, wl);
}

}  // namespace v3

// ---------------------------------------------------------------------------------------------
// Gram kernel v4: split-BF16 from pre-split planes. The row pass writes hi = bf16_rne(S) and
// lo = bf16_rne(S - hi) as two bf16 planes in its column-blocked layout (16-column blocks, one
// k-step, of all n rows: element (i, k) at [((k / 16) n + i) 16 + k % 16], so a step of a panel
// is 8 KB of dense contiguous memory); the tile kernel is then a plain bf16
// matrix-core product with three terms per pair of elements (lo.hi, hi.lo, hi.hi) and no
// conversion work in its loop.
//   * k-step = 16 columns: 32 bytes of each of the 256 rows of a panel, per plane. One wave
//     instruction moves 32 rows straight to LDS (two 16-byte chunks per row); a row's chunks are
//     swapped when (row >> 2) is odd, so the fragment reads of 8 consecutive rows cover all banks.
//   * Four LDS stages of 32 KB (A hi, A lo, B hi, B lo) and two register sets of operands, with
//     the same schedule and vmcnt-counted waits as v3 (every wave issues the same number of loads
//     per step; diagonal tiles load their B panel too).
//   * v_mfma_f32_32x32x16_bf16: lane l supplies row l % 32 and columns 8h .. 8h + 7 of the step
//     (h = l / 32), for A and B alike.
//   * The slices cover all of [0, ldh): past m the planes hold zeros, so every k-step is whole;
//     the reduction adds no tail columns for this kernel.
//   * Alternating slice sign as in v1: odd slices flip the sign bits of A's fragments.
namespace v4 {

constexpr int NW = 4;
constexpr int NT = 64 * NW;
constexpr int WT = 128;
constexpr int NB = WT / 32;
constexpr int KSB = 16;                          // bf16 columns per step
constexpr int ROWB = 2 * KSB;                    // 32 bytes per row and plane
constexpr int PANEL = T * ROWB;                  // 8 KB
constexpr int NS = 4;                            // LDS stages
constexpr int INSTR = T / 32 / NW;               // load instructions per wave, panel and plane (2)
constexpr int LOADS_PER_STEP = 4 * INSTR;        // A hi, A lo, B hi, B lo

typedef __attribute__((address_space(3))) void lds_void;

struct Stage {
  uint8_t ah[PANEL];
  uint8_t al[PANEL];
  uint8_t bh[PANEL];
  uint8_t bl[PANEL];
};

// Loop-invariant per-lane element offsets (inside one 16-column block of a plane) of the chunks
// this lane moves for a 256-row panel: wave instruction i carries rows 32 g .. 32 g + 31
// (g = wave + 4 i); lane l fills LDS row 32 g + l / 2, chunk slot l % 2, with column chunk
// (l % 2) ^ ((row >> 2) & 1). Rows past n are clamped to n - 1 (their products are never stored).
struct PanelOffs {
  uint32_t e[INSTR];
};

__device__ __forceinline__ void panel_offsets(int64_t n, int64_t row0, PanelOffs& po) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < INSTR; ++i) {
    const int g = wave + NW * i;
    const int r = 32 * g + (lane >> 1);
    const int c = (lane & 1) ^ ((r >> 2) & 1);
    const int64_t R = min(row0 + r, n - 1);
    po.e[i] = (uint32_t)((R << 4) + 8 * c);
  }
}

// One plane of one panel for the step at column kcol (a multiple of 16): every step lies inside
// [0, ldh), where the row pass wrote zeros past m, so nothing is masked.
__device__ __forceinline__ void issue_plane(const uint16_t* plane, int64_t n, int64_t kcol, const PanelOffs& po,
                                            uint8_t* panel) {
  const uint16_t* pb = plane + ((kcol >> 4) * n << 4);   // row 0 of this step's block, uniform
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < INSTR; ++i) {
    const int g = wave + NW * i;
    __builtin_amdgcn_global_load_lds((const void*)(pb + po.e[i]), (lds_void*)(panel + 32 * g * ROWB), 16, 0, 0);
  }
}

// One wave's operands of one k-step: hi and lo fragments of its 4 A and 4 B row blocks.
struct Frags {
  bf16x8 ah[NB], al[NB], bh[NB], bl[NB];
};

__global__ void __launch_bounds__(NT, 1)
gram_kernel_split(const uint16_t* __restrict__ hi, const uint16_t* __restrict__ lo, int64_t n,
                  int64_t kcap, int64_t ntri, int64_t nslice, int64_t kslice, float* __restrict__ part) {
  __shared__ Stage stg0, stg1, stg2, stg3;

  int64_t slice, tile;
  if (!work_item(blockIdx.x, ntri, nslice, slice, tile)) return;
  const uint32_t bflip = (slice & 1) ? 0x80008000u : 0u;

  int64_t ti, tj;
  tri_index(tile, ti, tj);
  ti = uni64(ti);
  tj = uni64(tj);
  const bool diag = (ti == tj);
  const int64_t rowA = ti * T, rowB = tj * T;
  const int64_t k0 = uni64(slice * kslice);
  const int64_t kend = min(kcap, k0 + kslice);
  const int64_t nsteps = uni64((kend > k0) ? (kend - k0) / KSB : 0);   // both multiples of 16

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wr = wave >> 1, wc = wave & 1;
  const int half = lane >> 5;
  const int l32 = lane & 31;

  f32x16 acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // Stage k of the ring, k a compile-time constant (see the scaled-FP8 kernel: the loop is unrolled
  // by NS so that every LDS access names its stage object).
  auto stage = [&](auto k) -> Stage& {
    constexpr int K = decltype(k)::value;
    if constexpr (K == 0) return stg0;
    else if constexpr (K == 1) return stg1;
    else if constexpr (K == 2) return stg2;
    else return stg3;
  };
  PanelOffs offA, offB;
  panel_offsets(n, rowA, offA);
  panel_offsets(n, rowB, offB);
  // Piece p of the refill of stage k with `step` (k = step mod NS): plane p of the four (A hi, A lo,
  // B hi, B lo; diagonal tiles load B too: uniform load counts). Steps past the slice's end load
  // the slice's last step again (never read as operands), so every step issues the same loads.
  auto issue_piece = [&](auto k, int64_t step, int p) {
    Stage& sp = stage(k);
    const int64_t kc = k0 + min(step, nsteps - 1) * KSB;
    if (p == 0) issue_plane(hi, n, kc, offA, sp.ah);
    else if (p == 1) issue_plane(lo, n, kc, offA, sp.al);
    else if (p == 2) issue_plane(hi, n, kc, offB, sp.bh);
    else issue_plane(lo, n, kc, offB, sp.bl);
  };
  auto issue_step = [&](auto k, int64_t step) {
#pragma unroll
    for (int p = 0; p < 4; ++p) issue_piece(k, step, p);
  };
  // Per-lane LDS byte offsets of fragment 0 of the wave's A and B rows inside a plane; fragment i
  // is 32 rows further on (+ 32 i ROWB), with the same swizzle ((row >> 2) & 1 depends on l32 only).
  int oA0, oB0;
  {
    const int sw = (l32 >> 2) & 1;
    oA0 = (wr * WT + l32) * ROWB + 16 * (half ^ sw);
    oB0 = (wc * WT + l32) * ROWB + 16 * (half ^ sw);
  }
  auto rd = [](const uint8_t* p) { return *reinterpret_cast<const bf16x8*>(p); };
  auto load_frags = [&](auto k, Frags& f, int oA, int oB) {
    const Stage& cu = stage(k);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      f.bh[j] = rd(cu.bh + oB + 32 * ROWB * j);
      f.bl[j] = rd(cu.bl + oB + 32 * ROWB * j);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      f.ah[i] = rd(cu.ah + oA + 32 * ROWB * i);
      f.al[i] = rd(cu.al + oA + 32 * ROWB * i);
    }
  };
  // term t of the product of A row block i with B row block j: lo.hi, hi.lo, hi.hi in that order
  auto mfma_term = [&](const Frags& f, int i, int j, int t) {
    const bf16x8 a = flip_sign(t == 0 ? f.al[i] : f.ah[i], bflip);
    const bf16x8 b = t == 1 ? f.bl[j] : f.bh[j];
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[i][j], 0, 0, 0);
  };
  // Step s (stage k) from operands cur (already in registers): the products of A row blocks
  // 0 .. NB - 2 run first; then the wave waits for step s + 1's loads (two later steps' loads may
  // stay in flight), meets the others at the barrier (every wave has read stage k, which it did
  // into cur one step earlier), reads step s + 1's operands into nxt and refills stage k with step
  // s + NS between the last row block's products. The step has no branch, so the
  // scheduling fences hold and the products overlap the waits.
  auto body = [&](auto k, Frags& cur, Frags& nxt, int64_t s) {
    constexpr int K = decltype(k)::value;
    int oA = oA0, oB = oB0;
    asm volatile("" : "+v"(oA), "+v"(oB));
#pragma unroll
    for (int i = 0; i < NB - 1; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int t = 0; t < 3; ++t) mfma_term(cur, i, j, t);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    DFI_WAIT_VM(2 * LOADS_PER_STEP);
    asm volatile("s_barrier" ::: "memory");
    load_frags(std::integral_constant<int, (K + 1) % NS>{}, nxt, oA, oB);
    __builtin_amdgcn_sched_barrier(0);
    // the last row block term by term (four independent accumulators between fences), with the
    // refill's planes 0 and 1, 2, 3 after the three terms
#pragma unroll
    for (int t = 0; t < 3; ++t) {
#pragma unroll
      for (int j = 0; j < NB; ++j) mfma_term(cur, NB - 1, j, t);
      __builtin_amdgcn_sched_barrier(0);
      if (t == 0) issue_piece(k, s + NS, 0);
      issue_piece(k, s + NS, t + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using K0 = std::integral_constant<int, 0>;
  using K1 = std::integral_constant<int, 1>;
  using K2 = std::integral_constant<int, 2>;
  using K3 = std::integral_constant<int, 3>;
  static_assert(NS == 4 && NB == 4, "the step loop is unrolled by the stage count");
  Frags f0, f1;
  if (nsteps > 0) {
    issue_step(K0{}, 0);
    issue_step(K1{}, 1);
    issue_step(K2{}, 2);
    issue_step(K3{}, 3);
    DFI_WAIT_VM(3 * LOADS_PER_STEP);
    asm volatile("s_barrier" ::: "memory");
    load_frags(K0{}, f0, oA0, oB0);
    int64_t s = 0;
    for (; s + 3 < nsteps; s += 4) {
      body(K0{}, f0, f1, s);
      body(K1{}, f1, f0, s + 1);
      body(K2{}, f0, f1, s + 2);
      body(K3{}, f1, f0, s + 3);
    }
    if (s < nsteps) body(K0{}, f0, f1, s);
    if (s + 1 < nsteps) body(K1{}, f1, f0, s + 1);
    if (s + 2 < nsteps) body(K2{}, f0, f1, s + 2);
    DFI_WAIT_VM(0);   // the trailing refills land in LDS before the workgroup ends
  }

  const float sgn = (slice & 1) ? -1.f : 1.f;
  float* out = part + (slice * ntri + tile) * (int64_t)(T * T);
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
      if (block_used(diag, rowA, rowB, wr * WT + i * 32, wc * WT + j * 32, n))
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = wr * WT + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
        const int col = wc * WT + j * 32 + l32;
        out[row * T + col] = sgn * acc[i][j][r];
      }
}

}  // namespace v4

// W_ij = sum over slices of the partial tiles (FP64, slice order) for i > j, plus the products of
// columns [ktail, m) that the tile kernel left out (FP64); W_ii = d_i + lambda.
// mirror != 0 also writes W_ji. A wave takes one row of a lower-triangle tile, a lane four consecutive
// columns of it (16-byte loads), eight slices in flight. Bound by the partial tiles' HBM reads. SPLIT
// (few tiles: the rows alone leave the chip idle): one row per workgroup, wave w a quarter of the slices,
// the four sums added in LDS in wave order; else 16 rows per workgroup, so that it reads 16 KB of every
// slice's tile in one piece. n = 4096, 32 slices (1.07 GB): 353 us with 4-byte loads a row per workgroup,
// 266 now (4.0 TB/s); n = 256, 241 slices: 29 against 10. The line between the forms: at n = 1024 (10
// tiles) both take 20 us, at n = 2048 (36) split takes 47, unsplit 34.
constexpr int RED_ROWS = 16;
template <bool SPLIT>
__device__ __forceinline__ void gram_reduce_body(const float* __restrict__ part, int64_t n, int64_t ntri, int64_t nslice,
                                                 const double* __restrict__ d, double lambda, double* __restrict__ W,
                                                 int mirror, const float* __restrict__ S, int64_t lds, int64_t ktail,
                                                 int64_t m, int64_t w) {
  constexpr int ROWS = SPLIT ? 1 : RED_ROWS;
  __shared__ double sums[SPLIT ? 4 : ROWS][T];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t tile = w / (T / ROWS);
  const int r = (int)(w - tile * (T / ROWS)) * ROWS + (SPLIT ? 0 : wave);
  int64_t ti, tj;
  tri_index(tile, ti, tj);
  ti = uni64(ti);
  tj = uni64(tj);
  const int64_t i = ti * T + r;
  const int64_t sstride = ntri * (int64_t)(T * T / 4);
  const int64_t j0 = tj * T + 4 * lane;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  if (i < n && j0 <= i && j0 < n) {   // (blocks above the diagonal or past n are not stored)
    const f32x4* pp = reinterpret_cast<const f32x4*>(part + tile * (int64_t)(T * T) + r * T) + lane;
    const int64_t s1 = SPLIT ? (wave + 1) * nslice / 4 : nslice;
    int64_t sl = SPLIT ? wave * nslice / 4 : 0;
    for (; sl + 8 <= s1; sl += 8) {
      f32x4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = pp[(sl + u) * sstride];
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] += (double)v[u][e];
    }
    if (sl < s1) {
      // the last few: loaded together too, in place of the missing ones the last slice again, not added
      f32x4 v[7];
#pragma unroll
      for (int u = 0; u < 7; ++u) v[u] = pp[min<int64_t>(sl + u, s1 - 1) * sstride];
#pragma unroll
      for (int u = 0; u < 7; ++u)
        if (sl + u < s1)
#pragma unroll
          for (int e = 0; e < 4; ++e) s[e] += (double)v[u][e];
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) sums[wave][4 * lane + e] = s[e];
  __syncthreads();
  if (i >= n) return;
  // columns c, c + 64, ... of the row (split: one column per thread)
#pragma unroll
  for (int e = 0; e < (SPLIT ? 1 : 4); ++e) {
    const int c = SPLIT ? (int)threadIdx.x : lane + 64 * e;
    const int64_t j = tj * T + c;
    if (j > i || j >= n) return;
    double v = SPLIT ? sums[0][c] + sums[1][c] + sums[2][c] + sums[3][c] : sums[wave][c];
    if (i == j) v = d[i] + lambda;
    else
      for (int64_t k = ktail; k < m; ++k) v += (double)S[i * lds + k] * (double)S[j * lds + k];
    W[i * n + j] = v;
    if (mirror && i != j) W[j * n + i] = v;
  }
}

template <bool SPLIT>
__global__ void __launch_bounds__(SPLIT ? 256 : 64 * RED_ROWS)
gram_reduce_kernel(const float* __restrict__ part, int64_t n, int64_t ntri, int64_t nslice,
                   const double* __restrict__ d, double lambda, double* __restrict__ W, int mirror,
                   const float* __restrict__ S, int64_t lds, int64_t ktail, int64_t m) {
  gram_reduce_body<SPLIT>(part, n, ntri, nslice, d, lambda, W, mirror, S, lds, ktail, m, blockIdx.x);
}

// many problems' reductions in one launch (lower triangles, no columns left out)
template <bool SPLIT>
__global__ void __launch_bounds__(SPLIT ? 256 : 64 * RED_ROWS) gram_reduce_jobs_kernel(JobList<GramReduceJob> l) {
  const int k = job_of(l, blockIdx.x);
  const GramReduceJob& j = l.job[k];
  gram_reduce_body<SPLIT>(j.part, j.n, j.ntri, j.nslice, j.d, j.lambda, j.W, 0, nullptr, 0, 0, 0, blockIdx.x - l.blk0[k]);
}

// FP32 products by gram_kernel_v2: eight rows lie within one buffer of 2^32 bytes.
bool use_v2(const GramPlan& p) { return p.prec == 0 && p.lds < ((int64_t)1 << 27); }

}  // namespace

GramPlan gram_plan(int64_t n, int64_t m, int64_t lds, int prec, bool aligned16, int q_override, int split_mode) {
  GramPlan p{};
  p.n = n;
  p.m = m;
  p.lds = lds;
  p.prec = prec;
  p.ntile = (n + T - 1) / T;
  p.ntri = p.ntile * (p.ntile + 1) / 2;
  // The base plan: slices per XCD (q), enough workgroups to fill 256 CUs several times with little tail,
  // while keeping at least ~2048 columns per slice.
  const int64_t maxq_cols = std::max<int64_t>(1, m / (8 * 2048));
  int64_t best_q = 1;
  double best_score = -1.0;
  for (int64_t q = 1; q <= 64; ++q) {
    if (q > maxq_cols && q > 1) break;
    const int64_t wgs = 8 * q * p.ntri;
    const int64_t rounds = (wgs + 255) / 256;
    const double eff = (double)wgs / (double)(rounds * 256);
    // prefer >= 4 rounds, then efficiency
    const double score = eff * (rounds >= 4 ? 1.0 : 0.5 + 0.125 * (double)rounds);
    if (score > best_score + 1e-9) {
      best_score = score;
      best_q = q;
    }
  }
  // (planes also for rows that are not 16-byte aligned: 1000 x 99999 row pass 149 + Gram 336 us, against 69 + 673 with the
  // split in the tile kernel)
  p.ldh = (prec == 1 && split_mode != 0) ? split_ldh(m) : 0;
  const int64_t cap = prec == 2 ? fp8_ldq(m) : (p.ldh > 0 ? p.ldh : m);   // columns the slices cover
  const int64_t kstep = (prec == 2) ? 64 : KS;
  auto columns = [&](int64_t ns) { return std::max<int64_t>(1, ((cap + ns - 1) / ns + kstep - 1) / kstep) * kstep; };
  p.nslice = 8 * (q_override > 0 ? (int64_t)q_override : best_q);
  if (q_override == 0) {
    // Then the cheapest of the base plan and the slice counts that just fill 1, 2, ... rounds of 256
    // workgroups. A round takes the columns of a slice at the tile kernel's rate on a full chip, every
    // work item writes and the reduction reads 256 KB of partials. (The base plan leaves most of the chip
    // idle for small n, and a round nearly empty where ntri is a little over a multiple of 32: at
    // n = 256, m = 1e5 FP32 48 workgroups took 550 us with the reduction, 241 take 140; at n = 2048, m = 1e4
    // split-BF16 288 took 220, 504 take 167.) Measured rates, us a column and tile: FP32 0.227
    // (0.258 unaligned rows; 0.34 in gram_kernel), split-BF16 from planes 0.075, inside the kernel 0.16, FP8 0.0141.
    // Never fewer slices than the base plan: a slice is summed in FP32 and the slices in FP64. (FP8 at n = 4096, m = 1e5:
    // 9 slices would take 905 us where 32 take 1200, but with 3.5 times as many products a sum in FP32; the codes of a
    // one-signed S, n = 300, m = 1e5, miss their exact Gram by 1.67e-6 with 8 slices, 1.65e-6 with 32.) Split-BF16
    // keeps an even count: odd slices are negated against the accumulation's bias.
    const double rate =
        prec == 2 ? 0.0141 : prec == 0 ? (use_v2(p) ? (aligned16 ? 0.227 : 0.258) : 0.34) : (p.ldh > 0 ? 0.075 : 0.16);
    auto cost = [&](int64_t ns) {
      const int64_t ks = columns(ns), slices = (cap + ks - 1) / ks, items = p.ntri * slices;
      const double u = (double)ks * rate + 3.0;
      double t = (double)((items + 255) / 256) * u;
      if (use_v2(p)) {   // a diagonal tile costs 9 / 16 of another, and they come last
        const int64_t off = (p.ntri - p.ntile) * slices, dia = p.ntile * slices;
        const double d = 0.5625 * (double)ks * rate + 3.0;
        t = off == 0 ? (double)((dia + 255) / 256) * d
                     : std::max((double)((off + 255) / 256) * u, ((double)off * u + (double)dia * d) / 256.0 + 0.5 * d);
      }
      return t + 0.145 * (double)items;
    };
    const int64_t lo = p.nslice;
    double best = cost(p.nslice);
    auto consider = [&](int64_t ns) {
      if (prec == 1) ns &= ~(int64_t)1;
      if (ns <= lo || columns(ns) < 256 || p.ntri * ns > 4352) return;
      const double c = cost(ns);
      if (c < best - 1e-9) {
        best = c;
        p.nslice = ns;
      }
    };
    for (int64_t r = 1; r < 8; ++r) consider(32 * r / p.ntri);   // (an eighth of the chip, ...)
    for (int64_t r = 1; r <= 17; ++r) consider(256 * r / p.ntri);
    if (use_v2(p) && p.ntile > 1)
      for (int64_t r = 1; r <= 17; ++r) consider(256 * r / (p.ntri - p.ntile));
  }
  p.kslice = columns(p.nslice);
  if (q_override <= 0) {   // no slice past the last column
    const int64_t used = (cap + p.kslice - 1) / p.kslice;
    p.nslice = prec == 1 ? (used + 1) & ~(int64_t)1 : used;
  }
  p.part_bytes = (size_t)p.nslice * (size_t)p.ntri * (size_t)(T * T) * sizeof(float);
  return p;
}

void gram_q_candidates(int64_t n, int64_t m, size_t max_part_bytes, int* out, int* count, int cap) {
  const int64_t ntile = (n + T - 1) / T;
  const int64_t ntri = ntile * (ntile + 1) / 2;
  const int64_t maxq = std::max<int64_t>(1, m / (8 * 2048));
  const int64_t fill = std::min<int64_t>(m / (8 * 256), 4352 / (8 * ntri));   // the limits of the built-in plan's slices
  static const int qs[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64};
  int c = 0;
  for (int q : qs) {
    if (q > 1 && q > std::max(maxq, fill)) break;
    if (q > 1 && (size_t)8 * q * ntri * T * T * sizeof(float) > max_part_bytes) break;
    if (c < cap) out[c++] = q;
  }
  *count = c;
}

hipError_t gram_launch_fp8(const GramPlan& p, const uint8_t* q, const uint8_t* sc, int64_t ldq, float* part,
                           hipStream_t st) {
  const dim3 grid((unsigned)(8 * items_per_xcd(p.ntri, p.nslice)));
  if ((ldq & 127) != 0 || ldq < p.m || p.nslice * p.kslice < ldq || (p.kslice & 63) != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(v3::gram_kernel_fp8, grid, dim3(v3::NT), 0, st, q, sc, p.n, ldq, p.ntri, p.nslice, p.kslice,
                     part);
  return hipGetLastError();
}

hipError_t gram_launch_fp8_grouped(const GramJob* jobs_dev, int njobs, int64_t nwg, hipStream_t st) {
  if (njobs < 1 || nwg < 1 || nwg > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(v3::gram_kernel_fp8_grouped, dim3((unsigned)nwg), dim3(v3::NT), 0, st, jobs_dev, njobs);
  return hipGetLastError();
}

hipError_t gram_launch_split(const GramPlan& p, const uint16_t* hi, const uint16_t* lo, float* part, hipStream_t st) {
  if (p.prec != 1 || p.ldh <= 0 || (p.ldh & 63) != 0) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(8 * items_per_xcd(p.ntri, p.nslice)));
  if (p.nslice * p.kslice < p.ldh || (p.kslice & 15) != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(v4::gram_kernel_split, grid, dim3(v4::NT), 0, st, hi, lo, p.n, p.ldh, p.ntri, p.nslice,
                     p.kslice, part);
  return hipGetLastError();
}

// Which tile kernel runs for an FP32 input S, and the first column it leaves to the reduction:
//   * FP32 products: v2 (direct-to-LDS), 16-byte aligned rows by 16 bytes, columns [0, m rounded down to 4); other rows by
//     4 bytes (four times the loads: 1024 x 99999 1030 us, aligned 905, v1 1340), all columns;
//   * split-BF16 without planes, or rows of 2^27 columns: v1 (register staging, conversion on the LDS store), all columns.
// (For split-BF16 the register-staged kernel converts each element once per workgroup; v2 would
// convert it once per reading wave, which measured slower.)
static bool vec_rows(const GramPlan& p, const float* S) {
  return ((p.lds & 3) == 0) && ((reinterpret_cast<uintptr_t>(S) & 15) == 0);
}

static int64_t tail_start(const GramPlan& p, const float* S) {
  if (p.prec == 2) return p.m;   // the FP8 kernel covers every column (zero codes past m)
  if (p.prec == 1 && p.ldh > 0) return p.m;   // the plane kernel covers every column (zeros past m)
  return use_v2(p) && vec_rows(p, S) ? (p.m & ~(int64_t)3) : p.m;
}

hipError_t gram_launch(const GramPlan& p, const float* S, float* part, hipStream_t st) {
  const bool vec = vec_rows(p, S);
  const dim3 grid((unsigned)(8 * items_per_xcd(p.ntri, p.nslice)));
  const dim3 grid2((unsigned)(8 * (v2::v2_per_xcd(p.ntri - p.ntile, p.nslice) + v2::v2_per_xcd(p.ntile, p.nslice))));
  if (use_v2(p) && vec) {
    hipLaunchKernelGGL(v2::gram_kernel_v2, grid2, dim3(v2::NT), 0, st, S, p.n, p.lds, p.m, p.ntile, p.nslice, p.kslice, part);
  } else if (use_v2(p)) {
    hipLaunchKernelGGL(v2::gram_kernel_v2_words, grid2, dim3(v2::NT), 0, st, S, p.n, p.lds, p.m, p.ntile, p.nslice, p.kslice, part);
  } else if (p.prec == 0) {
    hipLaunchKernelGGL((gram_kernel<0, false>), grid, dim3(NTHR), 0, st, S, p.n, p.lds, p.m, p.ntri, p.nslice, p.kslice, part);
  } else if (vec) {
    hipLaunchKernelGGL((gram_kernel<1, true>), grid, dim3(NTHR), 0, st, S, p.n, p.lds, p.m, p.ntri, p.nslice, p.kslice, part);
  } else {
    hipLaunchKernelGGL((gram_kernel<1, false>), grid, dim3(NTHR), 0, st, S, p.n, p.lds, p.m, p.ntri, p.nslice, p.kslice, part);
  }
  return hipGetLastError();
}

hipError_t gram_reduce(const GramPlan& p, const float* S, const float* part, const double* d, double lambda,
                       double* W, int mirror, hipStream_t st) {
  const int64_t ktail = tail_start(p, S);   // first column the tile kernel left out
  if (p.ntri <= 16)   // n <= 1280
    hipLaunchKernelGGL(gram_reduce_kernel<true>, dim3((unsigned)(p.ntri * T)), dim3(256), 0, st, part, p.n, p.ntri,
                       p.nslice, d, lambda, W, mirror, S, p.lds, ktail, p.m);
  else
    hipLaunchKernelGGL(gram_reduce_kernel<false>, dim3((unsigned)(p.ntri * (T / RED_ROWS))), dim3(64 * RED_ROWS), 0, st,
                       part, p.n, p.ntri, p.nslice, d, lambda, W, mirror, S, p.lds, ktail, p.m);
  return hipGetLastError();
}

hipError_t gram_reduce_jobs(const GramReduceJob* jobs, int count, hipStream_t st) {
  using L = JobList<GramReduceJob>;
  std::vector<GramReduceJob> small, large;   // the form of gram_reduce
  for (int k = 0; k < count; ++k) (jobs[k].ntri <= 16 ? small : large).push_back(jobs[k]);
  const hipError_t e = launch_jobs(small.data(), (int)small.size(), [](const GramReduceJob& j) { return j.ntri * T; },
                                   [&](const L& l, unsigned b) {
                                     hipLaunchKernelGGL(gram_reduce_jobs_kernel<true>, dim3(b), dim3(256), 0, st, l);
                                   });
  if (e != hipSuccess) return e;
  return launch_jobs(large.data(), (int)large.size(), [](const GramReduceJob& j) { return j.ntri * (T / RED_ROWS); },
                     [&](const L& l, unsigned b) {
                       hipLaunchKernelGGL(gram_reduce_jobs_kernel<false>, dim3(b), dim3(64 * RED_ROWS), 0, st, l);
                     });
}

}  // namespace dfi
