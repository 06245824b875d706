// Weight GEMMs of the fused rows (Algorithm 2's GEMM calls over [buffer + offset, size), Section V-C).
//
// y[m][n] = sum_k x[m][k] W[n][k], fp32 accumulation, M = live rows (small), W streamed once from HBM.
// The work is HBM-bound for M up to a few hundred (M flop per weight byte), so the design goal is to stream W
// at full bandwidth:
//   * W is re-tiled once at init into MFMA operand order: tile (n-tile of 16 columns, k-block of 32) is 1 KiB,
//     lane l holds W[n0 + l%16][k0 + 8*(l/16) .. +8], so every wave load is one contiguous, fully used 1 KiB;
//     tiles are ordered [column group of NT n-tiles][k-block][n-tile in group], so the K slice a wave streams is
//     one contiguous run of memory (NT KiB per k-block).
//   * a column group (NT n-tiles: 32 columns, or 64 for very wide matrices) x one K slice x all rows of
//     a row block is the unit of work; up to 16 rows one wave takes it and reads the rows' operand straight from L2/L1
//     (no LDS, no barriers); above that the rows' operand is staged through LDS once per block of 4 column groups and
//     shared by the block's 4 or 8 waves.
//   * matrices whose result a row-wise kernel would only finish (q|k|v, GELU input) and narrow gate|up matrices, K of moderate length:
//     all of K in a block, the slices in its waves, the job finished by it; a block per 32 columns up to 128 rows
//     (gemm16_whole_kernel), above that gemm16_parts_kernel.
//   * more than 128 rows (context passes, very wide windows): the contraction turns MFMA- and operand-bound.  A wave keeps
//     a 128 x 64 output tile and a block covers 256 rows x 256 columns (gemm16_rows_kernel), or, where such blocks would
//     leave the chip idle, smaller blocks, either with both operands in LDS (gemm16_tile_kernel) or, in context passes of few blocks,
//     with K in parts and the weights straight to registers (gemm16_parts_kernel); context_plan picks the block by a cost
//     model.  Taken in one slice, the kernel finishes the job itself: residual add, activation, or rotary and append.
//     Row blocks of one (column block, K slice) get workgroup ids that land on the same XCD, so the weight tiles cross HBM
//     once and are L2 hits for the others.
//   * split-K: for the fused iteration slice count and boundaries depend on (N, K) only -- never on M -- and partial
//     sums are written per slice and added by the consumer in slice order, so a row's result does not depend on which
//     other rows are live (the paper's premise that fused requests undergo identical operations).  A context pass
//     holds rows of one request and is sliced by that request's row count too (context_plan): few slices at hundreds
//     of rows, where the fp32 partial sums would outweigh the weights, more for short prompts.
//   * MFMA v_mfma_f32_16x16x32_{bf16,f16}: A = 16 columns of W, B = 16 rows of x, 32-deep: the accumulator tile is
//     y^T, so a lane holds 4 consecutive output columns of one row and stores them as one 16-byte write.
//   * gate|up of a gated MLP, up to 128 fused rows: no partial sums at all -- the two K halves (or the whole kernel's four slices)
//     are wave sets of a block and the activation is the kernel's epilogue (gated_lds_kernel), with gate and up columns
//     interleaved in the layout so that a lane holds both; above 128 rows the same slices go through memory.
// fp32 models (tiny configurations only) use a plain FMA kernel on the untiled matrix, with what follows the contraction as
// its epilogue.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "flover_dev.h"
#include "flover_kernels.h"

namespace flk {

// ---------------------------------------------------------------- re-tiling (init time)

__global__ void retile16_kernel(const uint16_t* __restrict__ W, u32x4_t* __restrict__ wt, int N, int K, int KB,
                                int ntile0, int tstep, int NT, long total) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  int lane = (int)(i & 63);
  long t = i >> 6;
  int kb = (int)(t % KB);
  int ntile = (int)(t / KB);
  int n = ntile * 16 + (lane & 15);
  int k = kb * 32 + (lane >> 4) * 8;
  u32x4_t v = {0u, 0u, 0u, 0u};
  if (n < N) v = *(const u32x4_t*)(W + (size_t)n * K + k);
  const int tile = ntile0 + ntile * tstep, g = tile / NT, tt = tile - g * NT;
  wt[(((size_t)g * KB + kb) * NT + tt) * 64 + lane] = v;
}

// ---------------------------------------------------------------- 16-bit MFMA kernel

// Columns n .. n+3 of a row of ldc fp32 results: partial sums (rows padded to whole fours), or a caller's rows, which may have any
// length and start at any element.
__device__ __forceinline__ void store_sums(float* row, int n, int ldc, const f32x4_t& v) {
  if (n + 4 <= ldc) *(f32x4_any*)(row + n) = v;
  else {
#pragma unroll
    for (int e = 0; e < 3; ++e)
      if (n + e < ldc) row[n + e] = v[e];
  }
}

// ---- direct variant: 4 independent waves per block, no LDS, no barriers; the rows' operand comes straight from L2/L1.
// grid = (ceil(ngroups/4), S, row blocks), block = 256; a wave owns NT n-tiles (16*NT columns) x one K slice x 16*MT rows.
// W is prefetched PFW k-blocks ahead, x PFA k-blocks ahead (PFW % PFA == 0).
template <int DT, int MT, int NT, int PFW, int PFA>
__global__ __launch_bounds__(256) void gemm16_direct_kernel(const uint16_t* __restrict__ x, const u32x4_t* __restrict__ wt,
                                                            float* __restrict__ part, int M, int N, int K, int ngroups,
                                                            int KB, int kbs, size_t slice_stride, int ldc,
                                                            int xmtt) {
  static_assert(PFW % PFA == 0, "ring shapes");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = blockIdx.x * 4 + wave;
  if (g >= ngroups) return;
  const int s = blockIdx.y;
  const int m0 = blockIdx.z * (16 * MT);
  const int kb0 = s * kbs;
  const int kb1 = min(KB, kb0 + kbs);

  f32x4_t acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[i][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const u32x4_t* wp = wt + ((size_t)g * KB) * NT * 64 + lane;                    // + (kb*NT + t)*64
  // rows' operand: row-major [M][K] (xmtt == 0) or fragment order with xmtt row tiles per k-block
  const size_t tstride = xmtt ? 512 : (size_t)16 * K, kstride = xmtt ? (size_t)xmtt * 512 : 32;
  static_assert(MT == 1, "row-major rows past M repeat the last one, here for one tile");
  const uint16_t* xp = xmtt ? x + (size_t)(m0 >> 4) * 512 + lane * 8
                            : x + (size_t)min(m0 + (lane & 15), M - 1) * K + (lane >> 4) * 8;     // + i*tstride + kb*kstride

  u32x4_t bq[PFW][NT], aq[PFA][MT];
  static_assert(PFW == PFA, "both rings turn together");
#pragma unroll
  for (int j = 0; j < PFW; ++j) {      // same order as the refills in the loop: the wait counts of the first turn match
    const int kk = min(kb0 + j, kb1 - 1);
#pragma unroll
    for (int t = 0; t < NT; ++t) bq[j][t] = __builtin_nontemporal_load(wp + ((size_t)kk * NT + t) * 64);
#pragma unroll
    for (int i = 0; i < MT; ++i) aq[j][i] = *(const u32x4_any*)(xp + i * tstride + kk * kstride);
    __builtin_amdgcn_sched_barrier(0);
  }
  // One turn of the ring.  The steady-state turns (TAIL = false: all PFW k-blocks exist) are free of branches, so the
  // compiler's wait counts for the in-order memory counter stay exact; sched_barrier keeps each refill where it is
  // written, right after the k-block that freed the slot.
  auto turn = [&](auto tail_, int kb) {
    constexpr bool tail = decltype(tail_)::value;
#pragma unroll
    for (int j = 0; j < PFW; ++j) {
      if (!tail || kb + j < kb1) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int t = 0; t < NT; ++t) acc[i][t] = mfma16<DT>(bq[j][t], aq[j % PFA][i], acc[i][t]);
      }
      if (!tail) {
        const int kw = min(kb + j + PFW, kb1 - 1);    // the last turns re-read the last block (in bounds, unused)
#pragma unroll
        for (int t = 0; t < NT; ++t) bq[j][t] = __builtin_nontemporal_load(wp + ((size_t)kw * NT + t) * 64);
        const int ka = min(kb + j + PFA, kb1 - 1);
#pragma unroll
        for (int i = 0; i < MT; ++i) aq[j % PFA][i] = *(const u32x4_any*)(xp + i * tstride + ka * kstride);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  int kb = kb0;
  for (; kb + PFW <= kb1; kb += PFW) turn(std::false_type{}, kb);
  if (kb < kb1) turn(std::true_type{}, kb);
  float* out = part + (size_t)s * slice_stride;
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int n = (g * NT + t) * 16 + (lane >> 4) * 4, m = m0 + i * 16 + (lane & 15);
      if (m < M) store_sums(out + (size_t)m * ldc, n, ldc, acc[i][t]);
    }
}

// The rows' operand of a chunk (KC k-blocks x MT row tiles) on its way to LDS: KC * MT pieces of 1 KiB, one wave load each, shared
// out to NW waves, up to FPW of them per wave (surplus ones repeat the last: same data, no branch).  Fragment order: a piece is a
// fragment.  Row-major: a piece is the chunk's 64 * KC bytes of 16 / KC rows, whole cache lines, which the store spreads over KC
// fragments -- sixteen rows' 64 bytes at a time, as the MFMA wants them, meet in the same cache channel where the row length is
// a power of two (call with SwiGLU, 11008 x 4096 at 40 / 70 / 101 / 128 rows: 54.9 / 60.7 / 67.6 / 75.5 -> 51.2 / 54.2 / 58.7 / 61.3 us;
// 50257 x 2048 at 100 rows 74.7 -> 57.8, the second launch counted).  In LDS a fragment's rows are permuted by an exclusive or (place()), so that neither the spread
// stores nor the reads collide.
template <int KC, int MT, int NW>
struct ChunkRows {
  static constexpr int FPW = (KC * MT + NW - 1) / NW, PIECES = 4 * KC;    // PIECES: 16-byte pieces of a row in a chunk
  const uint16_t* x;
  uint32_t step, limit;                          // elements per k-block, and the last offset a load may take
  uint32_t from[FPW], ahead[FPW], to[FPW];       // row (tile) in x, element within the chunk, place in the LDS buffer
  static __device__ int place(int kc, int quad, int row) { return quad * 16 + (row ^ ((kc & 1) * 4 + quad)); }   // row < 16
  // rows: how many there are (those past the last repeat it); K: their length; kend: end of the slice in k-blocks, past which its
  // last block is loaded again
  __device__ ChunkRows(const uint16_t* x_, int rows, int K, int kend, int xmtt, int w, int lane) : x(x_) {
    step = xmtt ? (uint32_t)xmtt * 512 : 32;
    limit = xmtt ? (uint32_t)(kend - 1) * step : (uint32_t)kend * 32 - 8;
#pragma unroll
    for (int j = 0; j < FPW; ++j) {
      const int f = min(w + NW * j, KC * MT - 1);
      if (xmtt) {
        from[j] = (f % MT) * 512 + lane * 8;
        ahead[j] = (f / MT) * step;
        to[j] = f * 64 + place(f / MT, lane >> 4, lane & 15);
      } else {
        const int row = f * (16 / KC) + lane / PIECES, p = lane % PIECES;
        from[j] = (uint32_t)min(row, rows - 1) * K;
        ahead[j] = p * 8;
        to[j] = ((p >> 2) * MT + (row >> 4)) * 64 + place(p >> 2, p & 3, row & 15);
      }
    }
  }
  __device__ void load(u32x4_t (&r)[FPW], int kb) const {      // the chunk that starts at k-block kb
#pragma unroll
    for (int j = 0; j < FPW; ++j) r[j] = *(const u32x4_any*)(x + (from[j] + min(kb * step + ahead[j], limit)));
  }
  __device__ void store(u32x4_t* buf, const u32x4_t (&r)[FPW]) const {
#pragma unroll
    for (int j = 0; j < FPW; ++j) buf[to[j]] = r[j];
  }
};

// ---- larger M (17..128 rows per block): the rows' operand is staged through LDS once per block and shared by its
// waves; a block covers GPB = 4 column groups (256 columns; 128 for matrices laid out in 32-column groups), each group
// by NT/NTW waves that own NTW of its n-tiles and stream their W tiles from HBM into registers, PF k-blocks ahead.
// From 33 rows up a wave owns 32 columns (8 waves per 256-column block): a single wave issues MFMAs at about 60% of
// the unit's rate, two waves per SIMD interleave and also hide each other's LDS and memory waits.
// LDS holds the x tile in MFMA fragment order ([k-block][m-tile][lane] x 16 B), so every ds_read_b128 of a fragment
// is 1 KiB contiguous and bank-conflict free.  Double-buffered chunks of KC k-blocks, one barrier per chunk.
// The per-(m, n) arithmetic (MFMA sequence over k) is identical to the direct kernel's.
template <int DT, int MT, int NT, int NTW, int KC, int PF, int GPB>
__global__ __launch_bounds__(64 * GPB * (NT / NTW)) void gemm16_lds_kernel(const uint16_t* __restrict__ x,
                                                                         const u32x4_t* __restrict__ wt,
                                                                         float* __restrict__ part, int M, int N, int K,
                                                                         int ngroups, int KB, int kbs,
                                                                         size_t slice_stride, int ldc, int nx,
                                                                         int nslices, int nz, int xmtt) {
  static_assert(PF % KC == 0 && NT % NTW == 0, "ring and tile shapes");
  constexpr int WPG = NT / NTW;                  // waves that share one column group, each taking NTW of its n-tiles
  constexpr int NW = GPB * WPG;                  // waves per block: GPB column groups (256 columns)
  __shared__ u32x4_t lds[2][KC * MT * 64];
  typedef ChunkRows<KC, MT, NW> Rows;
  constexpr int CPR = PF / KC;                   // chunks per turn of the W ring
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // 1-D grid, XCD-aware: workgroup ids go round-robin over the 8 XCDs (each with its own L2), so the row blocks of one
  // (column block, K slice) task are given ids 8 apart -- same XCD, dispatched back to back -- and the W tiles one of
  // them pulls from HBM are L2 hits for the others.  With a single row block this is the identity mapping.
  const int xcd = blockIdx.x & 7, qq = blockIdx.x >> 3;
  const int zb = qq % nz, task = (qq / nz) * 8 + xcd;
  if (task >= nx * nslices) return;              // padding of the grid (whole block)
  const int bx = task % nx, s = task / nx;
  const int g = bx * GPB + wave / WPG, sub = wave % WPG;
  const int gl = min(g, ngroups - 1);            // surplus waves repeat the last group (they still serve the barriers)
  const int m0 = zb * (16 * MT);
  const int kb0 = s * kbs;
  const int kb1 = min(KB, kb0 + kbs);
  const int nchunks = (kb1 - kb0 + KC - 1) / KC;

  f32x4_t acc[MT][NTW];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int t = 0; t < NTW; ++t) acc[i][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const u32x4_t* wp = wt + (((size_t)gl * KB) * NT + sub * NTW) * 64 + lane;     // + (kb*NT + t)*64
  const Rows rows(x + (xmtt ? (size_t)(m0 >> 4) * 512 : (size_t)m0 * K), M - m0, K, kb1, xmtt, wave, lane);
  int at[2];                                     // where a lane finds its part of a fragment, even and odd k-blocks of a chunk
#pragma unroll
  for (int kc = 0; kc < 2; ++kc) at[kc] = Rows::place(kc, lane >> 4, lane & 15);
  u32x4_t bq[PF][NTW], areg[Rows::FPW];
#pragma unroll
  for (int j = 0; j < PF; ++j) {
    const int kk = min(kb0 + j, kb1 - 1);
#pragma unroll
    for (int t = 0; t < NTW; ++t) bq[j][t] = __builtin_nontemporal_load(wp + ((size_t)kk * NT + t) * 64);
  }
  auto load_a = [&](int chunk) { rows.load(areg, kb0 + chunk * KC); };
  auto store_a = [&](int buf) { rows.store(lds[buf], areg); };
  load_a(0);
  store_a(0);
  __syncthreads();
  // One chunk: stage the next x tile, multiply this one, refill the W ring.  CC (position in the ring turn) is a
  // compile-time value; TAIL = the chunk may be the last one or short.  The steady-state loop below only runs
  // chunks that are full and have a successor, so its body is free of branches: the compiler's wait counts for the
  // in-order memory counter stay exact there (any branch in the body makes them collapse to "wait for all").
  auto chunk = [&](auto cc_, auto tail_, int c) {
    constexpr int cc = decltype(cc_)::value;
    constexpr bool tail = decltype(tail_)::value;
    const bool more = !tail || c + 1 < nchunks;
    if (more) load_a(c + 1);
    __builtin_amdgcn_sched_barrier(0);        // keep these loads ahead of the chunk's MFMAs (the scheduler sinks them to their use)
    const u32x4_t* la = lds[c & 1];
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
      const int kb = kb0 + c * KC + kc;
      if (!tail || kb < kb1) {
        u32x4_t af[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) af[i] = la[(kc * MT + i) * 64 + at[kc & 1]];
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int t = 0; t < NTW; ++t) acc[i][t] = mfma16<DT>(bq[cc * KC + kc][t], af[i], acc[i][t]);
      }
      const int kk = min(kb + PF, kb1 - 1);
#pragma unroll
      for (int t = 0; t < NTW; ++t) bq[cc * KC + kc][t] = __builtin_nontemporal_load(wp + ((size_t)kk * NT + t) * 64);
      __builtin_amdgcn_sched_barrier(0);      // refill right after the k-block that freed the slot
    }
    if (more) store_a((c + 1) & 1);
    __syncthreads();
  };
  int c = 0;
  for (; c + CPR < nchunks; c += CPR) {
    if constexpr (CPR >= 1) chunk(std::integral_constant<int, 0>{}, std::false_type{}, c);
    if constexpr (CPR >= 2) chunk(std::integral_constant<int, 1>{}, std::false_type{}, c + 1);
    if constexpr (CPR >= 3) chunk(std::integral_constant<int, 2>{}, std::false_type{}, c + 2);
    if constexpr (CPR >= 4) chunk(std::integral_constant<int, 3>{}, std::false_type{}, c + 3);
  }
  for (; c < nchunks; c += CPR) {               // the last turn of the ring
    if constexpr (CPR >= 1) if (c < nchunks) chunk(std::integral_constant<int, 0>{}, std::true_type{}, c);
    if constexpr (CPR >= 2) if (c + 1 < nchunks) chunk(std::integral_constant<int, 1>{}, std::true_type{}, c + 1);
    if constexpr (CPR >= 3) if (c + 2 < nchunks) chunk(std::integral_constant<int, 2>{}, std::true_type{}, c + 2);
    if constexpr (CPR >= 4) if (c + 3 < nchunks) chunk(std::integral_constant<int, 3>{}, std::true_type{}, c + 3);
  }
  if (g >= ngroups) return;
  float* out = part + (size_t)s * slice_stride;
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int t = 0; t < NTW; ++t) {
      const int n = (g * NT + sub * NTW + t) * 16 + (lane >> 4) * 4, m = m0 + i * 16 + (lane & 15);
      if (m < M) store_sums(out + (size_t)m * ldc, n, ldc, acc[i][t]);
    }
}

// A wave that does nothing but bring the rows' operand to LDS, a chunk ahead of the waves that multiply; barriers as theirs.  It stores
// a chunk into the buffer whose last fragments the others have read before the barrier behind them.
template <typename Rows>
__device__ __forceinline__ void stage_rows(const Rows& rows, u32x4_t* even, u32x4_t* odd, int kb0, int KC, int nchunks) {
  u32x4_t r[Rows::FPW];
  rows.load(r, kb0);
  rows.store(even, r);
  if (nchunks > 1) rows.load(r, kb0 + KC);
  __syncthreads();
  for (int c = 0; c < nchunks; ++c) {
    if (c + 1 < nchunks) {
      rows.store(c & 1 ? even : odd, r);
      if (c + 2 < nchunks) rows.load(r, kb0 + (c + 2) * KC);
    }
    __syncthreads();
  }
}

// ---- gated MLP input (fused iterations of 16-bit gated models): the gate|up contraction with the activation as its
// epilogue, so that neither partial sums nor the two projections reach memory and the activation needs no launch.
// The matrix is laid out in "paired" groups of 32 columns -- group j = [gate columns 16j..16j+15 | up columns
// 16j..16j+15] -- so a lane's accumulators of a group's two n-tiles are gate and up of the same four MLP columns.
// K is split in two halves inside the block: 2 * GPB waves = GPB column groups x 2 halves, each wave the MFMA chain over its
// half's k-blocks in order, each half with its own x tile in LDS (fragment order, double-buffered chunks of KC
// k-blocks, W ring PF k-blocks deep); at the end the second half hands its sums to the first through LDS, which adds
// first half + second half, applies silu(gate) * up and writes the result, rounded to the model dtype, as the next
// GEMM's row operand (row-major or fragment order).  The result of a row is the same for every MT and equal, bit for
// bit, to gemm() with the halves as two K slices followed by the stand-alone activation.
// Every chunk is full and the last ring turn is the only one whose chunks may lack a successor, so the steady state
// is free of branches.  Requires KB % 16 == 0.
// P > 0: P further waves per half copy the rows' operand, so that the others wait for weights alone, in the order in which they asked for
// them, and read a k-block's fragments from LDS while the one before it is multiplied (the barrier between two chunks comes ahead of the last
// k-block's products); without, all waves read LDS, then all multiply, between the same two barriers.  11008 x 4096, bf16, blocks of three
// groups, us without -> with copying waves -> and with fragments read ahead: 23 rows 30.6 -> 31.0 -> 30.4, 40 rows 32.0 -> 32.5 -> 30.7, 70 rows
// 36.0 -> 34.4 -> 33.4, 101 rows 43.0 -> 42.2 -> 40.8, 120 rows 48.1 -> 46.9 -> 46.0.  The memory (29 us at 6 rows: 6.2 TB/s) and, from 65 rows on, the
// products, 2.5 us per row tile, bound it; two rings as deep, or twice the copying waves, change nothing.  The same in gemm16_lds_kernel, whose
// waves read a fragment for one or two products only, gained nothing (12288 x 4096 at 70 / 101 rows 22.1 / 25.9 -> 21.9 / 24.9, 50257 x 2048 39.9 -> 40.6).
template <int DT, int MT, int KC, int PF, int GPB, int P>
__global__ __launch_bounds__(128 * (GPB + P)) void gated_lds_kernel(const uint16_t* __restrict__ x, const u32x4_t* __restrict__ wt,
                                                        void* __restrict__ act, int M, int F, int ngroups, int KB,
                                                        int xmtt) {
  static_assert(PF % KC == 0, "ring shape");
  // GPB column groups per block (32 columns each); without copying waves the GPB waves of a half stage its x tile
  constexpr int TILE = KC * MT * 64;             // a half's x tile
  __shared__ u32x4_t lds[4 * TILE > GPB * MT * 128 ? 4 * TILE : GPB * MT * 128];    // [half][buffer] tiles, then the hand-over
  typedef ChunkRows<KC, MT, (P > 0 ? P : GPB)> Rows;
  constexpr int CPR = PF / KC;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool stages = P > 0 && wave >= 2 * GPB;
  const int half = stages ? (wave - 2 * GPB) / (P > 0 ? P : 1) : wave / GPB, gw = wave % GPB;
  const int g = blockIdx.x * GPB + gw;
  const int gl = min(g, ngroups - 1);            // surplus waves repeat the last group (they still serve the barriers)
  const int K = KB * 32;
  const int kb0 = half * (KB >> 1), kb1 = kb0 + (KB >> 1);
  const int nchunks = (kb1 - kb0) / KC;
  if constexpr (P > 0) {
    if (stages) {
      stage_rows<Rows>(Rows(x, M, K, kb1, xmtt, (wave - 2 * GPB) % P, lane), lds + half * 2 * TILE, lds + half * 2 * TILE + TILE, kb0, KC, nchunks);
      __syncthreads();                           // the hand-over
      return;
    }
  }

  f32x4_t acc[MT][2];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int t = 0; t < 2; ++t) acc[i][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const u32x4_t* wp = wt + ((size_t)gl * KB) * 2 * 64 + lane;                    // + (kb*2 + t)*64
  const Rows rows(x, M, K, kb1, xmtt, gw, lane);
  int at[2];                                     // see gemm16_lds_kernel
#pragma unroll
  for (int kc = 0; kc < 2; ++kc) at[kc] = Rows::place(kc, lane >> 4, lane & 15);
  u32x4_t bq[PF][2], areg[Rows::FPW];
#pragma unroll
  for (int j = 0; j < PF; ++j)
#pragma unroll
    for (int t = 0; t < 2; ++t) bq[j][t] = __builtin_nontemporal_load(wp + ((size_t)(kb0 + j) * 2 + t) * 64);
  auto load_a = [&](int chunk) { rows.load(areg, kb0 + chunk * KC); };
  auto store_a = [&](int buf) { rows.store(lds + (half * 2 + buf) * TILE, areg); };
  if constexpr (P == 0) {
    load_a(0);
    store_a(0);
  }
  __syncthreads();
  u32x4_t af[P > 0 ? 2 : 1][MT];
  auto fragments = [&](u32x4_t (&f)[MT], const u32x4_t* la, int kc) {
#pragma unroll
    for (int i = 0; i < MT; ++i) f[i] = la[(kc * MT + i) * 64 + at[kc & 1]];
  };
  if constexpr (P > 0) fragments(af[0], lds + half * 2 * TILE, 0);
  // One chunk: stage the next x tile, multiply this one, refill the W ring.
  auto chunk = [&](auto cc_, auto last_, int c) {
    constexpr int cc = decltype(cc_)::value;
    constexpr bool last = decltype(last_)::value;
    const bool more = P == 0 && (!last || c + 1 < nchunks);
    if (more) load_a(c + 1);
    __builtin_amdgcn_sched_barrier(0);
    const u32x4_t* la = lds + (half * 2 + (c & 1)) * TILE;
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
      const int kb = kb0 + c * KC + kc, now = P > 0 ? (cc * KC + kc) & 1 : 0;
      if constexpr (P == 0) {
        fragments(af[0], la, kc);
      } else if (kc + 1 < KC) {
        fragments(af[now ^ 1], la, kc + 1);
      } else {
        __syncthreads();
        if (!last || c + 1 < nchunks) fragments(af[now ^ 1], lds + (half * 2 + ((c + 1) & 1)) * TILE, 0);
      }
      if constexpr (P > 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[i][t] = mfma16<DT>(bq[cc * KC + kc][t], af[now][i], acc[i][t]);
      const int kk = min(kb + PF, kb1 - 1);      // the last turn re-reads the last block (in bounds, unused)
#pragma unroll
      for (int t = 0; t < 2; ++t) bq[cc * KC + kc][t] = __builtin_nontemporal_load(wp + ((size_t)kk * 2 + t) * 64);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (more) store_a((c + 1) & 1);
    if constexpr (P == 0) __syncthreads();
  };
  auto ring_turn = [&](auto last_, int c) {
    static_assert(CPR <= 4, "chunks per ring turn");
    if constexpr (CPR >= 1) chunk(std::integral_constant<int, 0>{}, last_, c);
    if constexpr (CPR >= 2) chunk(std::integral_constant<int, 1>{}, last_, c + 1);
    if constexpr (CPR >= 3) chunk(std::integral_constant<int, 2>{}, last_, c + 2);
    if constexpr (CPR >= 4) chunk(std::integral_constant<int, 3>{}, last_, c + 3);
  };
  int c = 0;
  for (; c + CPR < nchunks; c += CPR) ring_turn(std::false_type{}, c);
  ring_turn(std::true_type{}, c);
  // second half -> first half through LDS (the x tiles are no longer read: every wave is past the last barrier)
  f32x4_t* red = (f32x4_t*)lds;
  if (half == 1) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int t = 0; t < 2; ++t) red[((gw * MT + i) * 2 + t) * 64 + lane] = acc[i][t];
  }
  __syncthreads();
  if (half == 1 || g >= ngroups) return;
  const int j = g * 16 + (lane >> 4) * 4;
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const f32x4_t gate = acc[i][0] + red[((gw * MT + i) * 2 + 0) * 64 + lane];
    const f32x4_t up = acc[i][1] + red[((gw * MT + i) * 2 + 1) * 64 + lane];
    const int m = i * 16 + (lane & 15);
    if (m < M) stv4<DT>(act, xrow_index(m, j, F, xmtt), act_swiglu(gate, up));
  }
}

// What a tile kernel does with its accumulators.
enum { EPI_PART = 0, EPI_GATED = 1, EPI_QKV = 2, EPI_ADD = 3, EPI_GELU = 4 };

// n-tile (of the block's B * WC) that a wave's u-th accumulator column holds: consecutive ones, except that the rotary
// epilogue needs the partners (i, i + d/2) of a head in one lane: accumulator columns u and u + B/2 are then d/2 apart.
template <int B, int WC, int EPI> __device__ __forceinline__ int tile_of(int wc, int u, int d) {
  if constexpr (EPI == EPI_QKV) {
    static_assert(B == 4 && WC % 2 == 0, "a head is one wave's or two waves' columns");
    if (d == 128) return (wc >> 1) * 8 + (wc & 1) * 2 + (u & 1) + (u >> 1) * 4;
  }
  return wc * B + u;
}

// What an epilogue reads (residual stream, bias, positions, rotary rows) is loaded for up to sixteen accumulators at once, before
// the first of them is finished: one after the other they cost about a microsecond per launch (six layers of 2048 columns, fp16,
// us per launch at 138 / 287 / 436 rows: q|k|v 20.3 / 21.1 / 26.2 -> 19.3 / 20.0 / 25.2, residual add of 2048 x 2048 17.1 -> 16.4 at
// 287 and 17.5 -> 16.7 at 436).
template <int DT, int A, int B, int WR, int WC, int EPI>
__device__ __forceinline__ void tile_epilogue(f32x4_t (&acc)[A][B], const TileOut& o, int M, int N, int mt0, int nt0, int wc, int s,
                                              int lane) {
  const int c4 = (lane >> 4) * 4;
  auto row = [&](int i) { return (mt0 + i) * 16 + (lane & 15); };
  auto column = [&](int u) { return (nt0 + tile_of<B, WC, EPI>(wc, u, o.d)) * 16 + c4; };
  f32x4_t bias[B];
  if constexpr (EPI == EPI_GELU || EPI == EPI_ADD || EPI == EPI_QKV) {
#pragma unroll
    for (int u = 0; u < B; ++u) bias[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (o.bias) {
#pragma unroll
      for (int u = 0; u < B; ++u) bias[u] = ldv4<DT>(o.bias, min(column(u), N - 4));
    }
  }
  if constexpr (EPI == EPI_PART) {
#pragma unroll
    for (int i = 0; i < A; ++i) {
      const int m = row(i);
      if (m >= M) continue;
      float* out = o.part + (size_t)s * o.slice_stride + (size_t)m * o.ldc;
#pragma unroll
      for (int u = 0; u < B; ++u)
        store_sums(out, column(u), o.ldc, acc[i][u]);
    }
  } else if constexpr (EPI == EPI_GATED) {      // n-tiles alternate gate and up of the same 16 MLP columns
#pragma unroll
    for (int i = 0; i < A; ++i) {
      const int m = row(i);
      if (m >= M) continue;
#pragma unroll
      for (int u = 0; u < B; u += 2) {
        const int j = ((nt0 + wc * B + u) >> 1) * 16 + c4;
        if (j < o.F) stv4<DT>(o.act, xrow_index(m, j, o.F, o.mtt), act_swiglu(acc[i][u], acc[i][u + 1]));
      }
    }
  } else if constexpr (EPI == EPI_GELU) {
#pragma unroll
    for (int i = 0; i < A; ++i) {
      const int m = row(i);
      if (m >= M) continue;
#pragma unroll
      for (int u = 0; u < B; ++u)
        if (column(u) < o.F) stv4<DT>(o.act, xrow_index(m, column(u), o.F, o.mtt), act_gelu<DT>(acc[i][u] + bias[u]));
    }
  } else if constexpr (EPI == EPI_ADD) {
    constexpr int G = A * B > 16 ? 16 / B : A;   // row tiles at a time
#pragma unroll
    for (int i0 = 0; i0 < A; i0 += G) {
      f32x4_t old[G][B];
#pragma unroll
      for (int i = 0; i < G; ++i)
#pragma unroll
        for (int u = 0; u < B; ++u) old[i][u] = ld4(o.part + (size_t)min(row(i0 + i), M - 1) * o.ldc + min(column(u), N - 4));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < G; ++i)
#pragma unroll
        for (int u = 0; u < B; ++u) {
          f32x4_t a = acc[i0 + i][u];
          if (o.bias) a += bias[u];
          if (row(i0 + i) < M && column(u) < N) *(f32x4_t*)(o.part + (size_t)row(i0 + i) * o.ldc + column(u)) = old[i][u] + a;
        }
    }
  } else {                                       // q | k | v columns of one head, rotary partners u and u + B/2
    const int H = o.H, half = o.d >> 1;
    int pos[A], slot[A];
#pragma unroll
    for (int i = 0; i < A; ++i) {
      pos[i] = o.pos[min(row(i), M - 1)];
      slot[i] = o.slot[min(row(i), M - 1)];
    }
    __builtin_amdgcn_sched_barrier(0);
    constexpr int G = A > 2 ? 2 : A;             // row tiles at a time
#pragma unroll
    for (int i0 = 0; i0 < A; i0 += G) {
      f32x4_t t0[G][B / 2], t1[G][B / 2];        // (cos, sin) of four consecutive pairs
      if (o.rope) {
#pragma unroll
        for (int i = 0; i < G; ++i)
#pragma unroll
          for (int u = 0; u < B / 2; ++u) {
            const float* tab = o.rope + ((size_t)pos[i0 + i] * half + (column(u) & (o.d - 1))) * 2;
            t0[i][u] = ld4(tab);
            t1[i][u] = ld4(tab + 4);
          }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 0; i < G; ++i) {
        const int m = row(i0 + i);
        if (m >= M) continue;
#pragma unroll
        for (int u = 0; u < B / 2; ++u) {
          const int n = column(u);
          if (n >= N) continue;
          const int t = n / H, which = o.third + t, r = n - t * H, hd = r / o.d, e = r - hd * o.d;
          f32x4_t a0 = acc[i0 + i][u], a1 = acc[i0 + i][u + B / 2];
          if (o.bias) { a0 += bias[u]; a1 += bias[u + B / 2]; }
          if (o.rope && which < 2)
            rope_rotate(a0, a1, f32x4_t{t0[i][u][0], t0[i][u][2], t1[i][u][0], t1[i][u][2]},
                        f32x4_t{t0[i][u][1], t0[i][u][3], t1[i][u][1], t1[i][u][3]});
          void* dst = which == 0 ? o.q : which == 1 ? o.kc : o.vc;
          const size_t at = which == 0 ? (size_t)m * H + r : (((size_t)slot[i0 + i] * (H / o.d) + hd) * o.Smax + pos[i0 + i]) * o.d + e;
          stv4<DT>(dst, at, a0);
          stv4<DT>(dst, at + half, a1);
        }
      }
    }
  }
}

// ---- up to 128 rows, K of moderate length (more rows: gemm16_parts_kernel): a block per column group (32 columns), all of K in one block, its S slices in the block's
// S waves, what follows the contraction as the epilogue -- no partial sums in memory and no launch that adds them up.  A wave is
// the direct kernel's: weights and rows' operand straight to registers, PF k-blocks ahead, no barrier before the hand-over of the
// sums through LDS.  They are added in slice order, so a row's bits are those of gemm() and the row-wise kernel behind it.
template <int DT, int MT, int S, int PF, int EPI>
__global__ __launch_bounds__(64 * S) void gemm16_whole_kernel(const uint16_t* __restrict__ x, const u32x4_t* __restrict__ wt, TileOut o, int M,
                                                              int N, int KB, int kbs, int xmtt) {
  __shared__ f32x4_t red[S][MT][2][64];
  const int lane = threadIdx.x & 63, s = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kb0 = s * kbs, kb1 = min(KB, kb0 + kbs), c4 = (lane >> 4) * 4;
  // the block's two n-tiles: a group of the layout (gate and up of the same columns where it is paired), or for a rotary epilogue
  // the partners (i, i + d/2) of a head
  int t0 = blockIdx.x * 2, t1 = t0 + 1;
  if (EPI == EPI_QKV && o.rope) {
    const int h = o.d >> 5;                      // n-tiles of half a head
    t0 = (int)blockIdx.x / h * 2 * h + (int)blockIdx.x % h;
    t1 = t0 + h;
  }
  const u32x4_t* w0 = wt + ((size_t)(t0 >> 1) * KB * 2 + (t0 & 1)) * 64 + lane;      // + kb * 128
  const u32x4_t* w1 = wt + ((size_t)(t1 >> 1) * KB * 2 + (t1 & 1)) * 64 + lane;
  // rows' operand: row-major (xmtt == 0; rows past M repeat the last one) or fragment order with xmtt row tiles per k-block
  const size_t kstride = xmtt ? (size_t)xmtt * 512 : 32;
  uint32_t xo[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
    xo[i] = xmtt ? (uint32_t)(i * 512 + lane * 8) : (uint32_t)min(i * 16 + (lane & 15), M - 1) * KB * 32 + (lane >> 4) * 8;
  u32x4_t bq[PF][2], aq[PF][MT];
  auto load = [&](int j, int kb) {
    const int kk = min(kb, kb1 - 1);             // past the slice: its last block once more (in bounds, unused)
    bq[j][0] = __builtin_nontemporal_load(w0 + (size_t)kk * 128);
    bq[j][1] = __builtin_nontemporal_load(w1 + (size_t)kk * 128);
#pragma unroll
    for (int i = 0; i < MT; ++i) aq[j][i] = *(const u32x4_any*)(x + xo[i] + kk * kstride);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int j = 0; j < PF; ++j) load(j, kb0 + j);
  f32x4_t acc[MT][2];
#pragma unroll
  for (int i = 0; i < MT; ++i) acc[i][0] = acc[i][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](int j) {
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      acc[i][0] = mfma16<DT>(bq[j][0], aq[j][i], acc[i][0]);
      acc[i][1] = mfma16<DT>(bq[j][1], aq[j][i], acc[i][1]);
    }
  };
  int kb = kb0;
  for (; kb + PF <= kb1; kb += PF)
#pragma unroll
    for (int j = 0; j < PF; ++j) {
      multiply(j);
      load(j, kb + j + PF);
    }
#pragma unroll
  for (int j = 0; j < PF - 1; ++j)
    if (kb + j < kb1) multiply(j);
  // what the epilogue reads, under way during the hand-over
  constexpr int OWN = (MT + S - 1) / S;          // row tiles a wave finishes: s, s + S, ...
  const int n0 = t0 * 16 + c4, n1 = t1 * 16 + c4, half = o.d >> 1;
  f32x4_t b0 = {0.f, 0.f, 0.f, 0.f}, b1 = b0;
  if ((EPI == EPI_QKV || EPI == EPI_GELU) && o.bias) {
    b0 = ldv4<DT>(o.bias, n0);
    b1 = ldv4<DT>(o.bias, n1);
  }
  int pos[OWN], slot[OWN];
  f32x4_t r0[OWN], r1[OWN];                      // (cos, sin) of four consecutive pairs
  if constexpr (EPI == EPI_QKV) {
#pragma unroll
    for (int q = 0; q < OWN; ++q) {
      const int m = min((s + q * S) * 16 + (lane & 15), M - 1);
      pos[q] = o.pos[m];
      slot[q] = o.slot[m];
    }
  }
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    red[s][i][0][lane] = acc[i][0];
    red[s][i][1][lane] = acc[i][1];
  }
  if (EPI == EPI_QKV && o.rope) {
#pragma unroll
    for (int q = 0; q < OWN; ++q) {
      const float* tab = o.rope + ((size_t)pos[q] * half + (n0 & (o.d - 1))) * 2;
      r0[q] = ld4(tab);
      r1[q] = ld4(tab + 4);
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < OWN; ++q) {
    const int i = s + q * S, m = i * 16 + (lane & 15);
    if (i >= MT) break;
    f32x4_t v[S][2];
#pragma unroll
    for (int p = 0; p < S; ++p) {
      v[p][0] = red[p][i][0][lane];
      v[p][1] = red[p][i][1][lane];
    }
    f32x4_t a0 = v[0][0], a1 = v[0][1];
#pragma unroll
    for (int p = 1; p < S; ++p) {
      a0 += v[p][0];
      a1 += v[p][1];
    }
    if ((EPI == EPI_QKV || EPI == EPI_GELU) && o.bias) {
      a0 += b0;
      a1 += b1;
    }
    if (m >= M) continue;
    if constexpr (EPI == EPI_PART) {
      store_sums(o.part + (size_t)m * o.ldc, n0, o.ldc, a0);
      store_sums(o.part + (size_t)m * o.ldc, n1, o.ldc, a1);
    } else if constexpr (EPI == EPI_GATED) {
      stv4<DT>(o.act, xrow_index(m, blockIdx.x * 16 + c4, o.F, o.mtt), act_swiglu(a0, a1));
    } else if constexpr (EPI == EPI_GELU) {
      stv4<DT>(o.act, xrow_index(m, n0, o.F, o.mtt), act_gelu<DT>(a0));
      stv4<DT>(o.act, xrow_index(m, n1, o.F, o.mtt), act_gelu<DT>(a1));
    } else {
      const int H = o.H, t = n0 / H, which = o.third + t, c = n0 - t * H;      // both tiles lie in the same third and head
      if (o.rope && which < 2)
        rope_rotate(a0, a1, f32x4_t{r0[q][0], r0[q][2], r1[q][0], r1[q][2]}, f32x4_t{r0[q][1], r0[q][3], r1[q][1], r1[q][3]});
      const int hd = c / o.d, e = c - hd * o.d;
      void* dst = which == 0 ? o.q : which == 1 ? o.kc : o.vc;
      const size_t at = which == 0 ? (size_t)m * H + c : (((size_t)slot[q] * (H / o.d) + hd) * o.Smax + pos[q]) * o.d + e;
      stv4<DT>(dst, at, a0);
      stv4<DT>(dst, at + (n1 - n0), a1);
    }
  }
}

// The rows' operand of a block as 1 KiB fragments: row tile mt0 + f of k-block kb0 + t is at base + t * step + offset(f).
// Row-major (xmtt == 0) or fragment order with xmtt row tiles per k-block; rows and row tiles past the last repeat it.
struct RowTiles {
  const char* base;
  size_t step;
  uint32_t row_bytes;
  int left, xmtt;                                // row-major: rows from mt0 on; fragment order: row tiles from mt0 on
  __device__ RowTiles(const uint16_t* x, int M, int K, int mt0, int kb0, int xmtt_) : xmtt(xmtt_) {
    row_bytes = (uint32_t)K * 2;
    if (xmtt) {
      base = (const char*)x + ((size_t)kb0 * xmtt + mt0) * 1024;
      step = (size_t)xmtt * 1024;
      left = xmtt - mt0;
    } else {
      base = (const char*)x + ((size_t)mt0 * 16 * K + kb0 * 32) * 2;
      step = 64;
      left = M - mt0 * 16;
    }
  }
  __device__ uint32_t offset(int f, int lane) const {
    return xmtt ? min(f, left - 1) * 1024 + lane * 16 : min(f * 16 + (lane & 15), left - 1) * row_bytes + (lane >> 4) * 16;
  }
};

// ---- context passes (hundreds of rows): the contraction is MFMA-bound there, so each wave keeps a 128 x 64 output
// tile (8 row tiles x 4 n-tiles, 128 accumulator registers): per k-block 32 MFMAs for 8 KiB of LDS reads and 4 KiB of W
// loads.  A block is 4 column units of 64 columns x 2 row halves = 8 waves over 256 rows x 256 columns.  The weights go
// straight to registers (each wave its own four fragments, PF k-blocks ahead), the rows' operand goes to LDS by
// asynchronous copies (16 fragments per k-block, L k-blocks ahead, a ring of L + 1 slots): with both operands through LDS
// its 128 bytes per cycle would be the bound.  One barrier per k-block, placed in the middle of the multiplications: the
// fragments of the next k-block are then read while this one's last row tiles are multiplied, so the matrix units see
// neither the barrier nor the LDS latency.  0.71 us per k-block (0.75 with the x tile staged through registers and a
// barrier per two k-blocks): 1024 rows x 12288 x 4096 102 -> 96 us, 288 rows x 22016 x 4096 100 -> 89 us; over the 192
// blocks of the former that is the rate per compute unit of an 8192-cubed library product on the whole chip.
// The per-(m, n) arithmetic is again the same MFMA sequence over k.
// EPI: what becomes of the accumulators (see tile_epilogue); all but partial sums need the whole of K in one slice.
template <int DT, int NTL, int EPI>
__global__ __launch_bounds__(512) void gemm16_rows_kernel(const uint16_t* __restrict__ x, const u32x4_t* __restrict__ wt,
                                                          TileOut o, int M, int N, int K, int ngroups, int KB, int kbs, int nx,
                                                          int nslices, int nz, int xmtt) {
  static_assert(NTL == 2 || NTL == 4, "layout groups");
  constexpr int A = 8, B = 4, PF = 4, L = 4, D = L + 1, MTB = 2 * A, F = MTB / 8;   // F: copies per wave and k-block
  __shared__ u32x4_t lds[D][MTB * 64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // 1-D grid, XCD-aware: row blocks of one (column block, K slice) task share an XCD (see gemm16_lds_kernel)
  const int xcd = blockIdx.x & 7, qq = blockIdx.x >> 3;
  const int zb = qq % nz, task = (qq / nz) * 8 + xcd;
  if (task >= nx * nslices) return;
  const int bx = task % nx, s = task / nx;
  const int g = bx * 4 + (wave >> 1), half = wave & 1;
  const int gl = min(g, ngroups - 1);
  const int kb0 = s * kbs, T = min(KB, kb0 + kbs) - kb0;
  const int mt0 = zb * MTB;
  const int live = min(A, max(0, (M + 15) / 16 - mt0 - half * A));     // of this wave's row tiles

  // the wave's four n-tiles are 4 / NTL consecutive column groups of the matrix layout (NTL tiles per group), or the rotary
  // partners' tiles of a head: those sit four n-tiles apart (d = 128)
  const bool split = EPI == EPI_QKV && o.d == 128;     // three times a multiple of four heads: whole blocks of 256 columns
  const int u0 = split ? bx * 16 + tile_of<B, 4, EPI>(wave >> 1, 0, 128) : gl * B;         // first n-tile
  const u32x4_t* wp = wt + (((size_t)(u0 / NTL) * KB + kb0) * NTL + u0 % NTL) * 64 + lane;   // + kb * NTL * 64
  const size_t far = split ? (size_t)(4 / NTL) * KB * NTL * 64 : NTL == 2 ? (size_t)KB * NTL * 64 : 128;   // n-tiles 2 and 3
  RowTiles rows(x, M, K, mt0, kb0, xmtt);
  uint32_t src[F];
#pragma unroll
  for (int j = 0; j < F; ++j) src[j] = rows.offset(wave + 8 * j, lane);
  // Copies and W loads past the slice repeat its last k-block (in bounds, unused): every k-block then issues the same
  // number of loads and the wait counts are constants.
  auto copy_rows = [&](int t, int slot) {
    const char* base = rows.base + (size_t)min(t, T - 1) * rows.step;
#pragma unroll
    for (int j = 0; j < F; ++j) copy_to_lds(base, src[j], lds[slot] + (wave + 8 * j) * 64);
  };
  u32x4_t bq[PF][B], af[4];
  auto load_w = [&](auto j_, int t) {
    constexpr int j = decltype(j_)::value;
    const u32x4_t* w = wp + (size_t)min(t, T - 1) * NTL * 64;
#pragma unroll
    for (int u = 0; u < B; ++u) bq[j][u] = w[(u & 1) * 64 + (u >> 1) * far];
  };
  f32x4_t acc[A][B];
#pragma unroll
  for (int i = 0; i < A; ++i)
#pragma unroll
    for (int u = 0; u < B; ++u) acc[i][u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // issue order as in the loop: copies, then W, k-block by k-block
  auto ahead = [&](auto j_) {
    copy_rows(decltype(j_)::value, decltype(j_)::value);
    __builtin_amdgcn_sched_barrier(0);
    load_w(j_, decltype(j_)::value);
    __builtin_amdgcn_sched_barrier(0);
  };
  ahead(std::integral_constant<int, 0>{});
  ahead(std::integral_constant<int, 1>{});
  ahead(std::integral_constant<int, 2>{});
  ahead(std::integral_constant<int, 3>{});
  static_assert(L == 4 && PF == 4, "prologue");
  copies_barrier<(F + B) * L - F>(false);        // the copies of k-block 0 have landed
  int slot = 0;                                  // of the k-block being multiplied
  // One k-block.  ROWS8 = all eight row tiles live (no branches); otherwise dead row tiles are skipped (wave-uniform).
  auto kblock = [&](auto j_, auto rows8_, auto last_, int t) {
    constexpr int j = decltype(j_)::value;
    constexpr bool rows8 = decltype(rows8_)::value;
    const int nslot = slot + 1 == D ? 0 : slot + 1, cslot = slot == 0 ? D - 1 : slot - 1;
    const u32x4_t *lw = lds[slot] + half * A * 64 + lane, *ln = lds[nslot] + half * A * 64 + lane;
#pragma unroll
    for (int i = 0; i < A; ++i) {
      if (i == A / 2) {
        // the copies of k-block t + 1 have landed; every wave has read k-block t - 1, whose slot is refilled.  In the last turn the W
        // loads feed nothing and are not made, so fewer loads follow those copies than the count says: wait for all.
        copies_barrier<(F + B) * (L - 1) - F>(decltype(last_)::value);
        copy_rows(t + L, cslot);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (rows8) {                               // the last two reads are the next k-block's first fragments
        af[(i + 2) % 4] = i + 2 < A ? lw[(i + 2) * 64] : ln[(i + 2 - A) * 64];
      } else if (i < live) {
        af[i % 4] = lw[i * 64];
      }
      if (rows8 || i < live) {
#pragma unroll
        for (int u = 0; u < B; ++u) acc[i][u] = mfma16<DT>(bq[j][u], af[i % 4], acc[i][u]);
        if (rows8) __builtin_amdgcn_sched_barrier(0);   // keeps every fragment's read two row tiles ahead of its use
      }
    }
    load_w(j_, t + PF);
    __builtin_amdgcn_sched_barrier(0);
    slot = nslot;
  };
  auto loop = [&](auto rows8_) {
    if (decltype(rows8_)::value) {
      af[0] = (lds[0] + half * A * 64 + lane)[0];
      af[1] = (lds[0] + half * A * 64 + lane)[64];
    }
    int t = 0;
    for (; t + PF <= T; t += PF) {
      kblock(std::integral_constant<int, 0>{}, rows8_, std::false_type{}, t);
      kblock(std::integral_constant<int, 1>{}, rows8_, std::false_type{}, t + 1);
      kblock(std::integral_constant<int, 2>{}, rows8_, std::false_type{}, t + 2);
      kblock(std::integral_constant<int, 3>{}, rows8_, std::false_type{}, t + 3);
    }
    if (t < T) kblock(std::integral_constant<int, 0>{}, rows8_, std::true_type{}, t);
    if (t + 1 < T) kblock(std::integral_constant<int, 1>{}, rows8_, std::true_type{}, t + 1);
    if (t + 2 < T) kblock(std::integral_constant<int, 2>{}, rows8_, std::true_type{}, t + 2);
  };
  // Two copies of the loop, chosen per wave (both pass the same barriers).
  if (live == A) loop(std::true_type{});
  else loop(std::false_type{});
  copies_barrier<0>(true);                       // no copy may still be under way when the block's LDS is given away
  if (g >= ngroups) return;
  tile_epilogue<DT, A, B, 2, 4, EPI>(acc, o, M, N, mt0 + half * A, bx * 16, wave >> 1, s, lane);
}

// ---- context passes: both operands through LDS by asynchronous copies (memory to LDS without registers).  Both operands
// already are sequences of 1 KiB MFMA fragments (the weights always, the rows unless they are row-major, where every lane
// simply points at its own 16 bytes), so one copy instruction of a wave lands one fragment and the reads back are
// conflict-free ds_read_b128.  A block is WR x WC waves, a wave owns A row tiles x B n-tiles; a stage is one k-block, D
// stages form a ring in LDS; the fragments of stage t + 1 are read while stage t is multiplied, one barrier per stage.
// What bounds it: the operand bytes through the L2s (about 24 TB/s over the chip; less while the weights come from HBM) at
// the small blocks, the 128 bytes per cycle of LDS at the large ones.  Its place is between 129 and a few hundred rows and
// at narrow matrices, where 256 x 256 blocks with up to 16 K slices left most compute units waiting (288 rows, cold
// weights, the slices' sums not counted): 6144 x 2048 28.7 -> 16.7 us, 2048 x 2048 20.5 -> 11.2, 8192 x 2048 28.0 -> 23,
// 512 x 512 12.7 -> 5.2 us.
template <int DT, int A, int B, int WR, int WC, int D, int EPI>
__global__ __launch_bounds__(64 * WR * WC) __attribute__((amdgpu_waves_per_eu(2))) void gemm16_tile_kernel(const uint16_t* __restrict__ x, const char* __restrict__ wt, TileOut o,
                                                                   int M, int N, int K, int ntiles, int NTL, int KB, int kbs,
                                                                   int ncb, int nrb, int tasks, int per, int xmtt) {
  constexpr int FA = A * WR, FB = B * WC, NW = WR * WC, F = (FA + FB) / NW;   // F: copies per wave and stage
  static_assert((FA + FB) % NW == 0 && D >= 2, "every wave copies the same number of fragments per stage");
  static_assert(F * (D - 1) < 64, "the wait count has six bits");
  __shared__ u32x4_t lds[D][(FA + FB) * 64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wr = wave / WC, wc = wave % WC;
  // workgroup ids go round-robin over the 8 XCDs: each XCD gets a contiguous run of tasks (row block fastest), so the row
  // blocks of a column block share its weight tiles in that XCD's L2
  const int task = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || task >= tasks) return;
  const int rb = task % nrb, cs = task / nrb, cb = cs % ncb, s = cs / ncb;
  const int kb0 = s * kbs, T = min(KB, kb0 + kbs) - kb0;
  const int mt0 = rb * FA, nt0 = cb * FB;        // first row tile / n-tile of the block

  static_assert(FA % NW == 0, "a copy instruction takes fragments of one operand");
  constexpr int FX = FA / NW;                    // of a wave's F copies per stage, the first FX are of the rows' operand
  RowTiles rows(x, M, K, mt0, kb0, xmtt);
  const int g0 = nt0 / NTL;
  const char* wbase = wt + ((size_t)g0 * KB + kb0) * NTL * 1024;
  uint32_t src[F];
#pragma unroll
  for (int j = 0; j < F; ++j) {
    const int f = wave + NW * j;
    if (j < FX) {
      src[j] = rows.offset(f, lane);
    } else {
      const int nt = min(nt0 + f - FA, ntiles - 1), g = nt / NTL;
      src[j] = ((uint32_t)(g - g0) * KB * NTL + (nt - g * NTL)) * 1024 + lane * 16;
    }
  }
  auto issue = [&](int slot) {                   // copies of the next stage
#pragma unroll
    for (int j = 0; j < F; ++j) copy_to_lds(j < FX ? rows.base : wbase, src[j], lds[slot] + (wave + NW * j) * 64);
    rows.base += rows.step;
    wbase += NTL * 1024;
  };
  u32x4_t fa[2][A], fb[2][B];
  auto fetch = [&](auto r_, int slot) {
    constexpr int r = decltype(r_)::value;
    const u32x4_t* l = lds[slot] + lane;
#pragma unroll
    for (int u = 0; u < B; ++u) fb[r][u] = l[(FA + tile_of<B, WC, EPI>(wc, u, o.d)) * 64];
#pragma unroll
    for (int i = 0; i < A; ++i) fa[r][i] = l[(wr * A + i) * 64];
  };
  f32x4_t acc[A][B];
#pragma unroll
  for (int i = 0; i < A; ++i)
#pragma unroll
    for (int t = 0; t < B; ++t) acc[i][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](auto r_) {
    constexpr int r = decltype(r_)::value;
#pragma unroll
    for (int i = 0; i < A; ++i)
#pragma unroll
      for (int u = 0; u < B; ++u) acc[i][u] = mfma16<DT>(fb[r][u], fa[r][i], acc[i][u]);
  };
  const std::integral_constant<int, 0> r0{};
  const std::integral_constant<int, 1> r1{};
#pragma unroll
  for (int t = 0; t < D; ++t)
    if (t < T) issue(t);
  copies_barrier<F * (D - 1)>(T < D);
  fetch(r0, 0);
  int t = 0, slot = 0;                           // slot = t % D
  // One step: stage t sits in registers `cur`; its slot in LDS is free once every wave is past the barrier, so the copies
  // of stage t + D go there, and the fragments of stage t + 1 are read while stage t is multiplied.  The last step reads
  // a slot whose contents nobody uses.
  auto step1 = [&](auto cur, auto nxt) {
    const bool more = t + D < T;
    copies_barrier<F * (D - 2)>(!more);
    if (more) issue(slot);
    slot = slot + 1 == D ? 0 : slot + 1;
    fetch(nxt, slot);
    __builtin_amdgcn_sched_barrier(0);
    multiply(cur);
    __builtin_amdgcn_sched_barrier(0);
    return ++t == T;
  };
  for (;;) {
    if (step1(r0, r1)) break;
    if (step1(r1, r0)) break;
  }
  tile_epilogue<DT, A, B, WR, WC, EPI>(acc, o, M, N, mt0 + wr * A, nt0, wc, s, lane);
}

// ---- context passes, the blocks of up to 128 x 256: K in WK parts inside the block.  A block is WC x WK = 8 waves; a wave owns A
// row tiles x B n-tiles over one part of the slice's k-blocks, so that the weights go straight to registers without any two
// waves loading the same ones (PF k-blocks ahead), and only the rows' operand, which the WC waves of a part share, goes through
// LDS (asynchronous copies, L k-blocks ahead).  A step is one k-block of every part.  With both operands through LDS its 128 bytes per
// cycle are the bound (64 x 128 blocks 0.165 us per k-block, here 0.11; 64 x 64 0.128 and 0.066; 128 x 256 0.40 and 0.36), which
// leaves the 110 bytes per nanosecond that reach a compute unit; the hand-over at the end costs 1 to 2 us.
template <int DT, int A, int B, int WC, int WK, int PF, int L, int EPI>
__global__ __launch_bounds__(64 * WC * WK) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm16_parts_kernel(
    const uint16_t* __restrict__ x, const u32x4_t* __restrict__ wt, TileOut o, int M, int N, int K, int ntiles, int NTL, int KB, int kbs,
    int ncb, int nrb, int tasks, int per, int xmtt) {
  constexpr int NW = WC * WK, F = A * WK / NW, D = L + 1;      // F: copies per wave and step
  constexpr int OWN = A / WK;                                  // row tiles a wave finishes
  static_assert(NW == 8 && A * WK % NW == 0 && A % WK == 0 && B % 2 == 0, "fragments divide among the waves");
  static_assert(PF >= L - 1 && (F + B) * (L - 1) - F < 64, "wait counts");
  constexpr int RT = OWN > 1 && (WK - 1) * B * NW * OWN > 96 ? OWN / 2 : OWN;   // row tiles per round of the hand-over
  constexpr int XF = D * WK * A, RF = (WK - 1) * B * NW * RT;
  __shared__ u32x4_t lds[(XF > RF ? XF : RF) * 64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wk = wave / WC, wc = wave % WC;
  const int task = (blockIdx.x & 7) * per + (blockIdx.x >> 3);  // see gemm16_tile_kernel
  if ((int)(blockIdx.x >> 3) >= per || task >= tasks) return;
  const int rb = task % nrb, cs = task / nrb, cb = cs % ncb, s = cs / ncb;
  const int kb0 = s * kbs, T = min(KB, kb0 + kbs) - kb0;
  const int mt0 = rb * A, nt0 = cb * B * WC;
  // part p: k-blocks first(p) .. first(p + 1) - 1 of the slice; every part has one at least (the host sees to it)
  auto first = [&](int p) { return p * (T / WK) + min(p, T % WK); };
  const int steps = (T + WK - 1) / WK, k0 = kb0 + first(wk), Tp = first(wk + 1) - first(wk);

  const RowTiles rows(x, M, K, mt0, 0, xmtt);
  uint32_t src[F];
  const char* from[F];
  int left[F];                                   // k-blocks of the part that are still to be copied behind the next one
#pragma unroll
  for (int j = 0; j < F; ++j) {
    const int f = wave + NW * j, p = f / A;
    src[j] = rows.offset(f % A, lane);
    from[j] = rows.base + (size_t)(kb0 + first(p)) * rows.step;
    left[j] = first(p + 1) - first(p) - 1;
  }
  // Copies and W loads past a part repeat its last k-block (in bounds, unused): every step issues the same number of loads and
  // the wait counts are constants.
  auto copy_rows = [&](int slot) {
#pragma unroll
    for (int j = 0; j < F; ++j) {
      copy_to_lds(from[j], src[j], lds + (slot * WK * A + wave + NW * j) * 64);
      from[j] += left[j] > 0 ? rows.step : 0;
      left[j] -= 1;
    }
  };
  const u32x4_t* wp[B / 2];                      // pairs of n-tiles lie side by side
#pragma unroll
  for (int u = 0; u < B; u += 2) {
    const int nt = min(nt0 + tile_of<B, WC, EPI>(wc, u, o.d), ntiles - 2);
    wp[u / 2] = wt + (((size_t)(nt / NTL) * KB + k0) * NTL + nt % NTL) * 64 + lane;
  }
  u32x4_t bq[PF][B], af[4];
  auto load_w = [&](auto j_, int t) {
    constexpr int j = decltype(j_)::value;
    const uint32_t at = (uint32_t)min(t, Tp - 1) * NTL * 64;
#pragma unroll
    for (int u = 0; u < B; ++u) bq[j][u] = wp[u / 2][at + (u & 1) * 64];
  };
  f32x4_t acc[A][B];
#pragma unroll
  for (int i = 0; i < A; ++i)
#pragma unroll
    for (int u = 0; u < B; ++u) acc[i][u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < L; ++t) copy_rows(t);
  __builtin_amdgcn_sched_barrier(0);
  auto prologue = [&](auto self, auto j_) -> void {
    constexpr int j = decltype(j_)::value;
    load_w(j_, j);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (j + 1 < PF) self(self, std::integral_constant<int, j + 1>{});
  };
  prologue(prologue, std::integral_constant<int, 0>{});
  copies_barrier<(L - 1) * F + PF * B>(false);   // the copies of step 0 have landed
  int slot = 0;
  af[0] = lds[(wk * A) * 64 + lane];
  af[1] = lds[(wk * A + 1) * 64 + lane];
  auto step = [&](auto j_, auto all_, int t) {
    constexpr int j = decltype(j_)::value;
    constexpr bool all = decltype(all_)::value;  // every part has a k-block left
    const int nslot = slot + 1 == D ? 0 : slot + 1, cslot = slot == 0 ? D - 1 : slot - 1;
    const u32x4_t *lw = lds + (slot * WK + wk) * A * 64 + lane, *ln = lds + (nslot * WK + wk) * A * 64 + lane;
#pragma unroll
    for (int i = 0; i < A; ++i) {
      if (i == A / 2) {
        // the copies of step t + 1 have landed; every wave has read step t - 1, whose slot is refilled; in the last turn wait for all
        // (see gemm16_rows_kernel)
        copies_barrier<(F + B) * (L - 1) - F>(!all);
        copy_rows(cslot);
        __builtin_amdgcn_sched_barrier(0);
      }
      af[(i + 2) % 4] = i + 2 < A ? lw[(i + 2) * 64] : ln[(i + 2 - A) * 64];
      if (all || t < Tp) {
#pragma unroll
        for (int u = 0; u < B; ++u) acc[i][u] = mfma16<DT>(bq[j][u], af[i % 4], acc[i][u]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    load_w(j_, t + PF);
    __builtin_amdgcn_sched_barrier(0);
    slot = nslot;
  };
  auto turn = [&](auto self, auto j_, auto all_, int t, int n) -> void {      // steps t .. of one turn of the W ring, n of them
    constexpr int j = decltype(j_)::value;
    if (decltype(all_)::value || j < n) {
      step(j_, all_, t + j);
      if constexpr (j + 1 < PF) self(self, std::integral_constant<int, j + 1>{}, all_, t, n);
    }
  };
  int t = 0;
  for (; t + PF < steps; t += PF) turn(turn, std::integral_constant<int, 0>{}, std::true_type{}, t, PF);
  turn(turn, std::integral_constant<int, 0>{}, std::false_type{}, t, steps - t);
  // The parts' sums: a wave finishes OWN of its row tiles and hands the others to the waves of the same columns, RT per owner and
  // round; added in the order of the parts.
  f32x4_t own[OWN][B];
  f32x4_t* red = (f32x4_t*)lds;
#pragma unroll
  for (int r = 0; r < OWN; r += RT) {
    if (r == 0) copies_barrier<0>(true);         // no copy may still be under way when its place is written
    else copies_barrier<0>(false);
#pragma unroll
    for (int p = 0; p < WK; ++p) {               // what part p finishes
      const int at = ((p * (WK - 1) + wk - (wk > p)) * WC + wc) * RT * B;
      if (p == wk) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
          for (int u = 0; u < B; ++u) own[r + i][u] = acc[p * OWN + r + i][u];
      } else {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
          for (int u = 0; u < B; ++u) red[(at + i * B + u) * 64 + lane] = acc[p * OWN + r + i][u];
      }
    }
    copies_barrier<0>(false);
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int u = 0; u < B; ++u) {
        f32x4_t v[WK];
#pragma unroll
        for (int p = 0; p < WK; ++p)             // the slot of part wk itself: any, replaced
          v[p] = red[(((wk * (WK - 1) + min(p - (p > wk), WK - 2)) * WC + wc) * RT * B + i * B + u) * 64 + lane];
        f32x4_t sum = wk == 0 ? own[r + i][u] : v[0];
#pragma unroll
        for (int p = 1; p < WK; ++p) sum += p == wk ? own[r + i][u] : v[p];
        own[r + i][u] = sum;
      }
  }
  tile_epilogue<DT, OWN, B, 1, WC, EPI>(own, o, M, N, mt0 + wk * OWN, nt0, wc, s, lane);
}

// ---------------------------------------------------------------- fp32 FMA kernel (tiny models)

// Lane l ends with the sum over the wave of v[l >> 2]: halves of the values are exchanged at distances 32, 16, 8 and 4 (15
// exchanges instead of 6 for each of the 16 values; all within the vector unit), then the last four lanes are added.
// Fixed order.
__device__ __forceinline__ float wave_sums16(float (&v)[16], int lane) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {                  // lower half of the wave: both halves of v[i], upper half: of v[i + 8]
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 8]), false, false);
    v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 4]), false, false);
    v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  const bool up8 = lane & 8, up4 = lane & 4;
#pragma unroll
  for (int i = 0; i < 2; ++i) v[i] = (up8 ? v[i + 2] : v[i]) + dpp_f<0x128>(up8 ? v[i] : v[i + 2]);      // row_ror:8
  float r = (up4 ? v[1] : v[0]) + dpp_f<0x141>(up4 ? v[0] : v[1]);     // row_half_mirror: the other four lanes, in reverse
  return sum_partner<2>(sum_partner<1>(r));
}

// A wave takes two output columns and 8 rows: lanes stride K four elements at a time, so that a row of up to 256 elements is
// one round of loads (3.1 us per launch at 7 rows x 256 x 256, 4.8 at 256 x 1024; one column and four bytes per lane and
// load: 5.2 on average, up to 10.5; the time is the launch and the round trips).  The second column is the next one, or the one that
// the epilogue needs beside it: the rotary partner, or up beside gate.  Every model of this type finishes in the epilogue
// (see tile_epilogue): tiny models are bound by their count of launches.
// NORM (1: layer norm, 2: RMS; K <= 256 U): x is the residual stream and every wave takes the norm of its rows while its weights are
// under way, in the order of norm_row, so that the bits are those of the norm in a launch of its own.
template <int EPI, int U, int NORM>
__global__ __launch_bounds__(256) void gemm32_kernel(const float* __restrict__ x, const float* __restrict__ W, TileOut o, int M, int N,
                                                     int K) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int pair = blockIdx.x * 4 + wave, half = o.d >> 1;
  const int c0 = EPI == EPI_QKV ? pair / half * o.d + pair % half : EPI == EPI_GATED ? pair : 2 * pair;
  const int c1 = EPI == EPI_QKV ? c0 + half : EPI == EPI_GATED ? pair + o.F : 2 * pair + 1;
  if (c0 >= (EPI == EPI_GATED ? o.F : N)) return;
  const int m0 = blockIdx.y * 8;
  // lanes 8r .. 8r+3 end with column c0 of row m0 + r, the next four with c1; what the epilogue reads goes out first
  const int m = m0 + (lane >> 3), mr = min(m, M - 1), c = min((lane & 4) ? c1 : c0, N - 1);
  float bias = 0.f, old = 0.f;
  int pos = 0, slot = 0;
  if (EPI != EPI_PART && EPI != EPI_GATED && o.bias) bias = ((const float*)o.bias)[c];
  if constexpr (EPI == EPI_ADD) old = o.part[(size_t)mr * o.ldc + c];
  if constexpr (EPI == EPI_QKV) {
    pos = o.pos[mr];
    slot = o.slot[mr];
  }
  float acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  const float *w0 = W + (size_t)c0 * K, *w1 = W + (size_t)min(c1, N - 1) * K;
  for (int k0 = lane * 4; NORM || k0 < K; k0 += U * 256) {     // U rounds of loads in flight; those past K count as zero
    f32x4_t a[U], b[U], v[U][8];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = min(k0 + u * 256, K - 4);
      a[u] = *(const f32x4_any*)(w0 + k);
      b[u] = *(const f32x4_any*)(w1 + k);
#pragma unroll
      for (int r = 0; r < 8; ++r) v[u][r] = *(const f32x4_any*)(x + (size_t)min(m0 + r, M - 1) * K + k);
    }
    f32x4_t g[U], bt[U];
    if constexpr (NORM != 0) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = min(k0 + u * 256, K - 4);
        g[u] = ld4((const float*)o.norm.g + k);
        if (NORM == 1) bt[u] = ld4((const float*)o.norm.b + k);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (NORM != 0) {
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        auto row_sum = [&](auto of) {
          float t = 0.f;
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const float w = group_sum<64>(k0 + u * 256 < K ? of(v[u][r]) : 0.f);
            t = u == 0 ? w : t + w;
          }
          return t;
        };
        float mean = 0.f, total;
        if constexpr (NORM == 2) {
          total = row_sum([](const f32x4_t& t) { return square_sum4(t); });
        } else {
          mean = row_sum([](const f32x4_t& t) { return sum4(t); }) / (float)K;
          total = row_sum([&](const f32x4_t& t) { return square_sum4(t - mean); });
        }
        const float inv = 1.0f / sqrtf(total / (float)K + o.norm.eps);
#pragma unroll
        for (int u = 0; u < U; ++u) v[u][r] = norm_value<NORM == 2>(v[u][r], mean, inv, g[u], NORM == 1 ? bt[u] : g[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k0 + u * 256 >= K) continue;
#pragma unroll
      for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[2 * r] = fmaf(v[u][r][e], a[u][e], acc[2 * r]);
          acc[2 * r + 1] = fmaf(v[u][r][e], b[u][e], acc[2 * r + 1]);
        }
    }
    if (NORM) break;                             // one round holds the row
  }
  const float sum = wave_sums16(acc, lane) + (EPI == EPI_PART || EPI == EPI_GATED ? 0.f : bias), other = __shfl_xor(sum, 4, 64);
  if (m >= M || (lane & 3)) return;
  if constexpr (EPI == EPI_QKV) {
    if (lane & 4) return;
    const int H = o.H, t = c0 / H, which = o.third + t, r = c0 - t * H, hd = r / o.d, e = r - hd * o.d;
    f32x4_t a0 = {sum, 0.f, 0.f, 0.f}, a1 = {other, 0.f, 0.f, 0.f};
    if (o.rope && which < 2) {
      const float* tab = o.rope + ((size_t)pos * half + e) * 2;
      rope_rotate(a0, a1, f32x4_t{tab[0], 0.f, 0.f, 0.f}, f32x4_t{tab[1], 0.f, 0.f, 0.f});
    }
    float* dst = (float*)(which == 0 ? o.q : which == 1 ? o.kc : o.vc);
    const size_t at = which == 0 ? (size_t)m * H + r : (((size_t)slot * (H / o.d) + hd) * o.Smax + pos) * o.d + e;
    dst[at] = a0[0];
    dst[at + half] = a1[0];
  } else if constexpr (EPI == EPI_GATED) {
    if (lane & 4) return;
    ((float*)o.act)[(size_t)m * o.F + c0] = act_swiglu(f32x4_t{sum, 0.f, 0.f, 0.f}, f32x4_t{other, 0.f, 0.f, 0.f})[0];
  } else {
    if (((lane & 4) ? c1 : c0) >= N) return;
    if constexpr (EPI == EPI_PART) o.part[(size_t)m * o.ldc + c] = sum;
    else if constexpr (EPI == EPI_ADD) o.part[(size_t)m * o.ldc + c] = old + sum;
    else ((float*)o.act)[(size_t)m * o.F + c] = act_gelu<DT_F32>(f32x4_t{sum, 0.f, 0.f, 0.f})[0];
  }
}

// ---------------------------------------------------------------- host side

GemmPlan gemm_plan(int dtype, int N, int K) {
  GemmPlan p{};
  p.N = N;
  p.K = K;
  p.ldc = part_ld(N);
  if (dtype == DT_F32) {
    p.Npad = N;
    p.NT = 0;
    p.KB = 0;
    p.S = 1;
    p.kbs = 0;
    return p;
  }
  p.Npad = (N + 63) / 64 * 64;
  p.KB = K / 32;
  // Everything below is a function of (N, K) only, never of the number of live rows.  Column groups of 32 (NT = 2) or 64
  // columns and S slices of K are chosen together, for the least time of a launch and of the kernel that reads the slices
  // back, averaged over row counts of 6 to 100 (mean 47): a block of four groups walks its k-blocks at one latency each
  // and all blocks share the memory rate, so more slices shorten the walk, cost their sums once to write and once to
  // read, and must not start a second round on the 256 compute units; slices that begin at the same power of two meet in
  // the same memory channels.  Fitted to 900 launches (16 shapes from 512 x 512 to 50257 x 2048 and 6656 x 17920, cold
  // weights, both widths, 1 to 16 slices; 11-13 % rms).  Against a fixed count of 800 wavefronts and 64-column groups above
  // 4096 columns, sums counted, at 6 / 23 / 60 / 100 rows: 6144 x 2048 (8 slices -> 3, 32 columns) 8.1 / 9.6 / 14.2 / 18.7 ->
  // 6.7 / 8.3 / 10.4 / 13.6 us, 12288 x 4096 (4 -> 2, 32 columns) 18.7 / 20.3 / 25.1 / 30.0 -> 17.9 / 18.8 / 22.1 / 27.5.
  double best = 0.0;
  for (int NT = 2; NT <= 4; NT += 2) {
    const int per_slice = (p.Npad / (16 * NT) + 3) / 4;
    for (int S = 1; S <= 16; ++S) {
      const int kbs = (p.KB + S - 1) / S;
      if (S > 1 && (kbs < 4 || (p.KB + kbs - 1) / kbs != S || per_slice * S > 256)) continue;
      const double walk = (NT == 2 ? 0.195 : 0.338) * kbs * ((per_slice * S + 255) / 256);
      const double stream = (NT == 2 ? 0.111 : 0.153) * p.Npad * K * 2e-6 * (S > 1 && kbs % 16 == 0 ? 1.1 : 1.0);
      const double cost = (NT == 2 ? 2.6 + std::sqrt(walk * walk + stream * stream) : 3.35 + std::max(walk, stream)) +
                          (0.4 + 0.25) * S * 47 * p.ldc * 4e-6;
      if (p.S == 0 || cost < best) {
        best = cost;
        p.NT = NT;
        p.S = S;
        p.kbs = kbs;
      }
    }
  }
  return p;
}

// A block per 32 columns with all of K in it (gemm16_whole_kernel) is the shorter way while all blocks run at once and a block's
// bytes (its columns and all rows, over K) stay few: every block reads all rows, at the 110 bytes per nanosecond that a compute
// unit gets.  Measured with the launch that it saves, us at 6 / 23 / 64 / 101 rows, two launches -> one: q|k|v of 2048 columns (192
// blocks) 9.3 / 10.8 / 13.5 / 17.2 -> 7.2 / 8.5 / 10.5 / 14.0, of 2560 (240) 11.1 / 13.0 / 16.2 / 20.9 -> 8.9 / 10.5 / 12.8 / 17.6, of
// 3072 (288) 14.1 / 15.2 / 18.6 / 23.3 -> 16.0 / 18.6 / 23.8 / 32.6; 8192 x 2048 with GELU (256) 10.7 / 12.1 / 15.3 / 19.4 -> 8.5 / 9.6 /
// 11.0 / 15.1, 10240 x 2560 (320) 13.0 / 14.9 / 19.1 / 23.6 -> 14.4 / 17.0 / 20.9 / 28.7, 4096 x 4096 (128 blocks, long K) 10.2 / 12.2 /
// 15.2 / 19.5 -> 10.9 / 12.9 / 16.5 / 22.6.  Four slices: with two, 48 rows and more are 10 to 40 % slower.
static bool whole_shape(int dtype, int N, int K) { return dtype != DT_F32 && (N + 31) / 32 <= 256 && K >= 512; }
static constexpr int kWholeSlices = 4;
static void take_whole(GemmPlan& p) {
  p.NT = 2;
  p.S = kWholeSlices;
  p.kbs = (p.KB + kWholeSlices - 1) / kWholeSlices;      // 16 k-blocks at least: the last slice is not empty
  p.whole = 1;
}
GemmPlan gemm_plan_finished(int dtype, int N, int K) {
  GemmPlan p = gemm_plan(dtype, N, K);
  if (whole_shape(dtype, N, K) && N % 32 == 0 && K <= 2560 && p.KB % kWholeSlices == 0) take_whole(p);
  return p;
}
// Only where the plan has these very slices, so that nothing changes where gemm_adds_up() is false.
GemmPlan gemm_plan_summed(int dtype, int N, int K) {
  GemmPlan p = gemm_plan(dtype, N, K);
  p.whole = whole_shape(dtype, N, K) && K <= 2560 && p.S == kWholeSlices && p.NT == 2;
  return p;
}

// gate|up of a gated MLP (N = 2F): paired 32-column groups, no K slices in memory (the fused kernels split K inside),
// when the shape allows it; otherwise the plain plan of a 2F-column matrix with gate and up side by side.
GemmPlan gemm_plan_gated(int dtype, int F, int K) {
  GemmPlan p = gemm_plan(dtype, 2 * F, K);
  if (dtype == DT_F32 || F % 32 != 0 || (K / 32) % 16 != 0) return p;
  p.NT = 2;
  p.S = 2;               // the two halves of K: partial sums of gemm(), the two in-kernel chains of the fused kernels
  p.kbs = p.KB / 2;
  p.paired = 1;
  // at any K, for the calls of few rows: the two kernels add up in another order and a row's bits do not depend on the row count, so one of them
  // serves all counts.  Calls with row-major rows, cold weights, gated_lds_kernel (blocks of two groups) -> this, us at 6 / 23 / 40 / 64 / 101 / 128
  // rows: 1376 x 512 5.2 / 6.2 / 6.9 / 7.8 / 10.0 / 10.7 -> 5.0 / 6.0 / 7.2 / 7.8 / 10.4 / 11.6, 2048 x 2560 10.7 / 13.9 / 15.6 / 17.4 / 21.4 / 23.5 -> 8.6 / 12.1 /
  // 16.8 / 19.9 / 27.3 / 32.0, 1024 x 6656 20.4 / 27.7 / 30.5 / 34.2 / 41.1 / 45.3 -> 14.3 / 21.7 / 30.2 / 39.2 / 54.9 / 64.8, 4096 x 4096 16.7 / 20.5 / 22.3 /
  // 24.8 / 29.3 / 31.6 -> 14.7 / 16.9 / 21.8 / 26.7 / 36.5 / 42.7: from about 40 rows on every block's own copy of all rows costs more than the idle units
  if (whole_shape(dtype, 2 * F, K)) take_whole(p);
  return p;
}

size_t gemm_tiled_bytes(int dtype, int N, int K) {
  if (dtype == DT_F32) return (size_t)N * K * 4;
  const size_t Npad = (size_t)(N + 63) / 64 * 64;
  return Npad * K * 2;
}

// Above 128 rows: estimated time (microseconds) of the contraction with one kernel and slice count, a latency-or-throughput
// model of the blocks that share a compute unit: a block's k-block step takes `step` alone and `busy` per block where
// several fill the unit; `start` is launch, ramp and drain, `store` the rate of the fp32 results (bytes per microsecond).
// Fitted to 3000 measured launches (16 matrix shapes from 512 x 512 to 35840 x 6656, 132 to 1024 rows, 1 to 8 slices,
// cold weights): 6-8 % rms per kernel, and the kernel and count it picks are on average 0.7 % slower than the best.
// That is the time of a launch that has the chip to itself; two pre-processing streams share it, and there the work per
// launch counts (blocks x steps over 256 compute units).  Weighed 7 : 3 in every mode: over 28 sets of 1 to 4 prompts of 130 to
// 1025 tokens at the 7B, GPT-1.3B and 30B shapes, 10 : 0 takes 0.997 of its time one after the other and 1.005 overlapped,
// 5 : 5 1.013 and 1.012.
struct TileKernel {
  int bm, bn, occ;      // rows and columns of a block, blocks a compute unit holds
  double start, step, busy, store;
  double w_start, w_step, w_store;   // see best_tile
};
static constexpr TileKernel kTile[] = {
    {256, 256, 1, 7.7, 0.628, 0.628, 4.3e6, 7.8, 0.79, 5.2e6},    // TILE_ROWS
    {128, 256, 1, 4.9, 0.411, 0.411, 4.0e6, 4.7, 0.53, 5.6e6},    // TILE_128X256
    {128, 128, 2, 3.7, 0.256, 0.238, 4.3e6, 3.8, 0.343, 5.6e6},   // TILE_128X128
    {64, 128, 3, 2.4, 0.205, 0.169, 4.9e6, 3.5, 0.22, 7.4e6},     // TILE_64X128
    {64, 64, 4, 2.15, 0.160, 0.107, 5.1e6, 3.4, 0.158, 8.7e6},    // TILE_64X64
};
static long tile_blocks(int tile, int M, const GemmPlan& p, int S) {
  const TileKernel& k = kTile[tile];
  const int ncols = tile == TILE_ROWS ? p.Npad : p.N;
  return (long)((M + k.bm - 1) / k.bm) * ((ncols + k.bn - 1) / k.bn) * S;
}
static double tile_cost(int tile, int M, const GemmPlan& p, int S, int kbs) {
  const TileKernel& k = kTile[tile];
  const long blocks = tile_blocks(tile, M, p, S), per_cu = (blocks + 255) / 256;
  const long full = per_cu / k.occ, rest = per_cu % k.occ;
  const double steps = full * std::max(k.step, k.busy * k.occ) + (rest ? std::max(k.step, k.busy * rest) : 0.0);
  return k.start + kbs * (0.7 * steps + 0.3 * k.busy * blocks / 256) + (double)S * M * p.N * 4.0 / k.store;
}

// Kernel and slice count of a context pass's GEMM: the pair with the least time, counting what the result costs the next
// kernel as well -- fp32 sums read back (4 TB/s) and a launch of its own, unless the kernel takes K in one slice and finishes the
// job in its epilogue.  Priced as if every one-slice kernel did (an unpaired gate|up matrix does not), and with the blocks in
// the table (q|k|v takes 128 columns where 64 are picked).  The table's figures are those of both operands through LDS; what
// parts_pay() launches in parts takes less than its price, so another block or more slices may be picked where it would be shorter.
GemmPlan context_plan(const GemmPlan& p, int dtype, int M, int max_slices) {
  GemmPlan q = p;
  if (dtype == DT_F32 || M <= 128) return q;
  const int smax = std::max(1, std::min(max_slices, 16));   // what the caller's partial-sum buffer holds; the row-wise
                                                             // kernels load up to 16 slices at once
  double best = 0.0;
  q.S = 0;
  for (int S = 1; S <= smax; ++S) {
    const int kbs = (p.KB + S - 1) / S;
    if ((p.KB + kbs - 1) / kbs != S) continue;                       // slice counts that leave an empty last slice
    for (int tile = TILE_ROWS; tile < TILE_KINDS; ++tile) {
      const bool finished = S == 1;
      const double cost = tile_cost(tile, M, p, S, kbs) + (finished ? 0.0 : (double)S * M * p.N * 4.0 / 4.0e6 + 1.5);
      if (q.S == 0 || cost < best) {
        best = cost;
        q.S = S;
        q.kbs = kbs;
        q.tile = tile;
      }
    }
  }
  return q;
}
// The slicing is given (a fused iteration of more than 128 rows, whose slices depend on the matrix alone): only the kernel, and
// the results do not depend on it.  Every k-block costs w_step per round of blocks on the 256 compute units: fitted to 1365
// launches of its own (21 matrix shapes from 1000 x 512 to 32000 x 6656 at the plan's slices, 129 to 1024 rows, cold weights;
// 6-7 % rms), for the model above, which weighs rounds and throughput for passes that share the chip, picked kernels 3.3 % off
// the best on average and up to 21 %, this one 0.9 % and 15 % (12288 x 4096 at 768 rows 131 -> 115 us, 6144 x 2048 at 384 rows
// 25.0 -> 20.6).
static int best_tile(int M, const GemmPlan& p) {
  auto cost = [&](int tile) {
    const TileKernel& k = kTile[tile];
    return k.w_start + p.kbs * k.w_step * ((tile_blocks(tile, M, p, p.S) + 255) / 256) + (double)p.S * M * p.N * 4.0 / k.w_store;
  };
  int at = TILE_ROWS;
  for (int tile = TILE_ROWS + 1; tile < TILE_KINDS; ++tile)
    if (cost(tile) < cost(at)) at = tile;
  return at;
}
void gemm_block(int M, const GemmPlan& p, int* rows, int* columns) {
  const TileKernel& k = kTile[p.tile < 0 ? best_tile(M, p) : p.tile];
  *rows = k.bm;
  *columns = k.bn;
}

hipError_t retile(int dtype, const void* W, int N, int K, void* tiled, int n_off, int NT, hipStream_t st, int tile_step) {
  if (dtype == DT_F32) {
    if (tile_step != 1) return hipErrorInvalidValue;
    return hipMemcpyAsync((char*)tiled + (size_t)n_off * K * 4, W, (size_t)N * K * 4, hipMemcpyDeviceToDevice, st);
  }
  const int KB = K / 32;
  const int ntiles = (N + 15) / 16;
  const long total = (long)ntiles * KB * 64;
  retile16_kernel<<<dim3((unsigned)((total + 255) / 256)), 256, 0, st>>>((const uint16_t*)W, (u32x4_t*)tiled, N, K, KB,
                                                                         n_off / 16, tile_step, NT, total);
  return hipGetLastError();
}

hipError_t zero_fill(void* p, size_t bytes, hipStream_t st) { return hipMemsetAsync(p, 0, bytes, st); }

template <int DT, int MT, int NT, int PFW, int PFA>
static void launch_direct(const void* x, const void* wt, float* part, int M, const GemmPlan& p, size_t ss, int xmtt,
                          hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  const int ngroups = p.Npad / (16 * NT);
  dim3 grid((ngroups + 3) / 4, p.S, (M + 16 * MT - 1) / (16 * MT));
  launch_timed(gemm16_direct_kernel<DT, MT, NT, PFW, PFA>, grid, dim3(256), st, ev0, ev1, (const uint16_t*)x,
               (const u32x4_t*)wt, part, M, p.N, p.K, ngroups, p.KB, p.kbs, ss, p.ldc, xmtt);
}
template <int DT, int MT, int NT, int NTW, int PF, int GPB = 4, int KC = 2>
static void launch_lds(const void* x, const void* wt, float* part, int M, const GemmPlan& p, size_t ss, int xmtt,
                       hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
                                                // GPB column groups per block: 256 columns, or 128 for the 32-column groups
                                                // (8 groups per block measured 3 % slower on the 7B stream)
  const int ngroups = p.Npad / (16 * NT);
  const int nx = (ngroups + GPB - 1) / GPB, nz = (M + 16 * MT - 1) / (16 * MT);
  const int tasks8 = (nx * p.S + 7) / 8 * 8;
  launch_timed(gemm16_lds_kernel<DT, MT, NT, NTW, KC, PF, GPB>, dim3(tasks8 * nz), dim3(64 * GPB * (NT / NTW)), st, ev0, ev1,
               (const uint16_t*)x, (const u32x4_t*)wt, part, M, p.N, p.K, ngroups, p.KB, p.kbs, ss, p.ldc, nx, p.S, nz, xmtt);
}

template <int DT, int NTL, int EPI>
static void launch_rows(const void* x, const void* wt, const TileOut& o, int M, const GemmPlan& p, int xmtt, hipStream_t st,
                        hipEvent_t ev0, hipEvent_t ev1) {
  const int ngroups = p.Npad / 64;            // units of 64 columns, whatever the layout's group width
  const int nx = (ngroups + 3) / 4, nz = (M + 255) / 256;
  const int tasks8 = (nx * p.S + 7) / 8 * 8;
  launch_timed(gemm16_rows_kernel<DT, NTL, EPI>, dim3(tasks8 * nz), dim3(512), st, ev0, ev1, (const uint16_t*)x,
               (const u32x4_t*)wt, o, M, p.N, p.K, ngroups, p.KB, p.kbs, nx, p.S, nz, xmtt);
}

template <int DT, int A, int B, int WR, int WC, int D, int EPI>
static void launch_tile(const void* x, const void* wt, const TileOut& o, int M, const GemmPlan& p, int xmtt, hipStream_t st,
                        hipEvent_t ev0, hipEvent_t ev1) {
  const int nrb = (M + 16 * A * WR - 1) / (16 * A * WR), ncb = (p.N + 16 * B * WC - 1) / (16 * B * WC);
  const int tasks = nrb * ncb * p.S, per = (tasks + 7) / 8;
  launch_timed(gemm16_tile_kernel<DT, A, B, WR, WC, D, EPI>, dim3(per * 8), dim3(64 * WR * WC), st, ev0, ev1, (const uint16_t*)x,
               (const char*)wt, o, M, p.N, p.K, p.Npad / 16, p.NT, p.KB, p.kbs, ncb, nrb, tasks, per, xmtt);
}
template <int DT, int A, int B, int WC, int WK, int PF, int L, int EPI>
static void launch_parts(const void* x, const void* wt, const TileOut& o, int M, const GemmPlan& p, int xmtt, hipStream_t st,
                         hipEvent_t ev0, hipEvent_t ev1) {
  const int nrb = (M + 16 * A - 1) / (16 * A), ncb = (p.N + 16 * B * WC - 1) / (16 * B * WC);
  const int tasks = nrb * ncb * p.S, per = (tasks + 7) / 8;
  launch_timed(gemm16_parts_kernel<DT, A, B, WC, WK, PF, L, EPI>, dim3(per * 8), dim3(64 * WC * WK), st, ev0, ev1, (const uint16_t*)x,
               (const u32x4_t*)wt, o, M, p.N, p.K, p.Npad / 16, p.NT, p.KB, p.kbs, ncb, nrb, tasks, per, xmtt);
}
// Whether a context pass's GEMM takes K in parts inside the block; the windows' slices are single chains, so they never do.
// us per launch, cold weights, both operands through LDS -> in parts: 64 x 64 blocks 2048 x 2048 at 287 / 436 rows (160 / 224 blocks) 11.3 /
// 11.5 -> 8.0 / 8.5, 4096 x 4096 at 138 (192) 28.6 -> 16.6, 2048 x 2048 at 943 (480 blocks, which share the compute units) 15.1 -> 17.4;
// 64 x 128 6144 x 2048 at 287 (240) 18.4 -> 16.4, at 436 (336) 26.3 -> 31.0; slices of 16 k-blocks 6.4 -> 7.4; 128 x 256 12288 x 4096 at 138 /
// 780 (192 / 336) 56.0 / 112 -> 52.9 / 104; 128 x 128 gains nothing (6144 x 2048 at 436 22.7 -> 22.4) and loses on short slices.
// Two overlapped passes share the compute units: with at most 240 blocks in parts two of 200 and 230 rows, GPT-1.3B shape, six layers, take 566
// us instead of 627 (7B shape, four layers, 932 for 943), but one after the other 1011 instead of 952; weighed as in context_plan, level.
// Row-major rows of an operation-level call come half a cache line at a time and every part fetches its own: gate|up, F x K at rows, LDS -> parts,
// us per call: 64 x 64 blocks 640 x 6656 at 287 35.3 -> 38.2, 1280 x 1024 at 200 26.2 -> 28.0; 64 x 128 3520 x 1024 at 129 28.6 -> 30.7; 128 x 256
// 14400 x 2048 at 256 62.3 -> 66.1, 4800 x 3584 at 640 69.2 -> 71.6, 11200 x 5632 at 200 111 -> 114, but long chains gain from 256 rows on:
// 11200 x 4608 at 256 111 -> 108, 14400 x 4608 at 640 267 -> 256, 17920 x 6656 at 300 254 -> 244.
static bool parts_pay(int tile, int M, const GemmPlan& p, bool row_major) {
  const int last = p.KB - (p.S - 1) * p.kbs;
  if (p.tile < 0 || tile == TILE_128X128 || last < 32) return false;
  if (row_major) return tile == TILE_128X256 && M >= 256 && last >= 144;
  return tile == TILE_128X256 || tile_blocks(tile, M, p, p.S) <= 256;
}
// 64-column blocks do not hold the rotary partners of a 128-wide head: that epilogue takes 128 columns instead
template <int DT, int EPI>
static void dispatch_tile(int tile, const void* x, const void* wt, const TileOut& o, int M, const GemmPlan& p, int xmtt, hipStream_t st,
                          hipEvent_t ev0, hipEvent_t ev1) {
  if (EPI == EPI_QKV && tile == TILE_64X64) tile = TILE_64X128;
  if (tile == TILE_ROWS) {
    if (p.NT == 4) {
      if constexpr (EPI != EPI_GATED) launch_rows<DT, 4, EPI>(x, wt, o, M, p, xmtt, st, ev0, ev1);   // paired layouts have NT = 2
    } else {
      launch_rows<DT, 2, EPI>(x, wt, o, M, p, xmtt, st, ev0, ev1);
    }
  }
  else if (parts_pay(tile, M, p, xmtt == 0)) {
    if (tile == TILE_128X256) launch_parts<DT, 8, 4, 4, 2, 4, 4, EPI>(x, wt, o, M, p, xmtt, st, ev0, ev1);
    else if (tile == TILE_64X128) launch_parts<DT, 4, 4, 2, 4, 4, 4, EPI>(x, wt, o, M, p, xmtt, st, ev0, ev1);
    else if constexpr (EPI != EPI_QKV) launch_parts<DT, 4, 2, 2, 4, 4, 3, EPI>(x, wt, o, M, p, xmtt, st, ev0, ev1);
  }
  else if (tile == TILE_128X256) launch_tile<DT, 4, 4, 2, 4, 4, EPI>(x, wt, o, M, p, xmtt, st, ev0, ev1);
  else if (tile == TILE_128X128) launch_tile<DT, 2, 4, 4, 2, 4, EPI>(x, wt, o, M, p, xmtt, st, ev0, ev1);
  else if (tile == TILE_64X128) launch_tile<DT, 2, 4, 2, 2, 4, EPI>(x, wt, o, M, p, xmtt, st, ev0, ev1);
  else if constexpr (EPI != EPI_QKV) launch_tile<DT, 2, 2, 2, 2, 4, EPI>(x, wt, o, M, p, xmtt, st, ev0, ev1);
}
// The whole-K kernel per count of row tiles; four k-blocks ahead, two where the rows' operand would take too many registers (eight
// were 3 to 25 % slower: a longer way to the first product).
template <int DT, int EPI, int MT>
static void launch_whole(const void* x, const void* wt, const TileOut& o, int M, const GemmPlan& p, int xmtt, hipStream_t st,
                         hipEvent_t ev0, hipEvent_t ev1) {
  launch_timed(gemm16_whole_kernel<DT, MT, kWholeSlices, MT <= 3 ? 4 : 2, EPI>, dim3((p.N + 31) / 32), dim3(64 * kWholeSlices), st, ev0, ev1,
               (const uint16_t*)x, (const u32x4_t*)wt, o, M, p.N, p.KB, p.kbs, xmtt);
}
constexpr int kSumRows = 64;
template <int DT, int EPI>
static void dispatch_whole(const void* x, const void* wt, const TileOut& o, int M, const GemmPlan& p, int xmtt, hipStream_t st,
                           hipEvent_t ev0, hipEvent_t ev1) {
  switch ((M + 15) / 16) {
    case 1: return launch_whole<DT, EPI, 1>(x, wt, o, M, p, xmtt, st, ev0, ev1);
    case 2: return launch_whole<DT, EPI, 2>(x, wt, o, M, p, xmtt, st, ev0, ev1);
    case 3: return launch_whole<DT, EPI, 3>(x, wt, o, M, p, xmtt, st, ev0, ev1);
    case 4: return launch_whole<DT, EPI, 4>(x, wt, o, M, p, xmtt, st, ev0, ev1);
  }
  if constexpr (EPI != EPI_PART) {               // sums: up to kSumRows rows
    switch ((M + 15) / 16) {
      case 5: return launch_whole<DT, EPI, 5>(x, wt, o, M, p, xmtt, st, ev0, ev1);
      case 6: return launch_whole<DT, EPI, 6>(x, wt, o, M, p, xmtt, st, ev0, ev1);
      case 7: return launch_whole<DT, EPI, 7>(x, wt, o, M, p, xmtt, st, ev0, ev1);
      default: return launch_whole<DT, EPI, 8>(x, wt, o, M, p, xmtt, st, ev0, ev1);
    }
  }
}
static bool takes_whole(const GemmPlan& p, int M) { return p.whole && M <= kWholeRows; }
// Above kWholeRows rows of a fused iteration a block still takes all of K and finishes the job: gemm16_parts_kernel, whose four parts are
// then the plan's slices (K is a multiple of four k-blocks), so that a row's bits are those of gemm16_whole_kernel.  The smallest block
// whose blocks all run at once, else 128 x 128.  us, 64 x 64 / 64 x 128 / 128 x 128 and in brackets the two launches with two or three
// slices in memory: 4096 x 2048 with SwiGLU at 160 rows (192 / 96 / 64 blocks) 10.6 / 15.6 / 20.6 [18.0], at 384 (384 / 192 / 96) 20.5 / 16.2 /
// 22.1 [23.5], at 1000 42.3 / 32.6 / 24.2 [36.5]; 8192 x 2048 with GELU at 160 (384 / 192 / 128) 23.8 / 19.5 / 25.8 [26.6], at 512 48.2 /
// 37.6 / 28.1 [44.0], at 1000 95.0 / 74.2 / 55.2 [77.8]; 6144 x 2048 q|k|v at 256 - / 19.0 / 25.6 [25.9], at 384 - / 29.0 / 25.3 [28.1], at 700 (288
// blocks of 128 x 128, the one size found where it is not ahead) - / 45.7 / 42.4 [42.0], with the rotation 45.1 / 43.8 [41.4].
static bool whole_window(const GemmPlan& p, int M) { return p.whole && M > kWholeRows && p.tile < 0; }
static bool one_round(int tile, int M, const GemmPlan& p) { return tile_blocks(tile, M, p, 1) <= 256; }
template <int DT, int EPI>
static void dispatch_whole_window(const void* x, const void* wt, const TileOut& o, int M, const GemmPlan& p, int xmtt, hipStream_t st,
                                  hipEvent_t ev0, hipEvent_t ev1) {
  GemmPlan q = p;
  q.S = 1;
  q.kbs = q.KB;
  if constexpr (EPI != EPI_QKV) {                // whose 128 columns hold the rotary partners
    if (one_round(TILE_64X64, M, p)) return launch_parts<DT, 4, 2, 2, kWholeSlices, 4, 3, EPI>(x, wt, o, M, q, xmtt, st, ev0, ev1);
  }
  if (one_round(TILE_64X128, M, p)) launch_parts<DT, 4, 4, 2, kWholeSlices, 4, 4, EPI>(x, wt, o, M, q, xmtt, st, ev0, ev1);
  else launch_parts<DT, 8, 4, 2, kWholeSlices, 4, 3, EPI>(x, wt, o, M, q, xmtt, st, ev0, ev1);
}
template <int EPI>
static hipError_t finish(int dtype, const void* x, const void* wt, const TileOut& o, int M, const GemmPlan& p, int xmtt, hipStream_t st,
                         hipEvent_t ev0, hipEvent_t ev1) {
  if (dtype == DT_F32) {
    const int pairs = EPI == EPI_GATED ? o.F : (p.N + 1) / 2;
    const dim3 grid((pairs + 3) / 4, (M + 7) / 8);
    auto launch = [&](void (*kernel)(const float*, const float*, TileOut, int, int, int)) {
      launch_timed(kernel, grid, dim3(256), st, ev0, ev1, (const float*)x, (const float*)wt, o, M, p.N, p.K);
    };
    const bool one = p.K <= 256;
    if (!o.norm.g) {
      launch(one ? gemm32_kernel<EPI, 1, 0> : gemm32_kernel<EPI, 4, 0>);
    } else if constexpr (EPI != EPI_ADD) {
      if (p.K > 1024) return hipErrorInvalidValue;
      if (o.norm.rms) launch(one ? gemm32_kernel<EPI, 1, 2> : gemm32_kernel<EPI, 4, 2>);
      else launch(one ? gemm32_kernel<EPI, 1, 1> : gemm32_kernel<EPI, 4, 1>);
    }
    return hipGetLastError();
  }
  if constexpr (EPI != EPI_ADD) {
    if (takes_whole(p, M)) {
      if (dtype == DT_BF16) dispatch_whole<DT_BF16, EPI>(x, wt, o, M, p, xmtt, st, ev0, ev1);
      else dispatch_whole<DT_F16, EPI>(x, wt, o, M, p, xmtt, st, ev0, ev1);
      return hipGetLastError();
    }
    if constexpr (EPI != EPI_PART) {
      if (whole_window(p, M)) {
        if (p.KB % kWholeSlices) return hipErrorInvalidValue;
        if (dtype == DT_BF16) dispatch_whole_window<DT_BF16, EPI>(x, wt, o, M, p, xmtt, st, ev0, ev1);
        else dispatch_whole_window<DT_F16, EPI>(x, wt, o, M, p, xmtt, st, ev0, ev1);
        return hipGetLastError();
      }
    }
  }
  if (dtype == DT_BF16) dispatch_tile<DT_BF16, EPI>(p.tile, x, wt, o, M, p, xmtt, st, ev0, ev1);
  else dispatch_tile<DT_F16, EPI>(p.tile, x, wt, o, M, p, xmtt, st, ev0, ev1);
  return hipGetLastError();
}
// Every wave repeats the norm of its eight rows, and where a SIMD takes several waves their norms follow each other: inside pays while
// that is less than the launch saved (3 us and the gap before it, 4 to 5 us of a chain).  us per launch, norm apart -> inside, by
// blocks of four waves: rows of 256 columns (one 16-byte piece per lane), layer norm 256 blocks 3.4 -> 4.9, 512 3.7 -> 6.6, 768 4.0 ->
// 8.2, 1000 4.0 -> 9.8, 6283 (an output projection of 50257) 11.6 -> 42.8, RMS 3.3 -> 4.2, 3.7 -> 5.6, 4.0 -> 7.0, 4.0 -> 7.6, 11.6 -> 32.9;
// of 512 to 1024 columns, layer norm 256 blocks 4.7 -> 8.4, 384 6.1 -> 14.8, 1024 9.2 -> 27.2, RMS 4.6 -> 7.2, 6.0 -> 10.7, 9.8 -> 17.2.
bool gemm_norms(int dtype, int M, const GemmPlan& p) {
  const long blocks = (long)(((p.N + 1) / 2 + 3) / 4) * ((M + 7) / 8);      // of gemm32_kernel
  return dtype == DT_F32 && p.K <= 1024 && M <= 32 && blocks <= (p.K <= 256 ? 512 : 256);
}
bool gemm_finishes(int dtype, const GemmPlan& p, int M) {
  return dtype == DT_F32 || takes_whole(p, M) || whole_window(p, M) || (M > 128 && p.S == 1 && p.tile >= 0);
}

hipError_t gemm_qkv(int dtype, const void* x, const void* wt, int M, const GemmPlan& p, const TileOut& o, int xmtt, hipStream_t st,
                    hipEvent_t ev0, hipEvent_t ev1) {
  return finish<EPI_QKV>(dtype, x, wt, o, M, p, xmtt, st, ev0, ev1);
}
hipError_t gemm_add(int dtype, const void* x, const void* wt, int M, const GemmPlan& p, float* res, const void* bias, int xmtt, hipStream_t st,
                    hipEvent_t ev0, hipEvent_t ev1) {
  TileOut o;
  o.part = res;
  o.ldc = p.N;
  o.bias = bias;
  return finish<EPI_ADD>(dtype, x, wt, o, M, p, xmtt, st, ev0, ev1);
}
hipError_t gemm_act(int dtype, bool swiglu, const void* x, const void* wt, int M, const GemmPlan& p, void* act, const void* bias, int xmtt,
                    hipStream_t st, hipEvent_t ev0, hipEvent_t ev1, const NormIn& norm) {
  TileOut o;
  o.norm = norm;
  o.act = act;
  o.bias = bias;
  o.F = swiglu ? p.N / 2 : p.N;
  o.mtt = xmtt;
  return swiglu ? finish<EPI_GATED>(dtype, x, wt, o, M, p, xmtt, st, ev0, ev1) : finish<EPI_GELU>(dtype, x, wt, o, M, p, xmtt, st, ev0, ev1);
}

// The copies to LDS move whole 16-byte pieces; operands of an operation-level call may start anywhere.
static bool aligned16(const void* x, const void* wt) { return (((uintptr_t)x | (uintptr_t)wt) & 15) == 0; }

template <int DT, int NT>
static void dispatch16(const void* x, const void* wt, float* part, int M, const GemmPlan& p, size_t ss, int xmtt,
                       hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  // up to 128 rows, and rows or weights off the 16-byte grid: through registers, row blocks of at most 128 rows
  const bool regs = M <= 128 || !aligned16(x, wt);
  if (M <= 16) launch_direct<DT, 1, NT, 8, 8>(x, wt, part, M, p, ss, xmtt, st, ev0, ev1);
  else if (M <= 32) launch_lds<DT, 2, NT, NT, 4, 4, (NT == 2 ? 4 : 2)>(x, wt, part, M, p, ss, xmtt, st, ev0, ev1);     // 4 waves, one per column group
  else if (NT == 2 && !p.paired && regs) {
    // 32-column groups above 32 rows: two waves per group, one n-tile each (8 waves per 128-column block); measured
    // 0.6 us (33-64 rows) and 1.5 us (65-128 rows) faster per launch than one wave per group.  For these groups chunks
    // of 4 k-blocks (half the barriers) are 0.2-1.5 us faster per launch at every row count; for the 64-column ones not.
    // one variant per count of 16-row tiles: a block stages and multiplies exactly the live tiles
    switch ((M + 15) / 16) {
      case 3: launch_lds<DT, 3, NT, 1, 4, 4, 4>(x, wt, part, M, p, ss, xmtt, st, ev0, ev1); break;
      case 4: launch_lds<DT, 4, NT, 1, 4, 4, 4>(x, wt, part, M, p, ss, xmtt, st, ev0, ev1); break;
      case 5: launch_lds<DT, 5, NT, 1, 4, 4, 4>(x, wt, part, M, p, ss, xmtt, st, ev0, ev1); break;
      case 6: launch_lds<DT, 6, NT, 1, 4, 4, 4>(x, wt, part, M, p, ss, xmtt, st, ev0, ev1); break;
      case 7: launch_lds<DT, 7, NT, 1, 4, 4, 4>(x, wt, part, M, p, ss, xmtt, st, ev0, ev1); break;
      default: launch_lds<DT, 8, NT, 1, 4, 4, 4>(x, wt, part, M, p, ss, xmtt, st, ev0, ev1);
    }
  }
  else if (regs && !(NT == 2 && p.paired)) {
    switch ((M + 15) / 16) {                                                                  // 8 waves, two per column group
      case 3: launch_lds<DT, 3, NT, 2, 4>(x, wt, part, M, p, ss, xmtt, st, ev0, ev1); break;
      case 4: launch_lds<DT, 4, NT, 2, 4>(x, wt, part, M, p, ss, xmtt, st, ev0, ev1); break;
      case 5: launch_lds<DT, 5, NT, 2, 4>(x, wt, part, M, p, ss, xmtt, st, ev0, ev1); break;
      case 6: launch_lds<DT, 6, NT, 2, 4>(x, wt, part, M, p, ss, xmtt, st, ev0, ev1); break;
      case 7: launch_lds<DT, 7, NT, 2, 4>(x, wt, part, M, p, ss, xmtt, st, ev0, ev1); break;
      default: launch_lds<DT, 8, NT, 2, 4>(x, wt, part, M, p, ss, xmtt, st, ev0, ev1);
    }
  }
  else if (M <= 64) launch_lds<DT, 4, NT, 2, 4>(x, wt, part, M, p, ss, xmtt, st, ev0, ev1);
  else if (regs) launch_lds<DT, 8, NT, 2, 4, 8>(x, wt, part, M, p, ss, xmtt, st, ev0, ev1);   // paired: 8 groups, 256 columns
  else {                                                                             // context passes, very wide windows
    TileOut o;
    o.part = part;
    o.slice_stride = ss;
    o.ldc = p.ldc;
    dispatch_tile<DT, EPI_PART>(p.tile < 0 ? best_tile(M, p) : p.tile, x, wt, o, M, p, xmtt, st, ev0, ev1);
  }
}

template <int DT, int MT, int KC, int PF, int GPB, int P>
static void launch_gated(const void* x, const void* wt, void* act, int M, const GemmPlan& p, int xmtt, hipStream_t st, hipEvent_t ev0,
                         hipEvent_t ev1) {
  const int F = p.N / 2, ngroups = F / 16;
  launch_timed(gated_lds_kernel<DT, MT, KC, PF, GPB, P>, dim3((ngroups + GPB - 1) / GPB), dim3(128 * (GPB + P)), st, ev0, ev1, (const uint16_t*)x,
               (const u32x4_t*)wt, act, M, F, ngroups, p.KB, xmtt);
}
// One variant per count of 16-row tiles; chunks of 4 k-blocks at one row tile (half the barriers), of 2 above.  P2: copying waves per half from two
// tiles up, as many as fill the four SIMDs evenly; none where twelve waves leave too few registers for a second set of fragments (GPB 4 and 5 from
// seven tiles up: 11008 x 4096 at 120 rows, GPB 4, 51 -> 72 us).  At GPB 5 the ring is 4 deep from three tiles on for the same reason.
template <int DT, int GPB, int P2>
static void dispatch_gated(const void* x, const void* wt, void* act, int M, const GemmPlan& p, int xmtt, hipStream_t st, hipEvent_t ev0,
                           hipEvent_t ev1) {
  constexpr int P7 = GPB <= 3 ? P2 : 0, RING = GPB <= 4 ? 8 : 4;
  switch ((M + 15) / 16) {
    case 1: return launch_gated<DT, 1, 4, 8, GPB, 0>(x, wt, act, M, p, xmtt, st, ev0, ev1);
    case 2: return launch_gated<DT, 2, 2, 8, GPB, P2>(x, wt, act, M, p, xmtt, st, ev0, ev1);
    case 3: return launch_gated<DT, 3, 2, RING, GPB, P2>(x, wt, act, M, p, xmtt, st, ev0, ev1);
    case 4: return launch_gated<DT, 4, 2, RING, GPB, P2>(x, wt, act, M, p, xmtt, st, ev0, ev1);
    case 5: return launch_gated<DT, 5, 2, 4, GPB, P2>(x, wt, act, M, p, xmtt, st, ev0, ev1);
    case 6: return launch_gated<DT, 6, 2, 4, GPB, P2>(x, wt, act, M, p, xmtt, st, ev0, ev1);
    case 7: return launch_gated<DT, 7, 2, 4, GPB, P7>(x, wt, act, M, p, xmtt, st, ev0, ev1);
    default: return launch_gated<DT, 8, 2, 4, GPB, P7>(x, wt, act, M, p, xmtt, st, ev0, ev1);
  }
}
template <int DT>
static void dispatch_gated(const void* x, const void* wt, void* act, int M, const GemmPlan& p, int xmtt, hipStream_t st, hipEvent_t ev0,
                           hipEvent_t ev1) {
  switch (gated_groups(p)) {
    case 2: return dispatch_gated<DT, 2, 2>(x, wt, act, M, p, xmtt, st, ev0, ev1);
    case 3: return dispatch_gated<DT, 3, 1>(x, wt, act, M, p, xmtt, st, ev0, ev1);
    case 4: return dispatch_gated<DT, 4, 2>(x, wt, act, M, p, xmtt, st, ev0, ev1);
    case 5: return dispatch_gated<DT, 5, 1>(x, wt, act, M, p, xmtt, st, ev0, ev1);
    default:                                     // M <= 64
      if (M <= 16) return launch_gated<DT, 1, 4, 8, 8, 0>(x, wt, act, M, p, xmtt, st, ev0, ev1);
      if (M <= 32) return launch_gated<DT, 2, 4, 8, 8, 0>(x, wt, act, M, p, xmtt, st, ev0, ev1);
      return launch_gated<DT, 4, 4, 4, 8, 0>(x, wt, act, M, p, xmtt, st, ev0, ev1);
  }
}

// Rows in fragment order (see xrow_index) from row-major ones that start at any element; rows past the last repeat it.  A block: a row
// tile, four k-blocks.
__global__ __launch_bounds__(256) void lay_rows_kernel(const uint16_t* __restrict__ x, u32x4_t* __restrict__ to, int M, int K, int KB, int mtt) {
  const int lane = threadIdx.x & 63, mt = blockIdx.x, kb = blockIdx.y * 4 + (threadIdx.x >> 6);
  if (kb >= KB) return;
  const int m = min(mt * 16 + (lane & 15), M - 1);
  to[((size_t)kb * mtt + mt) * 64 + lane] = *(const u32x4_any*)(x + (size_t)m * K + kb * 32 + (lane >> 4) * 8);
}

// The iteration's plan, up to gated_fused_rows(p) rows: one launch.  Above that gemm() with the plan's K slices as partial sums and the
// activation as its own launch -- the same chains, added in the same order, rounded once: bit-identical results (the one
// launch at 90 and 128 rows, call included: 17920 x 6656 139 -> 98 us, 17408 x 3072 93 -> 62).
// A whole plan is one launch there too; rows of an operation-level call, which are row-major, make its copies slow (half a cache line
// each, and none at all off the 16-byte grid), so with room for it
//   * where the blocks are one round and K is long the two launches stay (us, two -> one: 2048 x 6656 at 129 / 512 / 1000 rows 17 / 29 / 40
//     -> 34 / 36 / 48, 8192 x 4096 at 160 30.8 -> 32.7);
//   * where they are more, and off the grid, the rows are laid out in fragment order first (8192 x 4096 at 512 / 1000 rows, two launches /
//     one / laid out first 59 / 56 / 43 and 108 / 102 / 78; 8192 x 1536 at 1000 71 / 50 / 43; off the grid, two launches -> laid out: 2048 x
//     6656 at 129 rows 38 -> 25, 2752 x 512 at 160 16 -> 11.5).
// A context pass's plan: one slice -> the kernel that the plan names with the activation as its epilogue; any other slice count ->
// gemm() and the activation launch.
hipError_t gemm_gated(int dtype, const void* x, const void* wt, int M, const GemmPlan& p, void* act, float* part,
                      size_t slice_stride, int xmtt, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1, size_t room) {
  if (M <= 0) return hipSuccess;
  if (!p.paired || dtype == DT_F32) return hipErrorInvalidValue;
  const bool grid16 = aligned16(x, wt), window = whole_window(p, M) && xmtt == 0, fits = part && room >= (size_t)p.S * slice_stride * 4;
  const bool rounds = window && !one_round(TILE_64X128, M, p);
  const int mtt = (M + 15) / 16;
  if (window && (rounds || !grid16) && aligned16(part, wt) && part && room >= (size_t)mtt * 1024 * p.KB) {
    lay_rows_kernel<<<dim3(mtt, (p.KB + 3) / 4), 256, 0, st>>>((const uint16_t*)x, (u32x4_t*)part, M, p.K, p.KB, mtt);
    TileOut o;
    o.act = act;
    o.F = p.N / 2;
    return finish<EPI_GATED>(dtype, part, wt, o, M, p, mtt, st, ev0, ev1);
  }
  const bool apart = window && fits && (!grid16 || (p.K > 2560 && !rounds));
  if (!apart && (takes_whole(p, M) || (gemm_finishes(dtype, p, M) && grid16)))
    return gemm_act(dtype, true, x, wt, M, p, act, nullptr, xmtt, st, ev0, ev1);
  if (!apart && gemm_finishes(dtype, p, M)) {      // rows that cannot be copied to LDS: the iteration's launches, which need no
    const GemmPlan it = gemm_plan_gated(dtype, p.N / 2, p.K);                                         // partial sums either
    for (int m = 0; m < M; m += gated_fused_rows(it)) {
      const hipError_t e = gemm_gated(dtype, (const uint16_t*)x + (size_t)m * p.K, wt, std::min(M - m, gated_fused_rows(it)), it,
                                      (uint16_t*)act + (size_t)m * (p.N / 2), nullptr, 0, 0, st);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  if (M > gated_fused_rows(p) || p.S != 2) {
    hipError_t e = gemm(dtype, x, wt, M, p, part, slice_stride, xmtt, st, ev0, nullptr);   // timed from the first launch's
    if (e != hipSuccess) return e;                                                       // start to the second's end
    return activation(dtype, true, part, p.S, slice_stride, p.ldc, nullptr, act, M, p.N / 2, xmtt, st, true, ev1);
  }
  if (dtype == DT_BF16) dispatch_gated<DT_BF16>(x, wt, act, M, p, xmtt, st, ev0, ev1);
  else dispatch_gated<DT_F16>(x, wt, act, M, p, xmtt, st, ev0, ev1);
  return hipGetLastError();
}

// Every block of 32 columns reads all rows, row-major, 64 bytes at a time: one launch while the rows are few (us per call, two launches ->
// one, at 17 / 32 / 64 rows: 1536 x 512 10.7 -> 7.4 / 7.5 / 7.6, 4224 x 1024 10.9 / 10.6 / 10.6 -> 7.4 / 7.4 / 9.2, 4480 x 1536 10.7 / 10.8 / 11.7 ->
// 7.4 / 8.7 / 12.5, 4864 x 2048 10.8 / 10.8 / 12.9 -> 7.9 / 10.6 / 14.1, 4160 x 2560 10.8 / 11.1 / 14.0 -> 9.7 / 13.1 / 19.1).  Rows off the 16-byte
// grid take several times as long to load: up to 16 rows 10 to 17 -> 8 to 15, at 17 rows 10.8 -> 14.6 (4864 x 2048).
bool gemm_adds_up(int dtype, const GemmPlan& p, int M, const void* x) {
  const bool few = M <= 16 || (M <= kSumRows && (long)M * p.K <= 60000 && ((uintptr_t)x & 15) == 0);
  return p.S == 1 || (dtype != DT_F32 && p.whole && few);
}
hipError_t gemm_sum(int dtype, const void* x, const void* wt, int M, const GemmPlan& p, float* y, int ldy, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  if (!gemm_adds_up(dtype, p, M, x)) return hipErrorInvalidValue;
  TileOut o;
  o.part = y;
  o.ldc = ldy;
  if (p.S > 1) return finish<EPI_PART>(dtype, x, wt, o, M, p, 0, st, nullptr, nullptr);
  GemmPlan q = p;
  q.ldc = ldy;
  return gemm(dtype, x, wt, M, q, y, 0, 0, st);
}

hipError_t gemm(int dtype, const void* x, const void* wt, int M, const GemmPlan& p, float* part, size_t slice_stride,
                int xmtt, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1, const NormIn& norm) {
  if (M <= 0) return hipSuccess;
  if (dtype == DT_F32) {
    if (xmtt) return hipErrorInvalidValue;   // fp32 rows are always row-major
    TileOut o;
    o.norm = norm;
    o.part = part;
    o.ldc = p.ldc;
    return finish<EPI_PART>(dtype, x, wt, o, M, p, 0, st, ev0, ev1);
  } else if (dtype == DT_BF16) {
    if (p.NT == 4) dispatch16<DT_BF16, 4>(x, wt, part, M, p, slice_stride, xmtt, st, ev0, ev1);
    else dispatch16<DT_BF16, 2>(x, wt, part, M, p, slice_stride, xmtt, st, ev0, ev1);
  } else {
    if (p.NT == 4) dispatch16<DT_F16, 4>(x, wt, part, M, p, slice_stride, xmtt, st, ev0, ev1);
    else dispatch16<DT_F16, 2>(x, wt, part, M, p, slice_stride, xmtt, st, ev0, ev1);
  }
  return hipGetLastError();
}

}  // namespace flk
