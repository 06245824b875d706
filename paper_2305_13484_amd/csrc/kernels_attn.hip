// Ragged masked self-attention of one fused decode iteration: every live row attends over its own request's
// cached K/V rows [0, len) -- requests arrived at different times, so every row has its own length
// (temporal fusion, Section V-C; the attention itself sits in Algorithm 2's "...").
//
// HBM-bound (about 1 flop per byte, every K/V byte read once), so the kernel is a streamer:
//   * the cache is [slot][head][pos][d]: one head's rows are contiguous, a wave load instruction fetches
//     64 lanes x 16 B = 1 KiB of consecutive rows, each row spread over LPR = d*elem/16 adjacent lanes;
//   * the lane group that holds a row reduces q.k over its LPR lanes with DPP, keeps its own online softmax
//     state (m, l, o) over the rows it sees (rows r with r % (64/LPR) == group), and the groups are merged
//     once at the end -- no LDS, no barriers, registers only, occupancy hides latency;
//   * work is flattened to (row, chunk) x head so a launch has thousands of similar wave tasks however ragged the
//     lengths are: a row of len positions has ceil(len / CHUNK) chunks of equal length (no short remainder task, which
//     would leave the memory system under-used while the full-length tasks finish); chunking depends on the
//     request's own length only, and a row's chunks are merged in chunk order (results never depend on other rows): by a
//     second tiny kernel, or, where it is the shorter way, by the block that has taken all of them (attn_row_kernel);
//     where every row of a launch has one chunk, the first kernel writes the output itself.
// Context passes of 16-bit models take the matrix cores instead (attn_context_kernel).
#include <algorithm>
#include <type_traits>

#include "flover_dev.h"
#include "flover_kernels.h"

namespace flk {

// the pair at distance d (8, 16 or 32; a constant once the loops below are unrolled) added, or the larger of it
__device__ __forceinline__ float sum_over(float v, int d) { return d == 8 ? v + __shfl_xor(v, 8, 64) : d == 16 ? sum_partner<16>(v) : sum_partner<32>(v); }
__device__ __forceinline__ float max_over(float v, int d) { return d == 8 ? fmaxf(v, __shfl_xor(v, 8, 64)) : d == 16 ? max_partner<16>(v) : max_partner<32>(v); }

__device__ __forceinline__ int chunks_of(int len) { return ((unsigned)len + kAttnChunk - 1) / kAttnChunk; }

// A wave's share of one (row, head): cache rows [j0, j1), every cache row on LPR lanes, RPW rows per load, the lane groups merged at
// the end.
template <int DT, int D, int U>
struct AttnWave {
  static constexpr int EB = (DT == DT_F32) ? 4 : 2;
  static constexpr int EPL = 16 / EB;          // elements per lane
  static constexpr int LPR = D / EPL;          // lanes per row
  static constexpr int RPW = 64 / LPR;         // rows per wave load
  static constexpr int STEP = RPW * U;
  const char *kb, *vb;                         // this lane's piece of cache row 0
  int j1, grp;
  float qf[EPL], m, l, o[EPL];

  __device__ __forceinline__ void start(const void* kc, const void* vc, size_t head_off, int j1_, int lane) {
    const size_t off = head_off + (size_t)(lane % LPR) * 16;
    kb = (const char*)kc + off;
    vb = (const char*)vc + off;
    j1 = j1_;
    grp = lane / LPR;
    m = -INFINITY;
    l = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) o[e] = 0.f;
  }
  __device__ __forceinline__ void query(const u32x4_t& qr, float scale) {
    unpack16<DT>(qr, qf);
#pragma unroll
    for (int e = 0; e < EPL; ++e) qf[e] *= scale;
  }
  __device__ __forceinline__ void load(u32x4_t* kr, u32x4_t* vr, int jb) const {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = min(jb + u * RPW + grp, j1 - 1);      // clamp: stays inside the request's valid rows
      kr[u] = __builtin_nontemporal_load((const u32x4_t*)(kb + (size_t)r * D * EB));
      vr[u] = __builtin_nontemporal_load((const u32x4_t*)(vb + (size_t)r * D * EB));
    }
  }
  __device__ __forceinline__ void consume(const u32x4_t* kr, const u32x4_t* vr, int jb) {
    float s[U];
    float tmax = -INFINITY;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float kf[EPL];
      unpack16<DT>(kr[u], kf);
      float d0 = 0.f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) d0 = fmaf(qf[e], kf[e], d0);
      d0 = group_sum<LPR>(d0);
      s[u] = (jb + u * RPW + grp < j1) ? d0 : -INFINITY;
      tmax = fmaxf(tmax, s[u]);
    }
    const float mn = fmaxf(m, tmax);
    const float ms = (mn == -INFINITY) ? 0.f : mn;       // a group that has seen no valid row yet
    const float alpha = __expf(m - ms);                  // m = -inf -> 0
    l *= alpha;
#pragma unroll
    for (int e = 0; e < EPL; ++e) o[e] *= alpha;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float p = __expf(s[u] - ms);
      l += p;
      float vf[EPL];
      unpack16<DT>(vr[u], vf);
#pragma unroll
      for (int e = 0; e < EPL; ++e) o[e] = fmaf(p, vf[e], o[e]);
    }
    m = mn;
  }
  // Rows [j0, j1), whose first STEP are already under way in krA, vrA.  Two register buffers: the loads of the next rows are in flight
  // while the current ones are consumed.  Steady state without branches (the compiler's wait counts for the in-order memory counter
  // collapse to "wait for everything" around a branch, which would make consuming one buffer wait for the other's loads too); the
  // loads past the chunk re-read its last row.
  __device__ __forceinline__ void rows(u32x4_t (&krA)[U], u32x4_t (&vrA)[U], int j0) {
    u32x4_t krB[U], vrB[U];
    int jb = j0;
    for (; jb + 2 * STEP <= j1; jb += 2 * STEP) {
      load(krB, vrB, jb + STEP);
      __builtin_amdgcn_sched_barrier(0);
      consume(krA, vrA, jb);
      load(krA, vrA, jb + 2 * STEP);
      __builtin_amdgcn_sched_barrier(0);
      consume(krB, vrB, jb + STEP);
    }
    if (jb < j1) {                                         // one or two steps left (wave-uniform)
      const bool two = jb + STEP < j1;
      if (two) load(krB, vrB, jb + STEP);
      consume(krA, vrA, jb);
      if (two) consume(krB, vrB, jb + STEP);
    }
  }
  // merge the RPW lane groups (lanes with equal lane % LPR): butterfly over the group index bits
  __device__ __forceinline__ void merge_groups() {
    if constexpr (RPW > 1) {
      float mt = m;
#pragma unroll
      for (int dlt = LPR; dlt < 64; dlt <<= 1) mt = max_over(mt, dlt);
      const float w = (m == -INFINITY) ? 0.f : __expf(m - mt);
      l *= w;
#pragma unroll
      for (int e = 0; e < EPL; ++e) o[e] *= w;
#pragma unroll
      for (int dlt = LPR; dlt < 64; dlt <<= 1) {
        l = sum_over(l, dlt);
#pragma unroll
        for (int e = 0; e < EPL; ++e) o[e] = sum_over(o[e], dlt);
      }
      m = mt;
    }
  }
};

// A chunk's share of the merged row, w = exp(its maximum - the row's).
__device__ __forceinline__ void add_chunk(float& l, f32x4_t& o, float w, float lc, const f32x4_t& oc) {
  l = fmaf(w, lc, l);
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = fmaf(w, oc[e], o[e]);
}

// Where a launch's work comes from, in either case row by row, one item per chunk: a list in device memory (the fused
// iteration, and operation-level calls of more than 256 rows), or the rows' descriptors as a kernel argument (no copy to the
// device, no wait, no launch before this one).  There every wave finds item i by itself: lane t holds rows 4t .. 4t+3 and the
// wave adds up their chunk counts -- one round of loads and a handful of lane operations, no longer than a list's round of
// loads (both 67 us at 48 rows x 32 heads of up to 1000 positions, 128 wide, bf16; 31 us at 64 rows x 4 heads of up to 2000).
// A grid of rows x most chunks with block i = chunk i / M of row i % M needs no search, but leaves blocks without work and
// puts all chunks of a row on one XCD where M is a multiple of 8: 78 and 30 us.
struct ItemList {
  const int4* items;
  const int* row_len;
  __device__ int4 at(int i) const { return items[i]; }
  __device__ int len(int row) const { return row_len[row]; }
};
template <int CTRL, int ROWS> __device__ __forceinline__ int add_dpp(int v) {     // lanes without a source add zero
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false);
}
struct RowList {
  AttnRows r;
  int M;
  __device__ int4 at(int i) const {
    static_assert(kAttnRows == 4 * 64, "four rows per lane");
    const int lane = threadIdx.x & 63;
    int4 slot = {0, 0, 0, 0}, len = {0, 0, 0, 0};
    if (4 * lane < M) {                          // a few rows are a few of the argument's cache lines
      slot = *(const int4*)(r.slot + 4 * lane);
      len = *(const int4*)(r.len + 4 * lane);
    }
    const int n0 = chunks_of(len.x), n1 = n0 + chunks_of(len.y), n2 = n1 + chunks_of(len.z), n3 = n2 + chunks_of(len.w);
    int sum = n3;                                // inclusive scan over the wave
    sum = add_dpp<0x111, 0xf>(sum);              // row_shr 1, 2, 4, 8: within rows of 16 lanes
    sum = add_dpp<0x112, 0xf>(sum);
    sum = add_dpp<0x114, 0xf>(sum);
    sum = add_dpp<0x118, 0xf>(sum);
    sum = add_dpp<0x142, 0xa>(sum);              // lane 15 of rows 0 and 2 to rows 1 and 3
    sum = add_dpp<0x143, 0xc>(sum);              // lane 31 to rows 2 and 3
    const int own = __builtin_ctzll(__ballot(i < sum));      // the lane whose rows hold item i
    const int rel = i - (sum - n3);              // of that lane: the item within its four rows
    const int k = (rel >= n0) + (rel >= n1) + (rel >= n2);
    const int ch = rel - (k == 0 ? 0 : k == 1 ? n0 : k == 2 ? n1 : n2);
    return make_int4(__builtin_amdgcn_readlane(4 * lane + k, own), __builtin_amdgcn_readlane(ch, own),
                     __builtin_amdgcn_readlane(k == 0 ? slot.x : k == 1 ? slot.y : k == 2 ? slot.z : slot.w, own),
                     __builtin_amdgcn_readlane(k == 0 ? len.x : k == 1 ? len.y : k == 2 ? len.z : len.w, own));
  }
  __device__ int len(int row) const { return r.len[row]; }
};
struct RowOrder {             // rows as an argument, in the order of the blocks
  AttnRows r;
  int32_t row[kAttnRows];
  __device__ int4 at(int b) const { return make_int4(row[b], 0, r.slot[b], r.len[b]); }
};

// A wave takes one head of one item (row, chunk, slot, len).  side_by_side: grid = (n_head, items), block = 64, the heads of an item side by
// side, so that every XCD gets its share of a long row and every compute unit of few waves; otherwise grid = (items, n_head / 4), block = 256,
// wave w with head blockIdx.y * 4 + w (see wave_blocks).
// Writes the unnormalised partial (m, l, o[D]) of (row, chunk, head) at index (row * maxch + chunk) * n_head + head:
// the place depends on the row and the chunk alone, so the merge kernel finds a row's partials without looking anything up.
// ONE: no row of the launch has a second chunk, so the wave normalises and writes the output itself (what the merge kernel
// does with one chunk, bit for bit) and there is no merge launch.
template <int DT, int D, int U, bool ONE, class Src>
__global__ __launch_bounds__(256) void attn_partial_kernel(const void* __restrict__ q, const void* __restrict__ kc,
                                                           const void* __restrict__ vc, Src src, int nh, int side_by_side,
                                                           int Smax, int maxch,
                                                           float scale, float* __restrict__ pml, float* __restrict__ po,
                                                           void* __restrict__ out, int mtt) {
  typedef AttnWave<DT, D, U> Wave;
  constexpr int EPL = Wave::EPL, LPR = Wave::LPR;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int item = side_by_side ? blockIdx.y : blockIdx.x;
  const int hd = side_by_side ? blockIdx.x : blockIdx.y * 4 + wave;
  const int4 it = src.at(item);         // one load: the cache addresses below depend on nothing else
  const int row = it.x, ch = it.y, slot = it.z, len = it.w;
  // the row's ceil(len / kAttnChunk) chunks are made equally long, so that no wave task of a row is a short remainder
  const int nch = chunks_of(len);
  const int cr = (len + nch - 1) / nch;
  const int j0 = ch * cr, j1 = min(len, j0 + cr);
  const int li = lane % LPR;

  Wave w;
  w.query(*(const u32x4_t*)((const char*)q + ((size_t)(row * nh + hd) * D + li * EPL) * Wave::EB), scale);
  w.start(kc, vc, ((size_t)slot * nh + hd) * Smax * D * Wave::EB, j1, lane);
  u32x4_t krA[U], vrA[U];
  w.load(krA, vrA, j0);
  w.rows(krA, vrA, j0);
  w.merge_groups();
  const float m = w.m, l = w.l;
  const float(&o)[EPL] = w.o;
  if (w.grp != 0) return;
  if constexpr (ONE) {
#pragma unroll
    for (int e = 0; e < EPL; e += 4) {
      const f32x4_t v = f32x4_t{o[e], o[e + 1], o[e + 2], o[e + 3]} + 0.f;      // the merge adds to zero (-0 becomes +0)
      stv4<DT>(out, xrow_index(row, hd * D + li * EPL + e, nh * D, mtt), v / l);
    }
  } else {
    const size_t pi = ((size_t)row * maxch + ch) * nh + hd;
    float* op = po + pi * D + li * EPL;
#pragma unroll
    for (int e = 0; e < EPL; ++e) op[e] = o[e];
    if (li == 0) {
      pml[pi * 2] = m;
      pml[pi * 2 + 1] = l;
    }
  }
}

// A block per (row, head), a wave per chunk, the chunks merged through LDS: one launch, no partial results in memory.  grid = (n_head, M), a
// row's heads side by side, block = 64 * the most chunks of a row, kRowWaves waves at most (a wave then takes every kRowWaves-th chunk);
// waves without a chunk end at once, before the barrier, which waits for the others only.  blockIdx.y counts src,
// the longest row first, so that the launch does not end with the long rows: rows of up to 1900 positions in any order -> that order, 32 heads,
// bf16, us: 101 rows 240 -> 234 (caches of 2048 positions, whose heads lie 512 KB apart: 266 -> 243), 64 rows 157 -> 151, 24 rows 67 -> 62.
// 256 rows of up to 4096 positions 1253 us (6.85 TB/s); 1386 in two launches.  Streaming and merging are those of the other two kernels, in the same order: the same bits.
constexpr int kRowWaves = 8, kRowChunks = 16;
template <int DT, int D, int U, class Src>
__global__ __launch_bounds__(64 * kRowWaves) void attn_row_kernel(const void* __restrict__ q, const void* __restrict__ kc,
                                                                  const void* __restrict__ vc, Src src, int nh, int Smax, float scale,
                                                                  void* __restrict__ out, int mtt) {
  typedef AttnWave<DT, D, U> Wave;
  constexpr int EPL = Wave::EPL, LPR = Wave::LPR;
  __shared__ __attribute__((aligned(16))) float part[kRowChunks][D + 4];       // [chunk]: o, m, l
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int hd = blockIdx.x, li = lane % LPR;
  const int4 it = src.at(blockIdx.y);
  const int row = it.x, slot = it.z, len = it.w;
  const int nch = chunks_of(len);
  if (wave >= nch) return;
  const int cr = (len + nch - 1) / nch;                       // chunks of equal length, as in attn_partial_kernel
  Wave w;
  w.query(*(const u32x4_t*)((const char*)q + ((size_t)(row * nh + hd) * D + li * EPL) * Wave::EB), scale);
  for (int c = wave; c < nch; c += kRowWaves) {
    w.start(kc, vc, ((size_t)slot * nh + hd) * Smax * D * Wave::EB, min(len, (c + 1) * cr), lane);
    u32x4_t krA[U], vrA[U];
    w.load(krA, vrA, c * cr);
    w.rows(krA, vrA, c * cr);
    w.merge_groups();
    if (nch == 1) break;
    if (w.grp == 0) {
#pragma unroll
      for (int e = 0; e < EPL; ++e) part[c][li * EPL + e] = w.o[e];
      if (li == 0) {
        part[c][D] = w.m;
        part[c][D + 1] = w.l;
      }
    }
  }
  if (nch == 1) {
    if (w.grp != 0) return;
#pragma unroll
    for (int e = 0; e < EPL; e += 4) {
      const f32x4_t v = f32x4_t{w.o[e], w.o[e + 1], w.o[e + 2], w.o[e + 3]} + 0.f;
      stv4<DT>(out, xrow_index(row, hd * D + li * EPL + e, nh * D, mtt), v / w.l);
    }
    return;
  }
  __syncthreads();                                            // of the waves that have a chunk
  if (wave > 0 || lane >= D / 4) return;
  float m[kRowChunks];
  float top = -INFINITY, l = 0.f;
#pragma unroll
  for (int c = 0; c < kRowChunks; ++c)
    if (c < nch) {
      m[c] = part[c][D];
      top = fmaxf(top, m[c]);
    }
  f32x4_t o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < kRowChunks; ++c)
    if (c < nch) add_chunk(l, o, __expf(m[c] - top), part[c][D + 1], ld4(&part[c][lane * 4]));
  stv4<DT>(out, xrow_index(row, hd * D + lane * 4, nh * D, mtt), o / l);
}

// grid = (M, ceil(n_head / HPB)), block = 256: merges a row's chunks in chunk order, normalises, rounds to dtype.  A
// thread owns 4 consecutive elements of one head's output (D / 4 threads per head, HPB = 1024 / D heads per block).
// out is [M][nh * D] row-major (mtt == 0) or in the GEMM's fragment order with mtt row tiles.
// The partials of a row sit at a place known from the row index alone, so the loads of the first four chunks go out
// together with the load of the row's length (one memory round trip for rows of up to 4 chunks; slots of chunks the row
// does not have are read and never used); longer rows fetch the rest in a second round.
template <int DT, int D, class Src>
__global__ __launch_bounds__(256) void attn_merge_kernel(const float* __restrict__ pml, const float* __restrict__ po,
                                                         Src src, int maxch, int nh,
                                                         void* __restrict__ out, int mtt) {
  constexpr int FIRST = 4;
  constexpr int TPH = D / 4, HPB = 256 / TPH;
  const int row = blockIdx.x, hd = blockIdx.y * HPB + threadIdx.x / TPH, i = (threadIdx.x % TPH) * 4;
  if (hd >= nh) return;
  const size_t base = ((size_t)row * maxch) * nh + hd;       // + ch * nh
  float mc[FIRST], lc[FIRST];
  f32x4_t oc[FIRST];
#pragma unroll
  for (int j = 0; j < FIRST; ++j) {
    const size_t pi = base + (size_t)min(j, maxch - 1) * nh;
    const float2 ml = *(const float2*)(pml + pi * 2);
    mc[j] = ml.x;
    lc[j] = ml.y;
    oc[j] = ld4(po + pi * D + i);
  }
  const int nc = chunks_of(src.len(row));
  float red_m = -INFINITY;                                    // the global maximum needs the m of every chunk
#pragma unroll
  for (int j = 0; j < FIRST; ++j)
    if (j < nc) red_m = fmaxf(red_m, mc[j]);
  for (int c = FIRST; c < nc; ++c) red_m = fmaxf(red_m, pml[(base + (size_t)c * nh) * 2]);
  float l = 0.f;
  f32x4_t o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < FIRST; ++j)
    if (j < nc) {
      add_chunk(l, o, __expf(mc[j] - red_m), lc[j], oc[j]);
    }
  for (int c0 = FIRST; c0 < nc; c0 += 4) {      // longer rows: 4 chunks at a time, loads first, arithmetic in chunk order
    float m2[4], l2[4];
    f32x4_t o2[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const size_t pi = base + (size_t)min(c0 + j, nc - 1) * nh;
      const float2 ml = *(const float2*)(pml + pi * 2);
      m2[j] = ml.x;
      l2[j] = ml.y;
      o2[j] = ld4(po + pi * D + i);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (c0 + j < nc) {
        add_chunk(l, o, __expf(m2[j] - red_m), l2[j], o2[j]);
      }
  }
  stv4<DT>(out, xrow_index(row, hd * D + i, nh * D, mtt), o / l);
}

// ---------------------------------------------------------------- pre-processing variant (context decoder)
// Rows of one pre-processing pass are consecutive positions of ONE slot, so neighbouring rows read almost the same
// K/V rows.  Here a wave serves QB consecutive query rows at once: every K/V row it loads is used by all of them
// (causal mask per query), which divides the cache traffic of the context pass by up to QB.  Same chunking, same
// partial layout and the same merge kernel as above.
// grid = (n_blocks, n_head / 4), block = 256.  blocks[b] = (first row, rows in block (<= QB), chunk, -).
template <int DT, int D, int QB>
__global__ __launch_bounds__(256) void attn_prefill_kernel(const void* __restrict__ q, const void* __restrict__ kc,
                                                           const void* __restrict__ vc, const int4* __restrict__ blocks,
                                                           const int* __restrict__ row_slot,
                                                           const int* __restrict__ row_len, int nh, int Smax,
                                                           int maxch, float scale, float* __restrict__ pml,
                                                           float* __restrict__ po) {
  constexpr int EB = (DT == DT_F32) ? 4 : 2;
  constexpr int EPL = 16 / EB;
  constexpr int LPR = D / EPL;
  constexpr int RPW = 64 / LPR;
  constexpr int U = 2;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int4 bk = blocks[blockIdx.x];
  const int first = bk.x, nr = bk.y, ch = bk.z;
  const int hd = blockIdx.y * 4 + wave;
  const int slot = row_slot[first];
  const int len0 = row_len[first];                          // rows are consecutive positions: len_i = len0 + i
  const int j0 = ch * kAttnChunk, j1 = min(len0 + nr - 1, j0 + kAttnChunk);
  const int grp = lane / LPR, li = lane % LPR;

  float qf[QB][EPL];
#pragma unroll
  for (int i = 0; i < QB; ++i) {
    const int r = first + min(i, nr - 1);
    const u32x4_t qr = *(const u32x4_t*)((const char*)q + ((size_t)(r * nh + hd) * D + li * EPL) * EB);
    unpack16<DT>(qr, qf[i]);
#pragma unroll
    for (int e = 0; e < EPL; ++e) qf[i][e] *= scale;
  }
  const size_t head_off = ((size_t)slot * nh + hd) * Smax * D * EB + (size_t)li * 16;
  const char* kb = (const char*)kc + head_off;
  const char* vb = (const char*)vc + head_off;

  float m[QB], l[QB], o[QB][EPL];
#pragma unroll
  for (int i = 0; i < QB; ++i) {
    m[i] = -INFINITY;
    l[i] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) o[i][e] = 0.f;
  }
  for (int jb = j0; jb < j1; jb += RPW * U) {
    u32x4_t kr[U], vr[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = min(jb + u * RPW + grp, j1 - 1);
      kr[u] = *(const u32x4_t*)(kb + (size_t)r * D * EB);
      vr[u] = *(const u32x4_t*)(vb + (size_t)r * D * EB);
    }
    float kf[U][EPL], vf[U][EPL];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      unpack16<DT>(kr[u], kf[u]);
      unpack16<DT>(vr[u], vf[u]);
    }
#pragma unroll
    for (int i = 0; i < QB; ++i) {
      float sc[U];
      float tmax = -INFINITY;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float d0 = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) d0 = fmaf(qf[i][e], kf[u][e], d0);
        d0 = group_sum<LPR>(d0);
        sc[u] = (jb + u * RPW + grp < min(len0 + i, j1) && i < nr) ? d0 : -INFINITY;   // causal: key < len_i
        tmax = fmaxf(tmax, sc[u]);
      }
      const float mn = fmaxf(m[i], tmax);
      const float ms = (mn == -INFINITY) ? 0.f : mn;
      const float alpha = __expf(m[i] - ms);
      l[i] *= alpha;
#pragma unroll
      for (int e = 0; e < EPL; ++e) o[i][e] *= alpha;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float p = __expf(sc[u] - ms);
        l[i] += p;
#pragma unroll
        for (int e = 0; e < EPL; ++e) o[i][e] = fmaf(p, vf[u][e], o[i][e]);
      }
      m[i] = mn;
    }
  }
#pragma unroll
  for (int i = 0; i < QB; ++i) {
    float mi = m[i], lv = l[i];
    if constexpr (RPW > 1) {
      float mt = mi;
#pragma unroll
      for (int dlt = LPR; dlt < 64; dlt <<= 1) mt = max_over(mt, dlt);
      const float w = (mi == -INFINITY) ? 0.f : __expf(mi - mt);
      lv *= w;
#pragma unroll
      for (int e = 0; e < EPL; ++e) o[i][e] *= w;
#pragma unroll
      for (int dlt = LPR; dlt < 64; dlt <<= 1) {
        lv = sum_over(lv, dlt);
#pragma unroll
        for (int e = 0; e < EPL; ++e) o[i][e] = sum_over(o[i][e], dlt);
      }
      mi = mt;
    }
    const int r = first + i;
    if (i < nr && ch * kAttnChunk < len0 + i && grp == 0) {       // this chunk holds keys this query may see
      const size_t pi = ((size_t)r * maxch + ch) * nh + hd;
      float* op = po + pi * D + li * EPL;
#pragma unroll
      for (int e = 0; e < EPL; ++e) op[e] = o[i][e];
      if (li == 0) {
        pml[pi * 2] = mi;
        pml[pi * 2 + 1] = lv;
      }
    }
  }
}

// ---------------------------------------------------------------- context passes on the matrix cores
// 16-bit models.  The rows of a pass are consecutive positions of ONE slot; a block serves 64 of them for one
// head, a wave 16, and walks all the keys they may see, 32 at a time, so nothing is left to merge.  K and V of the
// next three steps are on their way to LDS by asynchronous copies (a ring of four steps), shared by the block's waves.
//   scores   S^T[key][query] = K . Q^T   : A = K rows (a lane's 16 bytes are 8 consecutive d of one key; copied in that
//                                          order), B = Q^T (8 consecutive d of one query);
//   softmax  per query = per output column: 8 values in the lane, then the 4 lane groups (2 lane swaps);
//   output   O^T[d][query] += V^T . P^T  : B = P^T is what the lane already holds from S^T (keys 4g..4g+3 of both
//            16-key tiles = its 8 k-slots), A = V^T by transposing LDS reads (ds_read_b64_tr_b16: 16 lanes give the
//            addresses of 4 keys x 16 d and get 4 keys of one d each).  V rows lie in LDS with their 16-byte pieces
//            permuted by key, so that the 16 keys of a read spread over the banks.
// P enters the second product as two 16-bit terms (value + rounding remainder), i.e. with 16 or more significant bits;
// m, l and the accumulators stay fp32.
// What bounds it: the chain of a step (LDS read, product, softmax, LDS read, product) at the few wavefronts a pass offers,
// hence 16 queries per wave: 32 halve the LDS reads per multiplication but also the blocks (943 rows x 32 heads: 75 us
// against 43; key chunks per wave with a merge launch, V through 2-byte LDS reads: 38 + 15).  290 rows x 16 heads: 16.4 us
// and a merge of 5.2 -> 11.9 us.  KP = 2: the block's keys are shared out, step by step, to two sets of waves, whose results are put
// together through LDS at the end; for passes whose blocks do not fill the chip (us, one part -> two, 16 heads of 128: 138 rows 10.6 ->
// 9.8, 287 16.1 -> 13.6, 436 22.8 -> 17.9; 32 heads: 500 rows (256 blocks) 25.5 -> 20.0, 943 (480 blocks) 47.8 -> 47.5; 52 heads, 400
// rows (364 blocks) 24.5 -> 26.2; 4 heads, 15 rows 5.1 -> 5.8; four parts: no faster than two).
template <int DT> __device__ __forceinline__ uint32_t pack2(float a, float b) {
  if constexpr (DT == DT_BF16) return (uint32_t)f32_to_bf16(a) | ((uint32_t)f32_to_bf16(b) << 16);
  else return (uint32_t)f32_to_f16(a) | ((uint32_t)f32_to_f16(b) << 16);
}
// Four V^T operands (8 keys of 16 d each) by transposing reads; a[i]: this lane's LDS address of operand i, the second
// 16 keys lie HI bytes further.  Written out with its own wait: after the builtin's form the compiler waits for every copy
// to LDS in flight.
template <int HI> __device__ __forceinline__ void read_transposed4(const uint32_t (&a)[4], u32x4_t (&v)[4]) {
  uint2 x[4], y[4];
  asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %4, %8 offset:%12\n\t"
               "ds_read_b64_tr_b16 %1, %9\n\tds_read_b64_tr_b16 %5, %9 offset:%12\n\t"
               "ds_read_b64_tr_b16 %2, %10\n\tds_read_b64_tr_b16 %6, %10 offset:%12\n\t"
               "ds_read_b64_tr_b16 %3, %11\n\tds_read_b64_tr_b16 %7, %11 offset:%12\n\t"
               "s_waitcnt lgkmcnt(0)"
               : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(y[0]), "=&v"(y[1]), "=&v"(y[2]), "=&v"(y[3])
               : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "n"(HI)
               : "memory");
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = u32x4_t{x[i].x, x[i].y, y[i].x, y[i].y};
}

// permutation of a V row's 16-byte pieces (pairs stay together): 8 consecutive keys put the same pair in 8 places
template <int D> __device__ __forceinline__ int swizzle(int key) { return D == 128 ? (key & 7) * 2 : ((key >> 1) & 3) * 2; }

template <int DT, int D, int KP>
__global__ __launch_bounds__(256 * KP) __attribute__((amdgpu_waves_per_eu(2))) void attn_context_kernel(
    const uint16_t* __restrict__ q, const char* __restrict__ kc, const char* __restrict__ vc, const int* __restrict__ row_slot,
    const int* __restrict__ row_len, int M, int nh, int Smax, int nrb, float scale, void* __restrict__ out, int mtt) {
  static_assert(DT != DT_F32, "16-bit models only");
  constexpr int KS = D / 32;                // MFMA steps over the head dimension
  constexpr int DTL = D / 16;               // output tiles over the head dimension
  constexpr int SEG = D / 8;                // 16-byte pieces of a row
  constexpr int RING = KP == 1 ? 4 : 3;
  constexpr int F = D / 32;                 // copies per wave and step: 2 * KS fragments of K and as many KiB of V by a part's 4 waves
  __shared__ __attribute__((aligned(1024))) u32x4_t lds[RING][KP][2][32 * SEG];   // [step][part][K fragments | V rows]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 3);
  const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), g = lane >> 4, n = lane & 15;
  // heads go round the XCDs, so that a head's K and V stay in one L2; the blocks with the most keys start first
  const int qq = blockIdx.x >> 3, hd = (qq / nrb) * 8 + (blockIdx.x & 7), rb = nrb - 1 - qq % nrb;
  if (hd >= nh) return;
  const int slot = row_slot[0], len0 = row_len[0];         // row r attends to keys 0 .. len0 + r - 1
  const int first = rb * 64 + wave * 16;                   // the wave's rows
  const int klen = len0 + min(M, (rb + 1) * 64) - 1;   // keys of the block's last row
  const int wlen = first < M ? len0 + min(M, first + 16) - 1 : 0;   // of the wave's last row
  const int T = (klen + 32 * KP - 1) / (32 * KP);
  const size_t head_off = ((size_t)slot * nh + hd) * Smax * D * 2;
  const char *kb = kc + head_off, *vb = vc + head_off;

  auto issue = [&](int t) {                                 // rows past the last key repeat it (masked below)
    u32x4_t(*buf)[32 * SEG] = lds[t % RING][part];
    const int k0 = (t * KP + part) * 32;
#pragma unroll
    for (int j = 0; j < F / 2; ++j) {
      const int f = wave + 4 * j;                           // K fragment: 16 keys x 32 d
      const int key = min(k0 + (f / KS) * 16 + n, klen - 1);
      copy_to_lds(kb, (uint32_t)key * D * 2 + (f % KS) * 64 + g * 16, buf[0] + f * 64);
    }
#pragma unroll
    for (int j = 0; j < F / 2; ++j) {
      const int u = (wave + 4 * j) * 64 + lane, kr = u / SEG;   // V piece: key kr of the step, place u % SEG
      const int seg = (u % SEG) ^ swizzle<D>(kr);
      copy_to_lds(vb, (uint32_t)min(k0 + kr, klen - 1) * D * 2 + seg * 16, buf[1] + (wave + 4 * j) * 64);
    }
  };
  // the 8 bytes of V this lane addresses for the first operand: key 4g + n/4, d 4 * (n % 4); 16 d further is a flip of the
  // piece's bits above bit 0 (the places of a row's pieces are permuted by an exclusive or as well)
  const int vk = 4 * g + (n >> 2);
  const uint32_t vaddr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds[0][part][1] +
                         (uint32_t)((vk * SEG + (((n & 3) >> 1) ^ swizzle<D>(vk))) * 16 + (n & 1) * 8);
  u32x4_t qf[KS];
  const uint16_t* qr = q + ((size_t)min(first + n, M - 1) * nh + hd) * D + g * 8;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qf[ks] = *(const u32x4_t*)(qr + ks * 32);
  f32x4_t oacc[DTL];
  float m = -INFINITY, l = 0.f;
  const int lim = first + n < M ? len0 + first + n : 0;     // causal: key < lim
#pragma unroll
  for (int dt = 0; dt < DTL; ++dt) oacc[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < RING - 1; ++t)
    if (t < T) issue(t);
  for (int t = 0; t < T; ++t) {
    copies_barrier<F * (RING - 2)>(t + RING - 2 >= T);      // step t has landed; every wave is done with step t - 1
    if (t + RING - 1 < T) issue(t + RING - 1);
    const int jb = (t * KP + part) * 32;
    if (jb >= wlen) continue;                               // wave-uniform: none of its rows sees these keys
    const u32x4_t* kl = lds[t % RING][part][0] + lane;
    u32x4_t kf[2][KS];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kf[kt][ks] = kl[(kt * KS + ks) * 64];
    // scores: rows = keys kt*16 + 4g + r, column = query n
    f32x4_t sacc[2];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      sacc[kt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) sacc[kt] = mfma16<DT>(kf[kt][ks], qf[ks], sacc[kt]);
    }
    float sc[8];
    float tmax = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = jb + kt * 16 + 4 * g + r;
        const float v = (key < lim) ? sacc[kt][r] * scale : -INFINITY;
        sc[kt * 4 + r] = v;
        tmax = fmaxf(tmax, v);
      }
    tmax = max_partner<32>(max_partner<16>(tmax));
    const float mn = fmaxf(m, tmax);
    const float ms = (mn == -INFINITY) ? 0.f : mn;
    const float alpha = __expf(m - ms);
    float p[8], ps = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      p[j] = __expf(sc[j] - ms);
      ps += p[j];
    }
    l = l * alpha + ps;                                     // per-lane share; the lane groups are added at the end
    m = mn;
#pragma unroll
    for (int dt = 0; dt < DTL; ++dt) oacc[dt] *= alpha;
    // The probabilities enter the second product as two 16-bit terms, p = hi + lo with hi = p rounded to the model
    // dtype and lo = (p - hi) rounded: 16 significant bits for bf16 (more for fp16), so that this kernel weighs the V
    // rows as accurately as the decode kernel's fp32 probabilities do (one term alone would add a rounding point
    // that the decode path does not have).
    float q_[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) q_[j] = p[j] - rdt<DT>(p[j]);
    const u32x4_t pb = u32x4_t{pack2<DT>(p[0], p[1]), pack2<DT>(p[2], p[3]), pack2<DT>(p[4], p[5]), pack2<DT>(p[6], p[7])};
    const u32x4_t pl = u32x4_t{pack2<DT>(q_[0], q_[1]), pack2<DT>(q_[2], q_[3]), pack2<DT>(q_[4], q_[5]), pack2<DT>(q_[6], q_[7])};
    // output: A = V^T, k-slot j of lane group g <-> key 4g + j (j < 4) or 16 + 4g + (j - 4), as in pb
#pragma unroll
    for (int d4 = 0; d4 < DTL; d4 += 4) {
      uint32_t at[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) at[i] = (vaddr + (t % RING) * (uint32_t)sizeof(lds[0])) ^ ((d4 + i) * 32);
      u32x4_t va[4];
      read_transposed4<16 * D * 2>(at, va);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        oacc[d4 + i] = mfma16<DT>(va[i], pl, oacc[d4 + i]);
        oacc[d4 + i] = mfma16<DT>(va[i], pb, oacc[d4 + i]);
      }
    }
  }
  // The parts' results of a query, put together by the first part's wave in the order of the parts
  if constexpr (KP > 1) {
    f32x4_t* room = (f32x4_t*)&lds[0][0][0][0];              // [part - 1][wave][DTL + 1][lane]
    static_assert(sizeof(lds) >= (size_t)(KP - 1) * 4 * (DTL + 1) * 64 * sizeof(f32x4_t), "hand-over space");
    copies_barrier<0>(true);
    f32x4_t* mine = room + (size_t)((part - 1) * 4 + wave) * (DTL + 1) * 64 + lane;
    if (part > 0) {
#pragma unroll
      for (int dt = 0; dt < DTL; ++dt) mine[dt * 64] = oacc[dt];
      mine[DTL * 64] = f32x4_t{m, l, 0.f, 0.f};
    }
    __syncthreads();
    if (part > 0) return;
    f32x4_t ml[KP];
    ml[0] = f32x4_t{m, l, 0.f, 0.f};
    float mt = m;
#pragma unroll
    for (int p = 1; p < KP; ++p) {
      ml[p] = room[(size_t)((p - 1) * 4 + wave) * (DTL + 1) * 64 + DTL * 64 + lane];
      mt = fmaxf(mt, ml[p][0]);
    }
    const float ms = mt == -INFINITY ? 0.f : mt;             // rows past the last: nothing is stored
    const float w0 = __expf(m - ms);
    l *= w0;
#pragma unroll
    for (int dt = 0; dt < DTL; ++dt) oacc[dt] *= w0;
#pragma unroll
    for (int p = 1; p < KP; ++p) {
      const float w = __expf(ml[p][0] - ms);                 // a part without a key for this row: 0
      l += w * ml[p][1];
#pragma unroll
      for (int dt = 0; dt < DTL; ++dt) oacc[dt] += w * room[(size_t)((p - 1) * 4 + wave) * (DTL + 1) * 64 + dt * 64 + lane];
    }
  }
  // lane (n, g) owns O[query n][d = dt*16 + 4g .. +3]
  l = sum_partner<32>(sum_partner<16>(l));
  if (first + n < M) {
#pragma unroll
    for (int dt = 0; dt < DTL; ++dt) stv4<DT>(out, xrow_index(first + n, hd * D + dt * 16 + 4 * g, nh * D, mtt), oacc[dt] / l);
  }
}

// ---------------------------------------------------------------- host side

constexpr int kGridY = 65535;      // the most blocks of a grid in y

// Blocks of one wave, or of four.  A compute unit streams about 40 bytes per ns whatever it holds, so while waves are few each should have a
// unit to itself, and a last round of blocks of four that is mostly empty leaves units idle beside full ones (waves 1024 -> 1056, 12 rows x 32
// heads: 19 -> 30 us).  Where many rows of many chunks fill the units anyway, blocks of four lead (whether by their size or by the order of their
// grid was not separated).  Graphs of calls, cold caches, rows of 1 to the stated positions, bf16, d = 128 unless stated, us, four -> one:
//   * one chunk per row, always: 9 x 16 heads (fp32) of 200 16.4 -> 12.7, 6 x 32 10.9 -> 9.7, 28 x 32 (fp32) of 256 22.8 -> 17.5, 63 x 16 (fp32, d = 64)
//     of 120 9.1 -> 8.2, 256 x 32 of 200 72.5 -> 70.1; level at 64 x 32 of 30 (fp32, d = 64 7.5 -> 8.0);
//   * a last round (of 256 x 4 waves) that leaves the launch 1.3 times the places it needs, up to 787 waves for one: 9 x 32 of 700 (448 waves) 17.3 -> 15.9,
//     6 x 52 of 700 (624) 17.2 -> 15.9, 23 x 16 of 1900 with short rows (592) 19.6 -> 18.5, 9 x 52 of 4096 (fp32, d = 64, 1248) 36.0 -> 31.5; loses most
//     just inside, 3 x 52 of 1300 (fp32, d = 64, 780) 21.9 -> 23.9; fuller ones 9 x 32 of 1000 (800) 19.6 -> 20.2, 3 x 52 of 4096 (988) 30.5 -> 32.1;
//   * more than one round and up to eight chunks, or rows of 512 bytes: 12 x 32 of 1000 (1056) 30.4 -> 25.8, 20 x 32 of 1900 (3424) 71.4 -> 68.9, 16 x 32
//     (fp32) of 1000 54.8 -> 44.8, 100 x 32 (fp32), one of 6000 among 300, 161 -> 149; 6 x 52 of 1900 (1820) 38.5 -> 40.5.  With more chunks of shorter
//     rows 16 x 32 (d = 64) of 8192 (8512) 100 -> 111, one of 8192 among 2000 51.1 -> 65.8, 30 x 52 (d = 64) of 8192 312 -> 339, 9 x 32 of 4096 68.0 -> 73.4.
static bool wave_blocks(int row_bytes, const AttnWork& w, int M, int nh) {
  if (w.chunk_grid || w.n_items > kGridY) return false;
  const long waves = (long)w.n_items * nh, places = (waves + 1023) / 1024 * 1024;
  return w.n_items == M || places * 10 >= waves * 13 || (waves > 1024 && (w.most <= 8 || row_bytes >= 512));
}
// Whether a block takes a whole (row, head), which saves the merge launch and the partial results but ties a row's chunks to one compute unit
// and holds the wave slots of the longest row.  us, two launches (the better of the two block shapes) -> one, bf16, d = 128 unless stated:
//   * up to two chunks, always: 9 rows x 32 heads of up to 300 13.7 -> 11.4, 32 x 32 19.5 -> 18.2, 101 x 32 46.1 -> 45.6, 256 x 32 110 -> 104; 557 shapes,
//     even and uneven, 0.86 of the time in the mean, 1.01 at most;
//   * up to 256 blocks and three chunks (four of short rows, d = 64): 6 x 32 of 700 14.4 -> 13.4, 16 x 16 of 800 15.5 -> 14.1, d = 64 9 x 12 of 1000
//     10.1 -> 9.6; four chunks 6 x 32 of 1000 15.3 -> 16.1, eight 23 -> 27.3; more blocks, three chunks: 9 x 32 of 700 16.1 -> 20.2;
//     131 shapes of three chunks 0.88, at most 0.99, 32 of four chunks of short rows 0.89, at most 0.93, but 79 of four chunks of longer rows 1.03, up to 1.21;
//   * from 1024 blocks, where the units are full anyway: 32 x 32 of 1000 50.6 -> 49.9, of 4000 195 -> 189, 64 x 32 of 1000 93.6 -> 86.5, of 4000
//     372 -> 331, 80 x 32 of 2000 219 -> 207, 64 x 16 of 2000 91.0 -> 85.9, 40 x 52 of 2000 185 -> 174, 101 x 12 (d = 64) of 2000 55.3 -> 52.0, 101 x 16
//     (fp32, d = 64) of 2000 136 -> 130; below, rows decide: 24 x 32 of 2000 69.8 -> 67.7, of 700 29.1 -> 29.3, 16 x 52 of 2000 73.5 -> 76.7
//     (938 shapes of 257 to 1023 blocks 1.00, up to 1.79).
//     From 1024 on the longest row has to end with the rest: at most a unit's share of all chunks.  One row of 4096 among rows of up to
//     100, 5.9 chunks a unit, 64 x 16 28.5 -> 46.1, (fp32) 70 x 16 41.1 -> 83.7, 64 x 32 (11.8) 44.8 -> 52.9; of up to 256, 40 x 32 (8.8) 43.8 -> 52.7;
//     128 x 16, four of 4096 among 400 (15.0) 69.4 -> 75.3.  At the share and above: 40 x 32, one of 2048 among 700 (11.1 for 8) 53.9 -> 51.3, 64 x 32
//     of 4096 (20.8 for 16) 102 -> 94, 128 x 32, four of 2048 among 400 (26) 103 -> 96; 250 x 32 (d = 64), one of 4096 among 100 (35) 41.7 -> 33.0.
//     Of 300 length sets, uneven ones above all, the share loses most at 141 x 24, one of 3586 among 73 (15.8 for 15), 40.7 -> 45.6, and 128 x 16, one
//     of 4096 among 700 (16.5 for 16), 77.9 -> 82.0, and forgoes most at 40 x 32, four of 4096 among 400 (13.5), 71.6 -> 65.1.
// With a row's heads apart in the grid (all of a row's blocks on one XCD where the rows are a multiple of eight) 128 x 32 of 2000 took 353 instead of 322.
bool attention_by_rows(int dtype, int d, const AttnWork& w, int M, int nh) {
  const long blocks = (long)M * nh;
  if (w.n_items == M || w.merge_last || w.most > kRowChunks || M > kGridY) return false;
  if (w.most <= 2 || (w.most <= (d * (dtype == DT_F32 ? 4 : 2) <= 128 ? 4 : 3) && blocks <= 256)) return true;
  return blocks >= 1024 && (long)w.n_items * nh >= (long)w.most * 256;
}
bool attention_merges(const AttnWork& w, int M) { return w.merge_last || (w.n_items != M && !w.by_rows); }
// By steps of 64 positions: one pass to count, one to place.
void longest_first(const int* len, int M, int* place) {
  constexpr int kSteps = kRowChunks * kAttnChunk / 64 + 1;
  auto step = [](int n) { return kSteps - 1 - std::min(kSteps - 1, n / 64); };
  int at[kSteps + 1] = {};
  for (int i = 0; i < M; ++i) ++at[step(len[i]) + 1];
  for (int k = 0; k < kSteps; ++k) at[k + 1] += at[k];
  for (int i = 0; i < M; ++i) place[i] = at[step(len[i])]++;
}
template <int DT, int D, class Src>
static void launch_attn(const void* q, const void* kc, const void* vc, const AttnWork& w, const Src& src, int M, int nh, int Smax,
                        void* out, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  const float scale = 1.0f / sqrtf((float)D);
  const bool one_chunk = w.n_items == M && !w.merge_last, single = wave_blocks(D * (DT == DT_F32 ? 4 : 2), w, M, nh);
  launch_timed(one_chunk ? attn_partial_kernel<DT, D, 4, true, Src> : attn_partial_kernel<DT, D, 4, false, Src>,
               single ? dim3(nh, w.n_items) : dim3(w.n_items, nh / 4), dim3(single ? 64 : 256), st, ev0, ev1, q, kc, vc, src, nh,
               single ? 1 : 0, Smax, w.maxch, scale, w.pml, w.po, out, w.out_mtt);
  if (one_chunk) return;
  attn_merge_kernel<DT, D, Src><<<dim3(M, (nh * D + 1023) / 1024), 256, 0, st>>>(w.pml, w.po, src, w.maxch, nh, out, w.out_mtt);
}
template <int DT, int D, class Src>
static void launch_rows(const void* q, const void* kc, const void* vc, const AttnWork& w, const Src& src, int M, int nh, int Smax,
                        void* out, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  launch_timed(attn_row_kernel<DT, D, 4, Src>, dim3(nh, M), dim3(64 * std::min(w.most, kRowWaves)), st, ev0, ev1, q, kc, vc, src, nh,
               Smax, 1.0f / sqrtf((float)D), out, w.out_mtt);
}
template <int DT, int D>
static void launch_attn(const void* q, const void* kc, const void* vc, const AttnWork& w, int M, int nh, int Smax, void* out,
                        hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  if (w.by_rows && w.rows) {
    RowOrder o;
    int place[kAttnRows];
    longest_first(w.rows->len, M, place);
    for (int i = 0; i < M; ++i) {
      o.row[place[i]] = i;
      o.r.slot[place[i]] = w.rows->slot[i];
      o.r.len[place[i]] = w.rows->len[i];
    }
    launch_rows<DT, D>(q, kc, vc, w, o, M, nh, Smax, out, st, ev0, ev1);
  } else if (w.by_rows) {
    launch_rows<DT, D>(q, kc, vc, w, ItemList{w.items, w.row_len}, M, nh, Smax, out, st, ev0, ev1);
  } else if (w.rows) {
    launch_attn<DT, D>(q, kc, vc, w, RowList{*w.rows, M}, M, nh, Smax, out, st, ev0, ev1);
  } else {
    launch_attn<DT, D>(q, kc, vc, w, ItemList{w.items, w.row_len}, M, nh, Smax, out, st, ev0, ev1);
  }
}

hipError_t decode_attention(int dtype, int d, const void* q, const void* kc, const void* vc, const AttnWork& w, int M,
                            int nh, int Smax, void* out, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  if (M <= 0 || w.n_items <= 0) return hipSuccess;
  if (d == 128) {
    if (dtype == DT_F32) launch_attn<DT_F32, 128>(q, kc, vc, w, M, nh, Smax, out, st, ev0, ev1);
    else if (dtype == DT_F16) launch_attn<DT_F16, 128>(q, kc, vc, w, M, nh, Smax, out, st, ev0, ev1);
    else launch_attn<DT_BF16, 128>(q, kc, vc, w, M, nh, Smax, out, st, ev0, ev1);
  } else {
    if (dtype == DT_F32) launch_attn<DT_F32, 64>(q, kc, vc, w, M, nh, Smax, out, st, ev0, ev1);
    else if (dtype == DT_F16) launch_attn<DT_F16, 64>(q, kc, vc, w, M, nh, Smax, out, st, ev0, ev1);
    else launch_attn<DT_BF16, 64>(q, kc, vc, w, M, nh, Smax, out, st, ev0, ev1);
  }
  return hipGetLastError();
}

// Two parts of the keys per block while every block gets a compute unit to itself and there are keys to share (see the kernel).
static int context_parts(int M, int blocks) { return M > 64 && blocks <= 256 ? 2 : 1; }
template <int DT, int D>
static void launch_prefill(const void* q, const void* kc, const void* vc, const AttnWork& w, int M, int nh, int Smax,
                           void* out, hipStream_t st) {
  const float scale = 1.0f / sqrtf((float)D);
  if constexpr (DT == DT_F32) {
    attn_prefill_kernel<DT, D, kPrefillQB><<<dim3(w.n_blocks, nh / 4), 256, 0, st>>>(
        q, kc, vc, w.blocks, w.row_slot, w.row_len, nh, Smax, w.maxch, scale, w.pml, w.po);
    attn_merge_kernel<DT, D, ItemList><<<dim3(M, (nh * D + 1023) / 1024), 256, 0, st>>>(w.pml, w.po, ItemList{w.items, w.row_len}, w.maxch,
                                                                                     nh, out, w.out_mtt);
  } else {
    const int nrb = (M + 63) / 64, blocks = (nh + 7) / 8 * 8 * nrb;
    auto launch = [&](auto parts_) {
      constexpr int parts = decltype(parts_)::value;
      attn_context_kernel<DT, D, parts><<<blocks, 256 * parts, 0, st>>>((const uint16_t*)q, (const char*)kc, (const char*)vc, w.row_slot,
                                                                       w.row_len, M, nh, Smax, nrb, scale, out, w.out_mtt);
    };
    if (context_parts(M, nh * nrb) == 2) launch(std::integral_constant<int, 2>{});
    else launch(std::integral_constant<int, 1>{});
  }
}

hipError_t prefill_attention(int dtype, int d, const void* q, const void* kc, const void* vc, const AttnWork& w, int M,
                             int nh, int Smax, void* out, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  if (d == 128) {
    if (dtype == DT_F32) launch_prefill<DT_F32, 128>(q, kc, vc, w, M, nh, Smax, out, st);
    else if (dtype == DT_F16) launch_prefill<DT_F16, 128>(q, kc, vc, w, M, nh, Smax, out, st);
    else launch_prefill<DT_BF16, 128>(q, kc, vc, w, M, nh, Smax, out, st);
  } else {
    if (dtype == DT_F32) launch_prefill<DT_F32, 64>(q, kc, vc, w, M, nh, Smax, out, st);
    else if (dtype == DT_F16) launch_prefill<DT_F16, 64>(q, kc, vc, w, M, nh, Smax, out, st);
    else launch_prefill<DT_BF16, 64>(q, kc, vc, w, M, nh, Smax, out, st);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------- memory shuffle copy (Section V-D)
// One launch moves every listed slot: block b -> (move, segment = (layer, K|V, head), piece of PIECE bytes).
// moves[i] = (src slot, dst slot, bytes per segment = len * d * elem, first block index).
// Sources lie outside the chosen window and destinations are holes inside it, so the two sets are disjoint and
// the copies can run in any order.
// The list is in device memory, or (operation-level calls of up to 64 moves) a kernel argument: no copy and no wait for it.
struct MoveList {
  const int4* moves;
  __device__ int4 at(int i) const { return moves[i]; }
};
struct MoveArgs {
  CompactMoves m;
  __device__ int4 at(int i) const { return m.move[i]; }
};
template <class Src>
__global__ __launch_bounds__(256) void compact_kernel(char* __restrict__ cache, Src moves, int n_moves, int nseg_per_slot, int C, size_t slot_bytes, int piece) {
  // binary search: last move whose first block <= blockIdx.x
  int lo = 0, hi = n_moves - 1;
  const int b = blockIdx.x;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (moves.at(mid).w <= b) lo = mid; else hi = mid - 1;
  }
  const int4 mv = moves.at(lo);
  const int bytes = mv.z;
  const int ppseg = (bytes + piece - 1) / piece;
  const int rel = b - mv.w;
  const int seg = rel / ppseg, pc = rel - seg * ppseg;
  // segment `seg` = (layer*2 + kv) * nh + head; cache is [(layer*2+kv)][C][nh][S][d]
  const int nh = nseg_per_slot;             // heads per (layer,kv) plane, passed by the host
  const int plane = seg / nh, head = seg - plane * nh;
  const size_t base = ((size_t)plane * C) * slot_bytes;
  const size_t head_bytes = slot_bytes / nh;
  const char* src = cache + base + (size_t)mv.x * slot_bytes + (size_t)head * head_bytes + (size_t)pc * piece;
  char* dst = cache + base + (size_t)mv.y * slot_bytes + (size_t)head * head_bytes + (size_t)pc * piece;
  const int n = min(piece, bytes - pc * piece);       // multiple of 16
  for (int off = threadIdx.x * 16; off < n; off += 256 * 16) {
    const u32x4_t v = __builtin_nontemporal_load((const u32x4_t*)(src + off));
    __builtin_nontemporal_store(v, (u32x4_t*)(dst + off));
  }
}

hipError_t compact(void* cache, int C, int nh, size_t slot_bytes, const void* moves_dev, const CompactMoves* moves_host, int n_moves,
                   int total_blocks, int piece, hipStream_t st) {
  if (n_moves <= 0 || total_blocks <= 0) return hipSuccess;
  if (moves_host) compact_kernel<<<total_blocks, 256, 0, st>>>((char*)cache, MoveArgs{*moves_host}, n_moves, nh, C, slot_bytes, piece);
  else compact_kernel<<<total_blocks, 256, 0, st>>>((char*)cache, MoveList{(const int4*)moves_dev}, n_moves, nh, C, slot_bytes, piece);
  return hipGetLastError();
}

}  // namespace flk
