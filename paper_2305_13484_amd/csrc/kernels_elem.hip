// Row-wise kernels of the fused decoder step (Algorithm 2's LayerNorm / GenericActivation calls over
// [buffer + offset, size), plus embedding, rotary + KV append and the greedy choice).
//
// Each consumes the split-K partial sums of the GEMM before it (added in slice order, then bias), so the epilogue of a
// GEMM with K slices lives in the next launch and nothing depends on how many rows are live; where a GEMM finishes the job
// itself (context passes with one slice, fp32 models) the norm finds the residual stream already added to.  All are HBM/L2
// streaming kernels: coalesced 16-byte-per-lane accesses, fixed reduction trees.
#include <algorithm>

#include "flover_dev.h"
#include "flover_kernels.h"

namespace flk {

// Sum of S split-K slices at 4 consecutive elements, added in slice order (s = 0, 1, 2, ...).  Up to 8 slices the
// code is straight-line for the given count -- one scalar jump on S, which is uniform over the grid, then all loads issued
// before the first addition, so a thread pays the memory latency once; beyond that (2048 columns of K = 8192: 13 slices)
// the loads are predicated one by one (straight-line code up to 16: the same time, 466 us against 467 for six layers).
template <int S>
__device__ __forceinline__ f32x4_t psum4_fixed(const float* __restrict__ p, size_t stride) {
  f32x4_t pv[S];
#pragma unroll
  for (int j = 0; j < S; ++j) pv[j] = ld4(p + (size_t)j * stride);
  f32x4_t v = pv[0];
#pragma unroll
  for (int j = 1; j < S; ++j) v += pv[j];
  return v;
}
__device__ __forceinline__ f32x4_t psum4(const float* __restrict__ part, int S, size_t stride, size_t idx) {
  const float* p = part + idx;
  switch (S) {
    case 1: return psum4_fixed<1>(p, stride);
    case 2: return psum4_fixed<2>(p, stride);
    case 3: return psum4_fixed<3>(p, stride);
    case 4: return psum4_fixed<4>(p, stride);
    case 5: return psum4_fixed<5>(p, stride);
    case 6: return psum4_fixed<6>(p, stride);
    case 7: return psum4_fixed<7>(p, stride);
    case 8: return psum4_fixed<8>(p, stride);
    default: break;
  }
  f32x4_t pv[16];
#pragma unroll
  for (int j = 0; j < 16; ++j)
    if (j < S) pv[j] = ld4(p + (size_t)j * stride);
  f32x4_t v = pv[0];
#pragma unroll
  for (int j = 1; j < 16; ++j)
    if (j < S) v += pv[j];
  for (int s = 16; s < S; ++s) v += ld4(p + (size_t)s * stride);
  return v;
}
// ---------------------------------------------------------------- residual add + norm
// x[m] += sum_s part[s][m] + bias   (skipped when part == nullptr), then
// h[m] = LayerNorm(x[m]) * g + b   (RMS == 0)   or   x[m] / rms(x[m]) * g   (RMS == 1), rounded to dtype.
// grid = M; H % 4 == 0, H <= 8192; part rows have length ldp.  All slice loads of a pass are issued before the first
// addition.  A row is worked by 16 virtual waves of 64 lanes x 4 consecutive elements (2 passes cover H); a block has
// 16 / VW real waves of VW virtual ones each, with the virtual waves' sums kept apart and added in the same order, so the
// result does not depend on VW.  VW = 1 (1024 threads) for an iteration's few rows, where the latency of one row counts
// (256 threads: 3 % of the 7B stream's tokens/s less; 290 rows of 2048 columns 6.8 us against 7.8); VW = 4 above 512 rows,
// where the rows in flight count: a compute unit holds eight of them instead of two, and the blocks fit beside another
// stream's GEMM (940 rows of 4096 beside a second context pass: 43.7 us -> 33.8).
// update(i): the row's new elements i..i+3, stored to x where they changed.
template <int DT, int RMS, int VW, class Update>
__device__ __forceinline__ void norm_row(Update update, int m, const void* __restrict__ g, const void* __restrict__ b,
                                         void* __restrict__ h, int H, float eps, int mtt) {
  __shared__ float red[2][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int PER = 2;
  auto column = [&](int w, int c) { return ((wave * VW + w) * 64 + lane + c * 1024) * 4; };
  // sum of one value per virtual wave and lane over the row, in an order that is the same for every VW
  auto row_sum = [&](float (&v)[VW], float* r) {
#pragma unroll
    for (int w = 0; w < VW; ++w) v[w] = group_sum<64>(v[w]);
    if (lane == 0) {
#pragma unroll
      for (int w = 0; w < VW; ++w) r[wave * VW + w] = v[w];
    }
    __syncthreads();
    float t = r[0];
    const int n = blockDim.x / 64 * VW;
#pragma unroll
    for (int i = 1; i < 16; ++i)
      if (i < n) t += r[i];
    return t;
  };
  f32x4_t v[VW][PER], gv[VW][PER], bv[VW][PER];
  float sum[VW];
#pragma unroll
  for (int w = 0; w < VW; ++w) {
    sum[w] = 0.f;
#pragma unroll
    for (int c = 0; c < PER; ++c) {
      const int i = column(w, c);
      v[w][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      gv[w][c] = v[w][c];
      bv[w][c] = v[w][c];
      if (i < H) {
        gv[w][c] = ldv4<DT>(g, i);                     // issued early: needed only after the reductions
        if (!RMS) bv[w][c] = ldv4<DT>(b, i);
        const f32x4_t t = update(i);
        v[w][c] = t;
        sum[w] += RMS ? square_sum4(t) : sum4(t);
      }
    }
  }
  const float total = row_sum(sum, red[0]);
  float mean = 0.f, inv;
  if (RMS) {
    inv = 1.0f / sqrtf(total / (float)H + eps);
  } else {
    mean = total / (float)H;
    float sq[VW];
#pragma unroll
    for (int w = 0; w < VW; ++w) {
      sq[w] = 0.f;
#pragma unroll
      for (int c = 0; c < PER; ++c)
        if (column(w, c) < H) sq[w] += square_sum4(v[w][c] - mean);
    }
    inv = 1.0f / sqrtf(row_sum(sq, red[1]) / (float)H + eps);
  }
#pragma unroll
  for (int w = 0; w < VW; ++w)
#pragma unroll
    for (int c = 0; c < PER; ++c) {
      const int i = column(w, c);
      if (i < H) stv4<DT>(h, xrow_index(m, i, H, mtt), norm_value<RMS != 0>(v[w][c], mean, inv, gv[w][c], bv[w][c]));
    }
}

template <int DT, int RMS, int VW>
__global__ __launch_bounds__(1024 / VW) void add_norm_kernel(float* __restrict__ x, const float* __restrict__ part, int S,
                                                             size_t stride, int ldp, const void* __restrict__ bias,
                                                             const void* __restrict__ g, const void* __restrict__ b,
                                                             void* __restrict__ h, int H, float eps, int mtt) {
  const int m = blockIdx.x;
  norm_row<DT, RMS, VW>([&](int i) {
    f32x4_t t = *(const f32x4_t*)(x + (size_t)m * H + i);
    if (part) {
      f32x4_t a = psum4(part, S, stride, (size_t)m * ldp + i);
      if (bias) a += ldv4<DT>(bias, i);
      t += a;
      *(f32x4_t*)(x + (size_t)m * H + i) = t;
    }
    return t;
  }, m, g, b, h, H, eps, mtt);
}

// ---------------------------------------------------------------- embedding + first norm
// x[m][i] = wte[tok[m]][i] (+ wpe[pos[m]][i]), then the norm above of that row: one launch for both (the embedding alone
// took 4 to 5 us of every pass, nearly all of it the launch and one round trip to memory).
// The row comes from the host's pinned memory (one 16-byte read per block, in place of a copy to the device ahead of the pass: an
// engine of its own that the stream waits for), and what later kernels read of it is written out here.
// tok < 0 feeds the token the previous iteration chose for its row -1 - tok: the best of that row's `parts` choices.
template <int DT, int RMS, int VW>
__global__ __launch_bounds__(1024 / VW) void embed_norm_kernel(const void* __restrict__ wte, const void* __restrict__ wpe,
                                                               const RowIn* __restrict__ rows, RowOut out,
                                                               const Choice* __restrict__ prev, int parts, float* __restrict__ x,
                                                               const void* __restrict__ g, const void* __restrict__ b,
                                                               void* __restrict__ h, int H, float eps, int mtt) {
  __shared__ RowIn row;
  const int m = blockIdx.x, tid = threadIdx.x;
  if (tid == 0) {
    RowIn r = rows[m];
    out.pos[m] = r.pos;
    out.slot[m] = r.slot;
    out.len[m] = r.pos + 1;
    if (r.tok < 0) r.tok = best_choice(prev + (size_t)(-1 - r.tok) * parts, parts);
    row = r;
  }
  __syncthreads();
  const int tk = row.tok, pos = row.pos, first = row.first;
  if (first >= 0) {
    const int nr = out.block_rows > 0 ? min(out.block_rows, (int)gridDim.x - m) : 1, len = pos + nr;
    const int chunks = out.block_rows == kEntryPerRow ? 1 : (len + kAttnChunk - 1) / kAttnChunk;
    for (int c = tid; c < chunks; c += blockDim.x)
      out.list[first + c] = out.block_rows > 0 ? make_int4(m, nr, c, 0) : make_int4(m, c, row.slot, len);
  }
  const size_t t = (size_t)tk * H, p = wpe ? (size_t)pos * H : 0;
  norm_row<DT, RMS, VW>([&](int i) {
    f32x4_t v = ldv4<DT>(wte, t + i);
    if (wpe) v += ldv4<DT>(wpe, p + i);
    *(f32x4_t*)(x + (size_t)m * H + i) = v;
    return v;
  }, m, g, b, h, H, eps, mtt);
}

// ---------------------------------------------------------------- QKV epilogue: bias, rotary, KV append
// part: [S][M][ldp] rows (q | k | v).  For row m (slot, pos) and head hd: q -> qout[m][hd][:] (dtype),
// k, v -> cache[slot][hd][pos][:] (dtype).  Rotary (LLaMA): pairs (i, i + d/2), cos/sin from a table [max_seq][d/2][2].
// grid = (M, 3): blockIdx.y picks q, k or v; block = n_head * d / 8: thread (hd, j) owns elements 4j..4j+3 and their
// partners 4j + d/2 .. of its vector.
template <int DT>
__global__ void qkv_post_kernel(const float* __restrict__ part, int S, size_t stride, int ldp,
                                const void* __restrict__ bias, const float* __restrict__ rope_cs,
                                const int* __restrict__ slot, const int* __restrict__ pos, void* __restrict__ qout,
                                void* __restrict__ kcache, void* __restrict__ vcache, int H, int nh, int d, int Smax) {
  const int m = blockIdx.x, which = blockIdx.y, half = d >> 1, tph = d >> 3;
  const int hd = threadIdx.x / tph, i = (threadIdx.x - hd * tph) * 4;
  const int c0 = which * H + hd * d + i, c1 = c0 + half;
  const float* p0 = part + (size_t)m * ldp + c0;
  const float* p1 = part + (size_t)m * ldp + c1;
  // Load order: the row's position first, then every split-K slice (their addresses need nothing else), and only then
  // the rotary table row, whose address waits for the position -- so that wait overlaps the slices' flight.
  const int p = pos[m];
  const bool rot = rope_cs && which < 2;
  f32x4_t a0 = ld4(p0), a1 = ld4(p1);
  f32x4_t u0[8], u1[8];
#pragma unroll
  for (int j = 0; j < 8; ++j)                             // slices 1..8; S is uniform over the grid: scalar branches
    if (1 + j < S) {
      u0[j] = ld4(p0 + (size_t)(1 + j) * stride);
      u1[j] = ld4(p1 + (size_t)(1 + j) * stride);
    }
  __builtin_amdgcn_sched_barrier(0);
  f32x4_t t0 = {1.f, 0.f, 1.f, 0.f}, t1 = t0;          // (cos, sin) of 4 consecutive pairs
  if (rot) {
    const float* t = rope_cs + ((size_t)p * half + i) * 2;
    t0 = ld4(t);
    t1 = ld4(t + 4);
  }
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (1 + j < S) { a0 += u0[j]; a1 += u1[j]; }
  for (int s0 = 9; s0 < S; s0 += 8) {                     // more than 9 slices: context passes of short prompts only
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const size_t o = (size_t)min(s0 + j, S - 1) * stride;
      u0[j] = ld4(p0 + o);
      u1[j] = ld4(p1 + o);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (s0 + j < S) { a0 += u0[j]; a1 += u1[j]; }
  }
  if (bias) { a0 += ldv4<DT>(bias, c0); a1 += ldv4<DT>(bias, c1); }
  if (rot) {
    const f32x4_t cs = {t0[0], t0[2], t1[0], t1[2]}, sn = {t0[1], t0[3], t1[1], t1[3]};
    rope_rotate(a0, a1, cs, sn);
  }
  if (which == 0) {
    stv4<DT>(qout, (size_t)m * H + hd * d + i, a0);
    stv4<DT>(qout, (size_t)m * H + hd * d + i + half, a1);
  } else {
    void* cache = which == 1 ? kcache : vcache;
    const size_t kv = (((size_t)slot[m] * nh + hd) * Smax + p) * d;
    stv4<DT>(cache, kv + i, a0);
    stv4<DT>(cache, kv + i + half, a1);
  }
}

// ---------------------------------------------------------------- MLP activation
// GPT:   a[m][j] = gelu_tanh(sum_s part[s][m][j] + b1[j])                            part row length ldp >= F
// LLaMA: a[m][j] = silu(gate) * up, gate = part[..][m][j], up = part[..][m][F + j]   part row length ldp >= 2F
// 4 consecutive j per thread; F % 4 == 0.
template <int DT, int SWIGLU>
__global__ __launch_bounds__(256) void act_kernel(const float* __restrict__ part, int S, size_t stride, int ldp,
                                                  const void* __restrict__ bias, void* __restrict__ a, int F, long total4,
                                                  int mtt, int paired) {
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total4) return;
  const int F4 = F >> 2;
  const long m = idx / F4;
  const int j = (int)(idx - m * F4) * 4;
  f32x4_t o;
  if (SWIGLU) {
    // gate column j and up column j: side by side halves of the row, or (paired) tiles of 16 interleaved
    const size_t gj = paired ? (size_t)(j >> 4) * 32 + (j & 15) : (size_t)j, uj = paired ? gj + 16 : (size_t)F + j;
    const f32x4_t g = psum4(part, S, stride, (size_t)m * ldp + gj);
    const f32x4_t u = psum4(part, S, stride, (size_t)m * ldp + uj);
    o = act_swiglu(g, u);
  } else {
    const f32x4_t t = psum4(part, S, stride, (size_t)m * ldp + j) + ldv4<DT>(bias, j);
    o = act_gelu<DT>(t);
  }
  stv4<DT>(a, xrow_index((int)m, j, F, mtt), o);
}

// ---------------------------------------------------------------- logits + greedy token
// logits[m][j] = sum_s part[s][m][j] (fp32, optionally stored, row length V); choice[m][p] = the largest of part p's columns,
// lowest j on ties.  grid = (M, parts), block = 512; part rows have length ldp (multiple of 4, >= V).  A block per row left
// the launch to one compute unit's latency and store rate (18.4 us at 23 rows x 50257, 13.0 us at 6 rows x 32000); whoever
// needs the token picks the best of the few parts (the host, and the next iteration's embedding).
// VEC: rows of logits are 16-byte aligned; otherwise lanes take single columns side by side.
template <bool VEC>
__global__ __launch_bounds__(512) void argmax_kernel(const float* __restrict__ part, int S, size_t stride, int ldp,
                                                     float* __restrict__ logits, Choice* __restrict__ choice, Choice* __restrict__ choice_host,
                                                     int V, int per) {
  __shared__ float bv[8];
  __shared__ int bi[8];
  const int m = blockIdx.x, first = blockIdx.y * per, last = min(V, first + per);
  const float* row = part + (size_t)m * ldp;
  float best = -INFINITY;
  int arg = kNoToken;
  auto take = [&](float v, int j) {                            // ascending j in a thread: the first maximum stays
    if (v > best) { best = v; arg = j; }
  };
  if constexpr (VEC) {
    for (int j0 = first + threadIdx.x * 4; j0 < last; j0 += 2 * 2048) {
      f32x4_t v[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) v[u] = psum4(part, S, stride, (size_t)m * ldp + min(j0 + u * 2048, ldp - 4));
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int j = j0 + u * 2048;
        if (j >= last) continue;
        if (logits) *(f32x4_t*)(logits + (size_t)m * V + j) = v[u];
#pragma unroll
        for (int e = 0; e < 4; ++e) take(v[u][e], j + e);
      }
    }
  } else {
    for (int j0 = first + threadIdx.x; j0 < last; j0 += 8 * 512) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = row[min(j0 + u * 512, last - 1)];
      for (int s = 1; s < S; ++s)
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] += row[(size_t)s * stride + min(j0 + u * 512, last - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int j = j0 + u * 512;
        if (j >= last) continue;
        if (logits) logits[(size_t)m * V + j] = v[u];
        take(v[u], j);
      }
    }
  }
#pragma unroll
  for (int dlt = 1; dlt < 64; dlt <<= 1) {
    const float ov = __shfl_xor(best, dlt, 64);
    const int oi = __shfl_xor(arg, dlt, 64);
    if (ov > best || (ov == best && oi < arg)) { best = ov; arg = oi; }
  }
  if ((threadIdx.x & 63) == 0) { bv[threadIdx.x >> 6] = best; bi[threadIdx.x >> 6] = arg; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 8; ++w)
      if (bv[w] > best || (bv[w] == best && bi[w] < arg)) { best = bv[w]; arg = bi[w]; }
    const size_t at = (size_t)m * gridDim.y + blockIdx.y;
    choice[at] = Choice{best, arg};
    choice_host[at] = Choice{best, arg};         // 8 bytes over the bus per part instead of a copy behind the iteration
  }
}

// ---------------------------------------------------------------- host launchers

#define FLK_DT_SWITCH(dtype, CALL)                        \
  switch (dtype) {                                        \
    case DT_F32: { constexpr int DT = DT_F32; CALL; } break;  \
    case DT_F16: { constexpr int DT = DT_F16; CALL; } break;  \
    default: { constexpr int DT = DT_BF16; CALL; } break;     \
  }

// Threads of a norm block: a row of fewer than 4096 columns leaves the later waves nothing but the barriers (their sums are zero), and
// without them more rows fit a compute unit (three prompts of 138 / 287 / 436 rows of 2048 columns, six layers: 1676 -> 1658 us; a few
// rows take the same time).
static int norm_threads(int H, int VW) { return VW > 1 ? 1024 / VW : std::min(1024, (H + 255) / 256 * 64); }

hipError_t embed_norm(int dtype, bool rms, const void* wte, const void* wpe, const RowIn* rows, const RowOut& out, const Choice* prev,
                      int parts, float* x, const void* g, const void* b, void* h, int M, int H, float eps, int mtt, hipStream_t st) {
  if (M <= 0) return hipSuccess;
#define FLK_EMBED(RMS, VW) \
  FLK_DT_SWITCH(dtype, (embed_norm_kernel<DT, RMS, VW><<<M, norm_threads(H, VW), 0, st>>>(wte, wpe, rows, out, prev, parts, x, g, b, h, H, eps, mtt)))
  if (M > 512) {         // as for add_norm
    if (rms) FLK_EMBED(1, 4) else FLK_EMBED(0, 4)
  } else {
    if (rms) FLK_EMBED(1, 1) else FLK_EMBED(0, 1)
  }
#undef FLK_EMBED
  return hipGetLastError();
}

hipError_t add_norm(int dtype, bool rms, float* x, const float* part, int S, size_t stride, int ldp, const void* bias,
                    const void* g, const void* b, void* h, int M, int H, float eps, int mtt, hipStream_t st) {
  if (M <= 0) return hipSuccess;
#define FLK_NORM(RMS, VW) \
  FLK_DT_SWITCH(dtype, (add_norm_kernel<DT, RMS, VW><<<M, norm_threads(H, VW), 0, st>>>(x, part, S, stride, ldp, bias, g, b, h, H, eps, mtt)))
  if (M > 512) {         // more rows than 1024-thread blocks fit the chip at once
    if (rms) FLK_NORM(1, 4) else FLK_NORM(0, 4)
  } else {
    if (rms) FLK_NORM(1, 1) else FLK_NORM(0, 1)
  }
#undef FLK_NORM
  return hipGetLastError();
}

hipError_t qkv_post(int dtype, const float* part, int S, size_t stride, int ldp, const void* bias, const float* rope_cs,
                    const int* slot, const int* pos, void* q, void* kcache, void* vcache, int M, int H, int nh, int d,
                    int Smax, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  FLK_DT_SWITCH(dtype, (qkv_post_kernel<DT><<<dim3(M, 3), nh * d / 8, 0, st>>>(part, S, stride, ldp, bias, rope_cs, slot, pos, q,
                                                                           kcache, vcache, H, nh, d, Smax)));
  return hipGetLastError();
}

hipError_t activation(int dtype, bool swiglu, const float* part, int S, size_t stride, int ldp, const void* bias, void* a,
                      int M, int F, int mtt, hipStream_t st, bool paired, hipEvent_t ev1) {
  if (M <= 0) return hipSuccess;
  if (paired && !swiglu) return hipErrorInvalidValue;
  const long total = (long)M * (F / 4);
  const unsigned grid = (unsigned)((total + 255) / 256);
  if (swiglu) {
    FLK_DT_SWITCH(dtype, (launch_timed(act_kernel<DT, 1>, dim3(grid), dim3(256), st, nullptr, ev1, part, S, stride, ldp, bias, a, F,
                                       total, mtt, paired ? 1 : 0)));
  } else {
    FLK_DT_SWITCH(dtype, (act_kernel<DT, 0><<<grid, 256, 0, st>>>(part, S, stride, ldp, bias, a, F, total, mtt, 0)));
  }
  return hipGetLastError();
}

// as many blocks per row as 2048 columns each, at most 8
int argmax_parts(int V) { return std::max(1, std::min(8, (V + 2047) / 2048)); }

hipError_t logits_argmax(const float* part, int S, size_t stride, int ldp, float* logits, Choice* choice, Choice* choice_host, int M, int V,
                         hipStream_t st) {
  if (M <= 0) return hipSuccess;
  const int parts = argmax_parts(V), per = ((V + parts - 1) / parts + 3) / 4 * 4;
  const dim3 grid(M, parts);
  if (V % 4 == 0 && ((uintptr_t)logits & 15) == 0) argmax_kernel<true><<<grid, 512, 0, st>>>(part, S, stride, ldp, logits, choice, choice_host, V, per);
  else argmax_kernel<false><<<grid, 512, 0, st>>>(part, S, stride, ldp, logits, choice, choice_host, V, per);
  return hipGetLastError();
}

}  // namespace flk
