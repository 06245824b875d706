// Host-side launchers of the HIP kernels (internal to the library; the public boundary is include/flover.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace flk {

// ---- weight GEMM
struct GemmPlan {
  int N, K;
  int Npad;   // N rounded up to 64 columns (16-bit dtypes)
  int NT;     // n-tiles (of 16 columns) per wave
  int KB;     // K / 32
  int S;      // split-K slices, a function of (N, K) only
  int kbs;    // k-blocks per slice
  int ldc;    // row length of the partial-sum slices (N rounded up to 4)
  int tile = -1;    // more than 128 rows: which kernel (TILE_*), -1 = left to gemm()
  int paired = 0;   // gate|up of a gated MLP in paired 32-column groups (see gemm_plan_gated)
  int whole = 0;    // in a fused iteration one block takes all of K and finishes the job (see gemm_plan_finished)
};
constexpr int kWholeRows = 128;
// kernels of more than 128 rows, by block shape: TILE_ROWS holds the weights in registers, the others copy both operands
// to LDS (gemm16_rows_kernel, gemm16_tile_kernel)
enum { TILE_ROWS = 0, TILE_128X256 = 1, TILE_128X128 = 2, TILE_64X128 = 3, TILE_64X64 = 4, TILE_KINDS = 5 };
inline int part_ld(int N) { return (N + 3) / 4 * 4; }
GemmPlan gemm_plan(int dtype, int N, int K);
// The same for a matrix whose result a row-wise kernel would only finish (q|k|v, the input of an ungated MLP), which the GEMM does
// itself in a fused iteration, and in a context pass of up to kWholeRows rows, where the shape makes that the shorter way.
GemmPlan gemm_plan_finished(int dtype, int N, int K);
GemmPlan gemm_plan_summed(int dtype, int N, int K);    // gemm_plan for a caller who wants the sum (gemm_sum)
// The norm of the rows ahead of an fp32 contraction, taken in the GEMM's own launch (gemm_norms): x is then the residual stream.
struct NormIn {
  const void *g = nullptr, *b = nullptr;   // [K]; no g: the rows as they are.  b: layer norm only
  bool rms = false;
  float eps = 0.f;
};
bool gemm_norms(int dtype, int M, const GemmPlan& p);
// Where a GEMM that finishes the job leaves its result (the members its kind of epilogue uses).
struct TileOut {
  float* part = nullptr;          // partial sums; or the residual stream [M][ldc] the result is added to
  size_t slice_stride = 0;
  int ldc = 0;
  const void* bias = nullptr;     // [N] dtype, may be null
  void* act = nullptr;            // activation [M][F], fragment order with mtt row tiles or row-major
  int F = 0, mtt = 0;
  const float* rope = nullptr;    // rotary table (null: none), positions and slots of the rows, destinations of q, k, v
  const int *pos = nullptr, *slot = nullptr;
  void *q = nullptr, *kc = nullptr, *vc = nullptr;
  int d = 0, Smax = 0;
  int H = 0, third = 0;           // columns of q, of k and of v; which of them the matrix starts with (1: k|v alone)
  NormIn norm;
};
// gate|up of a gated MLP with F columns each.  paired = 1: group j of the layout holds gate columns 16j..16j+15 then up
// columns 16j..16j+15 (re-tile gate with n_off = 0 and up with n_off = 16, both with tile_step = 2), K is cut in two
// halves (or as gemm_plan_finished does), gemm_gated() serves the fused iterations, and gemm() writes its partial sums in that column order (gate column
// j at (j/16)*32 + j%16, up column j 16 further).  paired = 0 (fp32, or a shape the fused kernels do not take): gemm_plan(2F, K), up after gate.
GemmPlan gemm_plan_gated(int dtype, int F, int K);
size_t gemm_tiled_bytes(int dtype, int N, int K);
// Slicing for a context pass of M rows of one request (a function of the matrix shape and of that request's own row
// count only): same tiling, its own number of K slices, at most max_slices (what the partial-sum buffer holds) and 16.
GemmPlan context_plan(const GemmPlan& p, int dtype, int M, int max_slices);
// Block of the kernel that gemm() takes for M > 128 rows (16-bit dtypes, operands on the 16-byte grid).
void gemm_block(int M, const GemmPlan& p, int* rows, int* columns);
// The contraction and what follows it in one launch: fp32 models always, 16-bit models in a fused iteration whose plan says so (whole)
// and in a context pass whose plan takes K in one slice (gemm_finishes); otherwise the caller goes through gemm() and the row-wise kernel.  gemm_qkv: bias, rotary, q and
// the cache rows (o: bias, rope, pos, slot, q, kc, vc, d, Smax, H, third).  gemm_add: res[M][N] += x . W^T + bias (bias may be null).
// gemm_act: GELU of x . W^T + bias, or SwiGLU (16-bit: paired layout; fp32: up after gate).  x is read and the activation written
// in the layout xmtt says.
bool gemm_finishes(int dtype, const GemmPlan& p, int M);
hipError_t gemm_qkv(int dtype, const void* x, const void* w_tiled, int M, const GemmPlan& p, const TileOut& o, int xmtt, hipStream_t st,
                    hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
hipError_t gemm_add(int dtype, const void* x, const void* w_tiled, int M, const GemmPlan& p, float* res, const void* bias, int xmtt,
                    hipStream_t st, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
hipError_t gemm_act(int dtype, bool swiglu, const void* x, const void* w_tiled, int M, const GemmPlan& p, void* act, const void* bias, int xmtt,
                    hipStream_t st, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr, const NormIn& norm = NormIn());
// Re-tile W [N][K] into `tiled` starting at output column n_off (multiple of 16) of a possibly larger matrix whose
// plan uses NT n-tiles per column group.
// Tile t of W lands at tile position n_off/16 + t * tile_step of the layout.
hipError_t retile(int dtype, const void* W, int N, int K, void* tiled, int n_off, int NT, hipStream_t st,
                  int tile_step = 1);
hipError_t zero_fill(void* p, size_t bytes, hipStream_t st);
// part[s][m][p.ldc] (slice stride in floats) = x[M][K] . W^T over slice s of K.
// xmtt == 0: x is row-major [M][K]; xmtt = ceil(M/16) (16-bit dtypes only): x is in fragment order
// (tiles of 16 rows x 32 k, [k-block][row tile], see xrow_index) and the buffer has room for M
// rounded up to 16, 32, 64, 128 or a multiple of 256 rows (row tiles past the last may be read).
// ev0 / ev1 (optional, here and below): take the start / end time stamps of the call's first / last dispatch.
hipError_t gemm(int dtype, const void* x, const void* w_tiled, int M, const GemmPlan& p, float* part,
                size_t slice_stride, int xmtt, hipStream_t st, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr,
                const NormIn& norm = NormIn());
// y[M][ldy] = x . W^T, rows row-major and y at any float, where one launch leaves the whole sum (gemm_adds_up): one slice, or a
// gemm_plan_summed that says so; the bits of gemm()'s slices added in order.
bool gemm_adds_up(int dtype, const GemmPlan& p, int M, const void* x);
hipError_t gemm_sum(int dtype, const void* x, const void* w_tiled, int M, const GemmPlan& p, float* y, int ldy, hipStream_t st);
// act[M][F] = silu(x . Wgate^T) * (x . Wup^T) rounded to the model dtype, for a paired plan (16-bit dtypes); x and act
// are both row-major (xmtt == 0) or both in fragment order with xmtt row tiles per k-block; reads the rows gemm() reads.
// part / slice_stride as for gemm(): used above gated_fused_rows(p) rows, where the contraction and the activation are
// two launches (same result, bit for bit).
// Groups of 32 columns that a block of gemm_gated() takes: as few as leave one block per compute unit, two at least; every block stages
// all rows, so narrower blocks in a second round lose (11008 x 4096, 688 groups, us at 6 / 40 / 101 rows: four groups, 172 blocks, 29.9 / 34.7 / 48.1,
// three, 230, 29.0 / 31.8 / 43.0, two, 344, 37.0 / 43.8 / 56.8).  Call included, four -> now: 6400 x 4096 (two) at 100 rows 55 -> 47, 17920 x 6656 (five;
// eight before) at 10 / 50 rows 98 / 107 -> 88 / 92.  Beyond five groups per unit: eight, whose sixteen waves leave registers for 64 rows.
inline int gated_groups(const GemmPlan& p) {
  const int per_unit = (p.N / 2 / 16 + 255) / 256;
  return per_unit <= 2 ? 2 : per_unit <= 5 ? per_unit : 8;
}
// rows up to which gemm_gated() is one launch for this plan, and up to which a caller of the operation may come without room for its two
// halves (F > 16384 took two launches above 64 rows once; the size that callers are told stays)
inline int gated_fused_rows(const GemmPlan& p) { return p.whole ? kWholeRows : gated_groups(p) > 5 ? 64 : 128; }
inline int gated_roomless_rows(const GemmPlan& p) { return p.whole ? kWholeRows : p.N / 2 > 16384 ? 64 : 128; }
// A whole plan is one launch at any row count (see the definition for row-major rows); part then is scratch of `room` bytes.
hipError_t gemm_gated(int dtype, const void* x, const void* w_tiled, int M, const GemmPlan& p, void* act, float* part,
                      size_t slice_stride, int xmtt, hipStream_t st, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr, size_t room = 0);

// ---- row-wise kernels
// A row's greedy choice is left in parts: the best logit of each part of the vocabulary and its column (kNoToken: none, a part
// of NaNs); best_choice gives the token, the lowest column on ties, 0 when there is none.
constexpr int kNoToken = 0x7fffffff;
struct Choice {
  float value;
  int token;
};
__host__ __device__ inline int best_choice(const Choice* c, int parts) {
  Choice b = c[0];
  for (int p = 1; p < parts; ++p)
    if (c[p].value > b.value || (c[p].value == b.value && c[p].token < b.token)) b = c[p];
  return b.token == kNoToken ? 0 : b.token;
}
int argmax_parts(int V);
// A pass's rows as the host leaves them in pinned memory.  The first kernel of a pass reads them there and lays out on the device
// what the others want.
struct alignas(16) RowIn {
  int32_t tok, pos, slot;
  int32_t first;           // number of the row's first entry in `list`, -1: none
};
struct RowOut {            // device memory
  int *pos, *slot, *len;   // [rows]; len = pos + 1, the rows of cache attended to
  int4* list;              // one entry per chunk of kAttnChunk positions: (row, chunk, slot, len), or where block_rows > 0 (row, rows
                           // of the block, chunk, -) for each block of consecutive positions, entered by its first row, or with
                           // kEntryPerRow (row, 0, slot, len)
  int block_rows;
};
constexpr int kEntryPerRow = -1;
// x = embedding of the rows (wpe: learned positions, may be null), h = the norm of it.  tok < 0: the token is the best of
// the previous iteration's choices for its row -1 - tok.
hipError_t embed_norm(int dtype, bool rms, const void* wte, const void* wpe, const RowIn* rows, const RowOut& out, const Choice* prev,
                      int parts, float* x, const void* g, const void* b, void* h, int M, int H, float eps, int mtt, hipStream_t st);
// `part` is the preceding GEMM's split-K output: S slices, `stride` floats apart, rows of `ldp` floats (ldp % 4 == 0).
// h (and the outputs of activation and of the attention calls below) feed a GEMM: with mtt = ceil(M/16) they are
// written in fragment order (16-bit dtypes; see gemm), with mtt == 0 row-major.
hipError_t add_norm(int dtype, bool rms, float* x, const float* part, int S, size_t stride, int ldp, const void* bias,
                    const void* g, const void* b, void* h, int M, int H, float eps, int mtt, hipStream_t st);
hipError_t qkv_post(int dtype, const float* part, int S, size_t stride, int ldp, const void* bias, const float* rope_cs,
                    const int* slot, const int* pos, void* q, void* kcache, void* vcache, int M, int H, int nh, int d,
                    int Smax, hipStream_t st);
// paired: gate and up columns of `part` interleaved in tiles of 16 (see gemm_plan_gated); gated activation only.
hipError_t activation(int dtype, bool swiglu, const float* part, int S, size_t stride, int ldp, const void* bias, void* a,
                      int M, int F, int mtt, hipStream_t st, bool paired = false, hipEvent_t ev1 = nullptr);
// choice: device memory, for the next iteration; choice_host: the same in pinned memory, for the host.
hipError_t logits_argmax(const float* part, int S, size_t stride, int ldp, float* logits, Choice* choice, Choice* choice_host, int M, int V,
                         hipStream_t st);

// ---- ragged decode attention
constexpr int kAttnChunk = 256;   // most positions of a wave task; fixed, so chunking depends on a request's own length only
constexpr int kAttnRows = 256;
struct alignas(16) AttnRows {   // row descriptors of an operation-level call, passed to the kernels by value; no rows: length 0
  int32_t slot[kAttnRows], len[kAttnRows];
};
struct AttnWork {          // device pointers unless stated
  const int4* items;       // [n_items] (row, chunk, slot of the row, cache rows of the row); by_rows: [M] (row, 0, slot, cache rows)
  const int* row_slot;     // [M]
  const int* row_len;      // [M] rows of cache attended to (>= 1)
  float* pml;              // [M][maxch][nh][2]: (m, l) of chunk ch of row r at ((r * maxch + ch) * nh + head)
  float* po;               // [M][maxch][nh][d]
  int n_items;
  int maxch;               // chunk slots per row in pml / po: at least ceil(longest row / kAttnChunk)
  int most;                // chunks of the longest row
  const int4* blocks = nullptr;   // pre-processing passes of fp32 models: (first row, rows <= kPrefillQB, chunk, -)
  int n_blocks = 0;
  const AttnRows* rows = nullptr;   // [host] set: the rows' descriptors (at most kAttnRows rows), instead of items and row_len
  bool by_rows = false;           // a block takes a whole (row, head): what attention_by_rows() says of the rest of this struct
  bool chunk_grid = false;        // blocks of four heads of a chunk, and the merge a launch of its own, whatever is shorter
  bool merge_last = false;        // the output shares memory with q or the caches: written by a launch of its own
  int out_mtt = 0;                // layout of the attention output: 0 row-major, else fragment order (see add_norm)
};
constexpr int kPrefillQB = 8;     // query rows one wave serves in a pre-processing pass of an fp32 model (an entry of blocks)
// ev0 / ev1 (optional) take the start / end time stamps of the streaming kernel's dispatch (the merge kernel follows).
hipError_t decode_attention(int dtype, int d, const void* q, const void* kc, const void* vc, const AttnWork& w, int M,
                            int nh, int Smax, void* out, hipStream_t st, hipEvent_t ev0 = nullptr,
                            hipEvent_t ev1 = nullptr);

// Whether a block should take a whole (row, head) with all its chunks; then place[i] of longest_first() is where row i goes in `items`.
bool attention_by_rows(int dtype, int d, const AttnWork& w, int M, int nh);
void longest_first(const int* len, int M, int* place);
// Whether decode_attention() launches a merge behind the streaming kernel.
bool attention_merges(const AttnWork& w, int M);

// Attention of a pre-processing pass: all M rows are consecutive positions of one slot (fp32: as listed in w.blocks, through
// the partial results; 16-bit: w.items, blocks, pml and po are not used).
hipError_t prefill_attention(int dtype, int d, const void* q, const void* kc, const void* vc, const AttnWork& w, int M,
                             int nh, int Smax, void* out, hipStream_t st);

// ---- memory shuffle copy
constexpr int kCompactPiece = 16384;   // bytes per block
struct CompactMoves {                  // a short list passed to the kernel by value
  static constexpr int kMost = 64;
  int4 move[kMost];
};
// moves (source slot, destination slot, bytes per segment, first block) from moves_host when set, else from moves_dev
hipError_t compact(void* cache, int C, int nh, size_t slot_bytes, const void* moves_dev, const CompactMoves* moves_host, int n_moves,
                   int total_blocks, int piece, hipStream_t st);

}  // namespace flk
