// Internal launcher interface between the stage runtime and the HIP kernels (gfx950).
// Every launcher only enqueues on `st`; shapes are validated by the runtime before.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace ls {

enum : uint32_t { F32 = 0, BF16 = 1 };

// printf-style setter of the thread-local message behind ls_last_error()
void set_last_error(const char* fmt, ...);

// One-shot request to time the next kernel launch that goes through launch_kernel() on this
// thread: the HIP runtime stamps `start` / `stop` with that kernel's own begin and end (no
// launch gap inside the span, unlike a pair of events recorded around the launch).
struct LaunchTiming {
  hipEvent_t start = nullptr, stop = nullptr;
  bool used = false;
};
LaunchTiming& launch_timing();

// dst[0..n) = src[0..n) (host), by value in the kernels' arguments.
void launch_write_int32(int32_t* dst, const int32_t* src, int n, hipStream_t st);

// What a GEMM does with its fp32 accumulators.
enum Epilogue : int {
  EPI_STORE = 0,   // out[M,N] in dtype
  EPI_RESID = 1,   // resid[M,N] (fp32) += acc
  EPI_SWIGLU = 2,  // W is [2N,K] (gate rows then up rows); out[M,N] = silu(gate) * up, dtype
  EPI_F32 = 3      // out[M,N] fp32
};

// row_seq[r] / row_pos[r]: sequence and cache position of every row of a call.
void launch_row_index_prefill(const int32_t* cu_seqlens, int batch, int total, int32_t* row_seq,
                              int32_t* row_pos, int32_t* last_rows, hipStream_t st);
// Decode: row b is sequence b at position seq_lens[b]; -1 marks a row that has no room left.
void launch_row_index_decode(const int32_t* seq_lens, int batch, int max_seq, int32_t* row_seq,
                             int32_t* row_pos, int32_t* last_rows, hipStream_t st);
void launch_seq_lens_set(const int32_t* cu_seqlens, int batch, int32_t* seq_lens, hipStream_t st);
void launch_seq_lens_inc(int batch, int max_seq, int32_t* seq_lens, hipStream_t st);

// Decode step, fused path: row maps + seq_lens increment + fp32 residual rows + their
// storage-type copy xb (times a gain) + per-16-column sums of squares ss_part[batch][d/16], one launch.
// table != nullptr: `in` holds int32 token ids and rows are gathered from the table.
// xb = storage-type copy of the rows times gamma (the gain of the first norm; nullptr: none).
void launch_decode_prologue(uint32_t dt, const void* table, const void* in, int32_t* seq_lens, int batch, int max_seq,
                            int d, int vocab, int32_t* row_seq, int32_t* row_pos, int32_t* last_rows, float* x,
                            void* xb, float* ss_part, const void* gamma, hipStream_t st);

void launch_embed(uint32_t dt, const void* table, const int32_t* tok, float* x, int rows, int d,
                  int vocab, hipStream_t st);
void launch_load_hidden(uint32_t dt, const void* in, float* x, size_t n, hipStream_t st);
void launch_store_hidden(uint32_t dt, const float* x, void* out, size_t n, hipStream_t st);

// y[r,:] = x[map ? map[r] : r, :] / sqrt(mean(x^2) + eps) * gamma
void launch_rmsnorm(uint32_t dt, const float* x, const void* gamma, void* y, int rows, int d,
                    float eps, const int32_t* row_map, hipStream_t st);

// Scratch for GEMM kernels that split K across workgroups (fp32 partial tiles).
struct GemmScratch {
  float* splitk = nullptr;
  size_t bytes = 0;
};
struct SkinnyFusion;

// C = A[M,K] * W[N,K]^T with fp32 accumulation; A, W in dtype.  `fusion` (decode steps only)
// folds an RMSNorm into the GEMM; the caller must have checked gemm_decode_fusable().
void launch_gemm(uint32_t dt, Epilogue epi, const void* A, const void* W, int M, int N, int K,
                 void* out, float* resid, hipStream_t st, const GemmScratch* scratch = nullptr,
                 const SkinnyFusion* fusion = nullptr);
bool gemm_decode_fusable(int M, int N, int K);
// fp32 bytes of split-K scratch that cover any GEMM of up to `rows` (<= 64) rows and `cols`
// columns (count 2F for the gate-up projection)
size_t gemm_scratch_bytes(int rows, size_t cols);

void launch_gemm_generic(uint32_t dt, Epilogue epi, const void* A, const void* W, int M, int N, int K,
                         void* out, float* resid, hipStream_t st);

// bf16 MFMA kernel for many-row GEMMs (prompt pass); needs K % 64 == 0.
bool gemm_mfma_supported(int M, int N, int K);
void launch_gemm_mfma(Epilogue epi, const void* A, const void* W, int M, int N, int K, void* out, float* resid,
                      hipStream_t st);
// The QKV projection of a prompt pass with RoPE and the KV-cache append in its epilogue: rotated
// query rows go to out[M,N] (N = (hq + 2 hkv) hd, key and value columns of `out` are not
// written), rotated keys and the values go to their cache rows (row_seq[m], row_pos[m]; rows
// with row_pos < 0 are skipped).  head_dim 64 or 128.
struct RopeAppend {
  const float* cs = nullptr;        // cos/sin table [max_seq][hd/2][2]
  const int32_t* row_seq = nullptr;
  const int32_t* row_pos = nullptr;
  int hq = 0, hkv = 0, hd = 0, max_seq = 0;
  __bf16* kc = nullptr;
  __bf16* vc = nullptr;
};
// out[M,N] = bf16(resid + A W^T), the stage's output rows; `resid` is not changed.
bool gemm_mfma_resid_out_supported(int M, int N, int K, const void* out);
void launch_gemm_mfma_resid_out(const void* A, const void* W, int M, int N, int K, const float* resid, void* out, hipStream_t st);
// resid = in + A W^T with `in` in bf16: the first residual add of a stage that is given hidden rows
bool gemm_mfma_resid_in_supported(int M, int N, int K, const void* in);
void launch_gemm_mfma_resid_in(const void* A, const void* W, int M, int N, int K, const void* in, float* resid, hipStream_t st);
bool gemm_mfma_rope_supported(int M, int N, int K, int hq, int hkv, int hd);
void launch_gemm_mfma_rope(const void* A, const void* W, int M, int N, int K, void* out, const RopeAppend& rope,
                           hipStream_t st);

// GEMM in tiles of bm rows x bn weight rows, K cut `splits` ways (gemm_tiled*.hip): row counts between the
// weight-streaming kernels and the 256 x 256 tiles in bf16, every fp32 GEMM whose K is a multiple of 16.
// Output: TILED_PART fp32 partial tiles part[split][M][N] (one split: an fp32 matrix), TILED_STORE
// the storage type, TILED_SWIGLU silu(gate) * up, TILED_ROPE as launch_gemm_mfma_rope.
enum TiledEpi : int { TILED_PART = 0, TILED_STORE = 1, TILED_SWIGLU = 2, TILED_ROPE = 3 };
// The tiles there are.  bf16 (gemm_tiled_bf16.hip): 16-row and 16-weight-row fragments of a wavefront, wavefront rows and
// columns, with SwiGLU too (gate and up are two fragments of one wavefront).  What a tile gains over the next best, where it
// gains most (7B, 13B and 70B projections, 24..400 rows, cold weights): 32 x 64 32 % (70B QKV, 24 rows), 32 x 96 9 % and
// 32 x 128 41 % (7B and 13B gate-up, 24), 48 x 48 7 % and 48 x 64 1 % (70B QKV and O, 45), 48 x 96 as fast as 64 x 96 (7B
// gate-up, 45), 64 x 48 11 % (7B QKV, 64), 64 x 64 18 % (13B QKV, 64), 64 x 96 10 % (7B gate-up, 64), 64 x 128 28 % (13B gate-up,
// 45), 64 x 224 6 % (70B gate-up, 64: 139.5 us, 64 x 128 148.1), 96 x 96 6 % (70B QKV, 120), 96 x 128 12 % (70B gate-up, 80),
// 96 x 192 4 % (7B QKV, 350), 128 x 64 16 % (7B down, 128), 128 x 96 5 % (70B QKV, 160), 128 x 128 13 % (70B QKV, 311),
// 128 x 192 12 % (7B QKV, 400), 160 x 96 4 % (7B QKV, 290), 160 x 128 20 % (70B QKV, 400), 160 x 192 12 % (7B gate-up, 311),
// 160 x 256 32 % (70B gate-up, 160), 256 x 128 18 % (70B gate-up, 192), 256 x 192 11 % (7B gate-up, 400).
#define LS_TILED_BF16(X)                                                                               \
  X(1, 2, 2, 2, false) X(2, 2, 1, 3, true) X(2, 2, 1, 4, true)                                          \
  X(1, 3, 3, 1, false) X(1, 2, 3, 2, false) X(3, 2, 1, 3, true)                                         \
  X(4, 1, 1, 3, false) X(2, 2, 2, 2, false) X(4, 2, 1, 3, true) X(2, 4, 2, 2, true) X(4, 2, 1, 7, true) \
  X(3, 3, 2, 2, false) X(3, 4, 2, 2, true) X(3, 6, 2, 2, true)                                          \
  X(4, 2, 2, 2, false) X(4, 3, 2, 2, false) X(4, 4, 2, 2, true) X(4, 6, 2, 2, true)                     \
  X(5, 3, 2, 2, false) X(5, 4, 2, 2, true) X(5, 6, 2, 2, true) X(5, 4, 2, 4, true)                      \
  X(8, 4, 2, 2, true) X(4, 6, 4, 2, true)
// fp32 on fp32 instructions (gemm_tiled_f32.hip): rows, weight rows, wavefront rows, fragments of a wavefront, SwiGLU.
#define LS_TILED_F32(X) \
  X(32, 64, 2, 1, 1, false) X(32, 128, 2, 1, 2, true) X(64, 64, 2, 2, 1, false) X(64, 128, 2, 2, 2, true) X(128, 64, 2, 4, 1, false)
// fp32 by bf16 products of split operands (gemm_split_f32.hip): rows at most, weight rows.
#define LS_SPLIT_TILES(X) X(96, 128) X(128, 128) X(176, 128) X(128, 192)
struct TiledPlan {
  int bm = 0, bn = 0, splits = 0;  // splits == 0: not supported
};
// The plan with the shortest estimated time, which `us` receives.  to_scratch: the output is partial tiles,
// splits * M * N floats, which have to fit scratch_bytes; otherwise it is the caller's matrix and K is not cut.  parts_bytes: room
// for the parts of A, without which the tiles of LS_SPLIT_TILES are not planned.
TiledPlan gemm_tiled_plan(uint32_t dt, int epi, int M, int N, int K, bool to_scratch, size_t scratch_bytes, float* us,
                          size_t parts_bytes = SIZE_MAX);
inline bool gemm_by_parts(uint32_t dt, const TiledPlan& p) { return dt == F32 && p.bm * p.bn >= 96 * 128; }
// parts: gemm_split_parts_bytes(M, K) of scratch for the parts of A, which the fp32 tiles of LS_SPLIT_TILES need.
bool launch_gemm_tiled(uint32_t dt, int epi, const TiledPlan& p, const void* A, const void* W, int M, int N, int K, void* out,
                       const RopeAppend& rope, hipStream_t st, void* parts = nullptr);
size_t gemm_split_parts_bytes(int M, int K);
// Estimated time of launch_gemm_mfma (ncols: output columns of a tile, 256 or with SwiGLU 128).
float gemm_mfma_us(int M, int N, int K, int ncols);

// fp32 GEMM of one to eight rows (gemm_rows_f32.hip), a plan with bm == 0.  gamma: A holds residual rows, their RMSNorm is
// what is multiplied (row_map: row m of the call is row row_map[m] of A).  add: the output is added to it (TILED_PART, no gamma).
// Both need a plan that does not cut K, the norm rows that gemm_rows_f32_norm_supported takes.
struct RowsF32Fusion {
  const float* gamma = nullptr;
  float eps = 0.f;
  const int32_t* row_map = nullptr;
  const float* add = nullptr;
};
int gemm_rows_f32_splits(int epi, int M, int N, int K, bool to_scratch, size_t scratch_bytes);
bool gemm_rows_f32_norm_supported(int M, int N, int K);
bool launch_gemm_rows_f32(int epi, const void* A, const void* W, int M, int N, int K, int splits, void* out, hipStream_t st,
                          const RowsF32Fusion& f = {});

// A whole generation step of a small fp32 model in one launch (step_small_f32.hip): the stage's layers and, with head_w, its
// LM head, whose logits go to `logits` and the rows' next tokens to `out`; without, the rows behind the last layer go there.
struct SmallStep {
  const float* w = nullptr;       // the first layer's block, the others layer_stride floats apart
  size_t layer_stride = 0, o_qkv = 0, o_o = 0, o_g2 = 0, o_gu = 0, o_d = 0;  // tensors of a block, in floats
  const float* table = nullptr;   // embedding rows: `in` holds token ids
  const float* in = nullptr;
  float* out = nullptr;
  const float *head_gain = nullptr, *head_w = nullptr;
  float* logits = nullptr;
  int layers = 0, d = 0, hq = 0, hkv = 0, hd = 0, F = 0, vocab = 0, max_seq = 0;
  int group = 0, cut_o = 0, cut_d = 0;  // powers of two: query heads per kv head, parts that the K of O and down is summed in
  float eps = 0.f;
  const float2* cs = nullptr;
  float *kc = nullptr, *vc = nullptr;
  size_t kv_layer = 0;            // floats
  float *qkv = nullptr, *attn = nullptr, *h = nullptr;  // the last layer's projections, attention output and SwiGLU output
  int32_t* seq_lens = nullptr;
  unsigned long long* xch = nullptr;  // SmallStepPlaces
  unsigned* epoch = nullptr;
};
// Where the workgroups of such a step hand each other activations, on the current device: a stage's own from its creation to
// its end, and null where it has no such steps or other stages hold all there is.
struct SmallStepPlaces {
  unsigned long long* xch = nullptr;
  unsigned* epoch = nullptr;  // the last step's tag
};
SmallStepPlaces take_small_step_places(int device, int d, int hq, int hkv, int hd, int F, int vocab);
void give_small_step_places(int device, SmallStepPlaces places);
bool small_step_supported(const SmallStep& a, int rows, int max_keys);
bool small_step_room(hipStream_t st);  // all workgroups of such steps on all queues can be on the stream's CUs together
void launch_small_step(const SmallStep& a, int rows, hipStream_t st);

// One pass over rows of width d (a multiple of 4, at most 8192).  Source: the residual rows plus `splits`
// partial tiles, the call's hidden rows, or embedding rows; the latter two also write the call's
// bookkeeping (row -> sequence and position, last rows, seq_lens).  Result: the stage's output rows
// (out), or the residual rows x (not with norm_only) and, with a gain, their RMSNorm y.
enum RowsSrc : int { ROWS_RESID = 0, ROWS_HIDDEN = 1, ROWS_EMBED = 2 };
struct RowsArgs {
  int rows = 0, d = 0;
  float* x = nullptr;
  const float* part = nullptr;
  int splits = 0;
  const void* in = nullptr;
  const void* table = nullptr;
  int vocab = 0;
  const int32_t* cu = nullptr;  // prompt pass: sequence bounds; nullptr: generation step
  int batch = 0, max_seq = 0;
  int32_t *row_seq = nullptr, *row_pos = nullptr, *last_rows = nullptr, *seq_lens = nullptr;
  void* out = nullptr;
  const void* gamma = nullptr;
  void* y = nullptr;
  float eps = 0.f;
  bool norm_only = false;
};
bool rows_supported(int d);
void launch_rows(uint32_t dt, int src, const RowsArgs& a, hipStream_t st);

// bf16 weight-streaming kernel for decode steps (M <= 64); needs N % 16 == 0, K % 128 == 0.
// ks = wavefronts that split K inside a workgroup (4, 8, 16), 0 = chosen from the shape.
// Optional RMSNorm fusion of the decode step (all pointers device memory).  The gain of a
// norm is applied by whoever PRODUCES the bf16 copy of the residual rows, the row scale by
// the GEMM that CONSUMES it:
//   xb_out != nullptr (EPI_RESID): also write xb_out[M,N] = bf16(x_new * gamma_out[n])
//     (gamma_out == nullptr: no gain) and each row's sum of squares of x_new per 16-column
//     tile to ss_out[M][N/16].
//   ss_in != nullptr (EPI_STORE / EPI_SWIGLU, EPI_F32 of up to 16 rows): X is such a copy; the accumulator is scaled
//     by 1/sqrt(sum(ss_in[row][0..n_part)) / K + eps) of its row in the epilogue.
struct SkinnyFusion {
  const float* ss_in = nullptr;
  int n_part = 0;
  float eps = 0.f;
  __bf16* xb_out = nullptr;
  float* ss_out = nullptr;
  const __bf16* gamma_out = nullptr;
};
bool gemm_skinny_supported(int M, int N, int K);
void launch_gemm_skinny(Epilogue epi, const void* X, const void* W, int M, int N, int K, void* out, float* resid,
                        int ks, hipStream_t st, const SkinnyFusion* fusion = nullptr);

// bf16 weight-streaming kernel for decode batches of 17..64 rows (K split across
// workgroups, X staged once per workgroup); needs N % 64 == 0, K % 128 == 0.
bool gemm_wide_supported(int M, int N, int K);
size_t gemm_wide_workspace_bytes(int M, int N, int K, bool glu);
void launch_gemm_wide(Epilogue epi, const void* X, const void* W, int M, int N, int K, void* out, float* resid,
                      float* splitk_ws, hipStream_t st, const SkinnyFusion* fusion);

// Rotate q (in place inside qkv) and k by the per-position cos/sin table, write k and v
// into the cache at [seq][kv head][pos].  qkv is [rows, (Hq+2Hkv)*hd].
void launch_rope_append(uint32_t dt, void* qkv, const float* cs_table, const int32_t* row_seq,
                        const int32_t* row_pos, int rows, int hq, int hkv, int hd, int max_seq,
                        void* kcache, void* vcache, hipStream_t st);

// Causal attention of every row against its sequence's cache positions 0..row_pos[r].
// q is read from qkv ([rows, qkv_stride]); out is [rows, Hq*hd].
// Attention of one layer, including RoPE and the KV-cache append of the call's rows.
// qkv [rows, (Hq+2Hkv)*hd] holds the un-rotated projections and may be rotated in place.
// Decode (cu_seqlens == nullptr): every row is the single new row of its sequence; max_len is
// then an upper bound of the keys a row attends to, and attn_scratch the buffer for the
// partial results of contexts that are split over several workgroups (may be nullptr).
// Prefill: sequence b owns rows [cu_seqlens[b], cu_seqlens[b+1]) at positions 0.., the
// longest sequence has max_len rows.  out is [rows, Hq*hd].
void launch_attention_block(uint32_t dt, const int32_t* cu_seqlens, int batch, int max_len, void* qkv,
                            const float* cs_table, void* kcache, void* vcache, const int32_t* row_seq,
                            const int32_t* row_pos, int rows, int hq, int hkv, int hd, int max_seq, void* out,
                            hipStream_t st, float* attn_scratch = nullptr, size_t attn_scratch_bytes = 0,
                            bool rope_done = false);

// Split-KV decode attention fused with RoPE and the cache append (bf16 and fp32); head_dim 64 or
// 128, Hq/Hkv in {1,2,4,8}.  max_keys: an upper bound of the cached keys of any row.  Where
// rows x kv heads are few, contexts are cut into chunks that run as workgroups of their own and leave
// partial results in `scratch` (attn_decode_scratch_bytes; none: one workgroup each).
bool attn_decode_supported(int hq, int hkv, int hd);
size_t attn_decode_scratch_bytes(int hq, int hkv, int hd, int max_keys);
int attn_decode_chunks(int rows, int hkv, int max_keys);  // workgroups that a (sequence, kv head) gets
void launch_attn_decode(uint32_t dt, const void* qkv, int qkv_stride, const float* cs_table, void* kc, void* vc,
                        const int32_t* row_seq, const int32_t* row_pos, int rows, int hq, int hkv, int hd,
                        int max_seq, void* out, hipStream_t st, int max_keys, float* scratch, size_t scratch_bytes);

// Workgroups of a decode attention launch: a (sequence, kv head, chunk of the context) each, chunks in grid z.
// Workgroup ids go round the eight XCDs; with the heads in x (heads_first) those of one sequence are spread over them, and
// no XCD gets all of a ragged batch's longest contexts.
struct AttnGrid {
  unsigned x, y, z;
  int heads_first;
};
AttnGrid attn_decode_grid(int rows, int hkv, int nchunk);

// bf16 decode attention on the matrix cores for grouped-query models (head_dim 128,
// 2 <= Hq/Hkv <= 16), fused with RoPE and the cache append like launch_attn_decode.
bool attn_decode_gqa_supported(int hq, int hkv, int hd);
// max_keys: an upper bound of the keys any row attends to in this step (cached + the new one);
// contexts longer than 512 keys are cut into chunks that run as workgroups of their own and
// leave partial results in `scratch` (attn_decode_gqa_scratch_bytes; none: one workgroup per
// sequence and kv head whatever its length).
size_t attn_decode_gqa_scratch_bytes(int rows, int hq, int hkv, int max_keys);
void launch_attn_decode_gqa(const void* qkv, int qkv_stride, const float* cs_table, void* kc, void* vc,
                            const int32_t* row_seq, const int32_t* row_pos, int rows, int hq, int hkv, int max_seq,
                            void* out, hipStream_t st, int max_keys, float* scratch, size_t scratch_bytes);

// bf16 flash-style causal attention for the prompt pass; head_dim 64 or 128.
bool attn_prefill_supported(int hq, int hkv, int hd);
void launch_attn_prefill(const void* qkv, int qkv_stride, const void* kc, const void* vc, const int32_t* cu_seqlens,
                         int batch, int rows, int max_len, int hq, int hkv, int hd, int max_seq, void* out, hipStream_t st);

// The same in fp32; head_dim 64 or 128.
bool attn_prefill_f32_supported(int hq, int hkv, int hd);
void launch_attn_prefill_f32(const void* qkv, int qkv_stride, const void* kc, const void* vc, const int32_t* cu_seqlens,
                             int batch, int max_len, int hq, int hkv, int hd, int max_seq, void* out, hipStream_t st);

void launch_attention_generic(uint32_t dt, const void* qkv, int qkv_stride, const void* kcache,
                              const void* vcache, const int32_t* row_seq, const int32_t* row_pos, int rows,
                              int hq, int hkv, int hd, int max_seq, void* out, hipStream_t st);

// tok[r] = index of the largest logit of row r, lowest index on ties.
void launch_argmax(const float* logits, int rows, int vocab, int32_t* tok, hipStream_t st);

}  // namespace ls
