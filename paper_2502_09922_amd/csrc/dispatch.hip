// Shape-based choice between the kernels of one operator.  GEMMs: what the stage's plans (gemm_tiled_plan) leave;
// fp32 takes the generic kernel here, bf16 an MFMA kernel wherever its shape constraints hold.  Attention: the
// kernel for the type and head shape, else the generic one.
#include "kernels.hpp"

namespace ls {

bool gemm_decode_fusable(int M, int N, int K) { return gemm_skinny_supported(M, N, K); }

size_t gemm_scratch_bytes(int rows, size_t cols) {
  const size_t r = rows < 64 ? rows : 64;
  return 8 * r * cols * sizeof(float);  // up to 8 K splits
}

void launch_gemm(uint32_t dt, Epilogue epi, const void* A, const void* W, int M, int N, int K, void* out,
                 float* resid, hipStream_t st, const GemmScratch* scratch, const SkinnyFusion* fusion) {
  if (dt == BF16 && M <= 64) {
    // 17..64 rows: the wide kernel, if its shape constraints hold and the scratch is large enough
    if (M > 16 && scratch && scratch->splitk && gemm_wide_supported(M, N, K) &&
        gemm_wide_workspace_bytes(M, N, K, epi == EPI_SWIGLU) <= scratch->bytes) {
      launch_gemm_wide(epi, A, W, M, N, K, out, resid, scratch->splitk, st, fusion);
      return;
    }
    if (gemm_skinny_supported(M, N, K)) {
      launch_gemm_skinny(epi, A, W, M, N, K, out, resid, 0, st, fusion);
      return;
    }
  }
  if (dt == BF16 && M > 64 && gemm_mfma_supported(M, N, K)) {
    launch_gemm_mfma(epi, A, W, M, N, K, out, resid, st);
    return;
  }
  launch_gemm_generic(dt, epi, A, W, M, N, K, out, resid, st);
}

// Heads first but where few sequences are cut into chunks, and as far as y goes (65535); x takes any number.  A layer of 16 query
// and 4 kv heads, contexts of 500..4000 keys, rows first / heads first: 4 sequences 41.3 / 44.0 us, 16 54.0 / 57.2, 32 80.3 / 82.0,
// 48 95.1 / 88.1; 8 kv heads, 16 sequences 69.6 / 70.4, 40 121.2 / 109.6.  16 heads, 4 sequences of 1000 keys: 39.0 / 40.9.
// fp32, 2 kv heads, 48 sequences of 200..1500 keys: 58.3 / 54.9 us the kernel.
constexpr int ROWS_FIRST_ROWS = 32;
constexpr long ROWS_FIRST_PAIRS = 128;
AttnGrid attn_decode_grid(int rows, int hkv, int nchunk) {
  const bool heads_first = (nchunk == 1 || rows > ROWS_FIRST_ROWS || (long)rows * hkv > ROWS_FIRST_PAIRS) && rows <= 65535;
  return heads_first ? AttnGrid{(unsigned)hkv, (unsigned)rows, (unsigned)nchunk, 1} : AttnGrid{(unsigned)rows, (unsigned)hkv, (unsigned)nchunk, 0};
}

void launch_attention_block(uint32_t dt, const int32_t* cu_seqlens, int batch, int max_len, void* qkv,
                            const float* cs_table, void* kcache, void* vcache, const int32_t* row_seq,
                            const int32_t* row_pos, int rows, int hq, int hkv, int hd, int max_seq, void* out,
                            hipStream_t st, float* attn_scratch, size_t attn_scratch_bytes, bool rope_done) {
  const bool decode = cu_seqlens == nullptr;
  const int qkv_stride = (hq + 2 * hkv) * hd;
  if (dt == BF16 && decode && attn_decode_gqa_supported(hq, hkv, hd)) {
    launch_attn_decode_gqa(qkv, qkv_stride, cs_table, kcache, vcache, row_seq, row_pos, rows, hq, hkv, max_seq, out, st,
                           max_len, attn_scratch, attn_scratch_bytes);
    return;
  }
  if (decode && attn_decode_supported(hq, hkv, hd)) {
    launch_attn_decode(dt, qkv, qkv_stride, cs_table, kcache, vcache, row_seq, row_pos, rows, hq, hkv, hd, max_seq, out, st,
                       max_len, attn_scratch, attn_scratch_bytes);
    return;
  }
  if (!rope_done) launch_rope_append(dt, qkv, cs_table, row_seq, row_pos, rows, hq, hkv, hd, max_seq, kcache, vcache, st);
  if (dt == BF16 && !decode && attn_prefill_supported(hq, hkv, hd)) {
    launch_attn_prefill(qkv, qkv_stride, kcache, vcache, cu_seqlens, batch, rows, max_len, hq, hkv, hd, max_seq, out, st);
    return;
  }
  if (dt == F32 && !decode && attn_prefill_f32_supported(hq, hkv, hd)) {
    launch_attn_prefill_f32(qkv, qkv_stride, kcache, vcache, cu_seqlens, batch, max_len, hq, hkv, hd, max_seq, out, st);
    return;
  }
  launch_attention_generic(dt, qkv, qkv_stride, kcache, vcache, row_seq, row_pos, rows, hq, hkv, hd, max_seq, out, st);
}

}  // namespace ls

// For the tests; not declared in ls_stage.h: grid and order of a decode attention launch.
extern "C" void ls_test_attn_decode_grid(int rows, int hkv, int nchunk, int out[4]) {
  const ls::AttnGrid g = ls::attn_decode_grid(rows, hkv, nchunk);
  out[0] = (int)g.x; out[1] = (int)g.y; out[2] = (int)g.z; out[3] = g.heads_first;
}
