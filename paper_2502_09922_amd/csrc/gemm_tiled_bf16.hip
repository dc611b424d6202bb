// bf16 tiled GEMM (gemm_tiled_bf16.hpp): the choice of the epilogue, and the one of partial tiles.
#include "gemm_tiled_bf16.hpp"

namespace ls {

#define LS_ARGS const TiledPlan &p, const void *A, const void *W, int M, int N, int K, void *out, const RopeAppend &rope, hipStream_t st
bool launch_gemm_tiled_bf16_store(LS_ARGS);
bool launch_gemm_tiled_bf16_swiglu(LS_ARGS);
bool launch_gemm_tiled_bf16_rope(LS_ARGS);

bool launch_gemm_tiled_bf16(int epi, LS_ARGS) {
  switch (epi) {
    case TILED_PART: return launch_epi<TILED_PART>(p, A, W, M, N, K, out, rope, st);
    case TILED_STORE: return launch_gemm_tiled_bf16_store(p, A, W, M, N, K, out, rope, st);
    case TILED_SWIGLU: return launch_gemm_tiled_bf16_swiglu(p, A, W, M, N, K, out, rope, st);
    case TILED_ROPE: return launch_gemm_tiled_bf16_rope(p, A, W, M, N, K, out, rope, st);
  }
  return false;
}

}  // namespace ls
