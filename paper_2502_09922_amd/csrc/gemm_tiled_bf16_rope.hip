// bf16 tiled GEMM (gemm_tiled_bf16.hpp), epilogue TILED_ROPE.
#include "gemm_tiled_bf16.hpp"

namespace ls {
bool launch_gemm_tiled_bf16_rope(const TiledPlan& p, const void* A, const void* W, int M, int N, int K, void* out,
                               const RopeAppend& rope, hipStream_t st) {
  return launch_epi<TILED_ROPE>(p, A, W, M, N, K, out, rope, st);
}
}  // namespace ls
