// bf16 instances of the tiled GEMM (gemm_tiled.hpp).
#include "gemm_tiled.hpp"

namespace ls {
bool launch_gemm_tiled_bf16(int epi, const TiledPlan& p, const void* A, const void* W, int M, int N, int K, void* out,
                            const RopeAppend& rope, hipStream_t st) {
  return tiled::launch_t<bf16>(epi, p, A, W, M, N, K, out, rope, st);
}
}  // namespace ls
