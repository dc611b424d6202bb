// fp32 GEMM of one to eight rows: C[M,N] = A[M,K] W[N,K]^T on vector FMAs.
//
// Bound by streaming W once (at one row two multiply-adds per four bytes), for small matrices by the latency
// of a launch.  A wavefront owns R rows of W and walks K in pieces of 256 floats, 16 bytes per lane
// and row: whole cache lines, non-temporal, U pieces of each row in flight, no LDS and no barrier.
// The activation rows come through the caches.  A lane keeps its own partial sums and the 64 lanes are added by a
// fixed exchange at the end, so results do not depend on timing.  K is cut over gridDim.y where
// the rows of W alone leave CUs idle; the row kernel adds the parts.
// The tiled GEMM pads one row to 32 and pays a barrier per k-step: a layer of the 7B shape, one row, took 244 us
// through it and takes 176 here (0.81 GB of weights); the tiny model's generation 776 and 647 us.
// A step of the tiny model is nothing but launches, 3 us each: with the norms and the residual adds in here its
// generation (32 tokens, then 8 steps) takes 500 us instead of 620.
#include "kernels.hpp"
#include "device_util.hpp"

namespace ls {

namespace {

// Rows whose norm the GEMM takes along: a wavefront keeps them in its registers, 256 columns to a piece, up to NORM_MAX
// columns.  Every wavefront (N / 4 of them) normalises every piece again, which has to take less than the launch it saves:
// three layers of a step, norms launched / taken along, 512 columns (two pieces) 1 row 81 / 73 us, 8 rows 106 / 106; 768
// columns 5 rows 102 / 101, 6 rows 107 / 108, 8 rows 117 / 132; layer and head of 32000 entries, 384 columns 2 rows 45.3 / 44.6,
// 3 rows 47.0 / 48.0; 768 columns 1 row 49.8 / 48.5, 2 rows 54.4 / 54.8, 8 rows 76 / 152.
constexpr int NORM_MAX = 1024, NORM_PIECES = 16;
constexpr long NORM_WORK = 160000;  // pieces times N

// NORM: A holds residual rows and every wavefront normalises the ones it multiplies, all of K at once (K <= 256 U).  The
// sums are those of k_rows in the order of k_rows, so a norm that is launched on its own gives the same bits.
// ADD (TILED_PART): the sums are added to f.add.  An instance of its own, as f is not in registers when a kernel starts: without
// one the weights' first loads waited for it (8 rows, 1024 columns, K cut: 5.1 -> 6.3 us).
template <int EPI, int M, int R, int U, bool NORM, bool ADD>
__global__ void __launch_bounds__(256)
k_gemm_rows_f32(const float* __restrict__ A, const float* __restrict__ W, int N, int K, float* out, RowsF32Fusion f) {
  constexpr bool GLU = EPI == TILED_SWIGLU;
  constexpr int C = GLU ? R / 2 : R;  // output columns of a wavefront
  const int lane = threadIdx.x & 63;
  const int n0 = (blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * C;
  if (n0 >= N) return;
  const int nv = K >> 2;  // 16-byte pieces of a row
  const int nb = (nv + 63) >> 6;
  const int b0 = (int)((long)blockIdx.y * nb / gridDim.y), b1 = (int)((long)(blockIdx.y + 1) * nb / gridDim.y);
  const f32x4* w[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int n = min(n0 + r % C, N - 1) + (GLU && r >= C ? N : 0);
    w[r] = reinterpret_cast<const f32x4*>(W + (size_t)n * K);
  }
  const float* a[M];
#pragma unroll
  for (int m = 0; m < M; ++m) a[m] = A + (size_t)(NORM && f.row_map ? f.row_map[m] : m) * K;
  float base[ADD ? C : 1][M];  // what the sums are added to
  if constexpr (ADD)
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int m = 0; m < M; ++m) base[c][m] = f.add[(size_t)m * N + min(n0 + c, N - 1)];
  float acc[R][M];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int m = 0; m < M; ++m) acc[r][m] = 0.f;
  for (int b = b0; b < b1; b += U) {
    f32x4 wv[U][R], xv[U][M];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = (b + u) * 64 + lane;
      const bool live = b + u < b1 && i < nv;
#pragma unroll
      for (int r = 0; r < R; ++r) wv[u][r] = live ? __builtin_nontemporal_load(w[r] + i) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int m = 0; m < M; ++m)
        xv[u][m] = live ? reinterpret_cast<const f32x4*>(a[m])[i] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if constexpr (NORM) {
      f32x4 gv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = (b + u) * 64 + lane;
        gv[u] = i < nv ? reinterpret_cast<const f32x4*>(f.gamma)[i] : f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int m = 0; m < M; ++m) {
        float tot = 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const f32x4 v = xv[u][m];
          float ss = 0.f;
          ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
          tot += wave_sum(ss);
        }
        const float inv = 1.0f / sqrtf(tot / (float)K + f.eps);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) xv[u][m][e] = xv[u][m][e] * inv * gv[u][e];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[r][m] = fmaf(wv[u][r][e], xv[u][m][e], acc[r][m]);
  }
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int m = 0; m < M; ++m) {
      float v = row16_sum(acc[r][m]);
      v += __shfl_xor(v, 16);
      acc[r][m] = v + __shfl_xor(v, 32);
    }
  if (lane != 0) return;
#pragma unroll
  for (int c = 0; c < C; ++c)
    if (n0 + c < N)
#pragma unroll
      for (int m = 0; m < M; ++m) {
        float v = GLU ? silu_f(acc[c][m]) * acc[C + c][m] : acc[c][m];
        if constexpr (ADD) v += base[c][m];
        out[((size_t)blockIdx.y * M + m) * N + n0 + c] = v;
      }
}

template <int EPI, int M>
void launch_m(const float* A, const float* W, int N, int K, int splits, float* out, const RowsF32Fusion& f, hipStream_t st) {
  constexpr int R = 4, U = M <= 2 ? 4 : 2, C = EPI == TILED_SWIGLU ? R / 2 : R;
  const dim3 grid((unsigned)((N + 4 * C - 1) / (4 * C)), (unsigned)splits);
  if (f.gamma) {  // as many pieces as a row has: the registers of more cost wavefronts
    if (K <= 256) launch_kernel(k_gemm_rows_f32<EPI, M, R, 1, true, false>, grid, dim3(256), 0, st, A, W, N, K, out, f);
    else if (K <= 512) launch_kernel(k_gemm_rows_f32<EPI, M, R, 2, true, false>, grid, dim3(256), 0, st, A, W, N, K, out, f);
    else if constexpr (M * 3 <= NORM_PIECES) launch_kernel(k_gemm_rows_f32<EPI, M, R, 4, true, false>, grid, dim3(256), 0, st, A, W, N, K, out, f);
  } else if constexpr (EPI == TILED_PART) {
    if (f.add) launch_kernel(k_gemm_rows_f32<EPI, M, R, U, false, true>, grid, dim3(256), 0, st, A, W, N, K, out, f);
    else hipLaunchKernelGGL((k_gemm_rows_f32<EPI, M, R, U, false, false>), grid, dim3(256), 0, st, A, W, N, K, out, f);
  } else {
    launch_kernel(k_gemm_rows_f32<EPI, M, R, U, false, false>, grid, dim3(256), 0, st, A, W, N, K, out, f);
  }
}

template <int EPI>
bool launch_e(const float* A, const float* W, int M, int N, int K, int splits, float* out, const RowsF32Fusion& f, hipStream_t st) {
  switch (M) {
    case 1: launch_m<EPI, 1>(A, W, N, K, splits, out, f, st); return true;
    case 2: launch_m<EPI, 2>(A, W, N, K, splits, out, f, st); return true;
    case 3: launch_m<EPI, 3>(A, W, N, K, splits, out, f, st); return true;
    case 4: launch_m<EPI, 4>(A, W, N, K, splits, out, f, st); return true;
    case 5: launch_m<EPI, 5>(A, W, N, K, splits, out, f, st); return true;
    case 6: launch_m<EPI, 6>(A, W, N, K, splits, out, f, st); return true;
    case 7: launch_m<EPI, 7>(A, W, N, K, splits, out, f, st); return true;
    case 8: launch_m<EPI, 8>(A, W, N, K, splits, out, f, st); return true;
  }
  return false;
}

}  // namespace

// 0: not supported.  512 workgroups (two per CU) where K is long enough, at least two pieces of a row per part.
int gemm_rows_f32_splits(int epi, int M, int N, int K, bool to_scratch, size_t scratch_bytes) {
  if (M < 1 || M > 8 || epi == TILED_ROPE || K < 4 || K % 4) return 0;
  if (to_scratch && (size_t)M * N * sizeof(float) > scratch_bytes) return 0;
  const int wgs = (N + 15) / 16, nb = (K / 4 + 63) / 64;
  int s = 1;
  while (to_scratch && s < 8 && wgs * s < 512 && nb >= 4 * s && (size_t)(2 * s) * M * N * sizeof(float) <= scratch_bytes) s *= 2;
  return s;
}

bool gemm_rows_f32_norm_supported(int M, int N, int K) {
  const int pieces = M * ((K + 255) / 256);
  return M >= 1 && M <= 8 && K >= 4 && K % 4 == 0 && K <= NORM_MAX && pieces <= NORM_PIECES && (long)pieces * N <= NORM_WORK;
}

bool launch_gemm_rows_f32(int epi, const void* A, const void* W, int M, int N, int K, int splits, void* out, hipStream_t st,
                          const RowsF32Fusion& f) {
  const float *a = (const float*)A, *w = (const float*)W;
  if ((f.gamma && (f.add || splits != 1 || !gemm_rows_f32_norm_supported(M, N, K))) || (f.add && (splits != 1 || epi != TILED_PART))) return false;
  switch (epi) {
    case TILED_PART: return launch_e<TILED_PART>(a, w, M, N, K, splits, (float*)out, f, st);
    case TILED_STORE: return launch_e<TILED_STORE>(a, w, M, N, K, splits, (float*)out, f, st);
    case TILED_SWIGLU: return launch_e<TILED_SWIGLU>(a, w, M, N, K, splits, (float*)out, f, st);
  }
  return false;
}

}  // namespace ls
