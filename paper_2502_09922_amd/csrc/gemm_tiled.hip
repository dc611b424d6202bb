// Choice of the tiled GEMM's tile and K split (gemm_tiled_bf16.hip, gemm_tiled_f32.hip, gemm_split_f32.hip), its launcher, and the row kernel
// that stands between two GEMMs: adds the K-split partials to the residual rows and normalises.
#include "kernels.hpp"
#include "device_util.hpp"

#include <cmath>

namespace ls {

bool launch_gemm_tiled_bf16(int epi, const TiledPlan& p, const void* A, const void* W, int M, int N, int K, void* out,
                            const RopeAppend& rope, hipStream_t st);
bool launch_gemm_tiled_f32(int epi, const TiledPlan& p, const void* A, const void* W, int M, int N, int K, void* out,
                           const RopeAppend& rope, hipStream_t st);

bool launch_gemm_split_f32(int epi, const TiledPlan& p, const void* A, void* parts, const void* W, int M, int N, int K, void* out,
                           const RopeAppend& rope, hipStream_t st);

bool gemm_tiled_supported(uint32_t dt, int epi, int M, int N, int K) {
  const size_t e = dt == F32 ? 4 : 2, wrows = (size_t)N * (epi == TILED_SWIGLU ? 2 : 1);
  // half k-steps; whole 16-column fragments; 32-bit byte offsets into both operands
  return M >= 1 && N >= 16 && N % 16 == 0 && K >= 64 && K % (int)(64 / e) == 0 && wrows * K * e < (1ull << 32) &&
         (size_t)M * K * e < (1ull << 32);
}

// One fp32 layer of the 7B shape on vector FMAs / through the tiles: 1 row 176 / 244 us, 4 rows and the LM head
// 299 / 352, 8 rows 219 / 250; the FMAs of each further row cost 6 us, the tiles nothing up to 32.
constexpr int ROWS_F32_MAX = 8;

// Time of a launch, in microseconds, from sweeps over the tiles (7B, 13B and 70B layers, 12..1024 rows in bf16,
// 24..512 in fp32, cold weights).  bf16: a k-step of a workgroup costs 0.02 us + 2.4 ns per row it brings into LDS,
// whatever the arithmetic (48 x 48 0.24, 64 x 64 0.33, 64 x 128 0.47, 128 x 128 0.58, 160 x 192 0.85, 256 x 128 0.9 us
// measured; a sixth more where only two stages fit: 256 x 192 1.33); rows past the end of the call are not fetched,
// and the tiles of a column wait for the same weight lines, so that it is their mean that counts; one tile row is a
// little faster than two of the same lines (7B gate-up, 128 rows, 128 x 128 44.0, 96 x 192 46.9, 64 x 192 48.4 us;
// 13B, 256 rows, 256 x 128 76.3, 160 x 256 82.7; 70B 244 and 262).  Weights do not come from memory faster than 6.4
// TB/s.  Chosen so, the four projections at 11 row counts of the 7B shape take 1584 us together, the fastest tile and
// split of each 1552.  fp32: at least the matrix work (64 x 64 at 0.4, 64 x 128 at 0.46 TFLOP/s per CU); by split
// operands 0.39 us + 0.055 per pair of 16-row fragments and wavefront (96 x 128 1.05..1.1, 128 x 128 1.2..1.4, 176 x
// 128 1.6..1.7, 128 x 192 1.9..2.1 us measured) and the kernel in front, whose launch and tall tiles do not pay for
// small matrices (two layers of 512 columns, 97..512 rows on fp32 instructions 103..196 us, by split operands
// 175..263; 1024 columns, 97 rows 152 and 244, 311 rows 251 and 292).  One workgroup fits a CU, so the launch takes as
// many rounds as its fullest XCD has workgroups for its 32 CUs; every K split writes and reads an fp32 tile.
TiledPlan gemm_tiled_plan(uint32_t dt, int epi, int M, int N, int K, bool to_scratch, size_t scratch_bytes, float* us,
                          size_t parts_bytes) {
  TiledPlan best;
  float best_us = 1e30f, best_rank = 1e30f;
  if (dt == F32 && M <= ROWS_F32_MAX) {  // bm == 0: the kernel for few fp32 rows
    best.splits = gemm_rows_f32_splits(epi, M, N, K, to_scratch, scratch_bytes);
    if (best.splits) {
      if (us) *us = 0.f;
      return best;
    }
  }
  if (gemm_tiled_supported(dt, epi, M, N, K)) {
    const int kb = dt == F32 ? 32 : 64, nk = (K + kb - 1) / kb;
    const float stream = (float)N * (epi == TILED_SWIGLU ? 2 : 1) * (float)K * 2.f / 6.4e6f + 3.f;
    auto consider = [&](int bm, int bn, float step, float extra) {
      const int ncols = epi == TILED_SWIGLU ? bn / 2 : bn;
      const int tiles_m = (M + bm - 1) / bm, panels = ((N + ncols - 1) / ncols + 7) / 8;
      if (dt == BF16) {
        if (bm > 32 && bm >= 2 * M) return;  // more than half of the products for rows that are not there
        step = 0.02f + 0.0024f * ((float)((M + 7) / 8 * 8) / (float)tiles_m + (float)bn);
        if ((bm + bn) * 128 * 3 > 160 * 1024) step *= 1.18f;
      }
      for (int s = 1; s <= 8; ++s) {
        // partial tiles, also those of a single split, have to fit the scratch
        if ((to_scratch && (size_t)s * M * N * sizeof(float) > scratch_bytes) || (s > 1 && (!to_scratch || nk < 2 * s))) break;
        const long per_xcd = (long)panels * tiles_m * s;
        auto estimate = [&](float a_step) {
          float t = (float)((per_xcd + 31) / 32) * ((float)((nk + s - 1) / s) * a_step + 2.5f);
          if (dt == BF16) {  // whichever is longer, and some more where both are alike
            const float a = t * t, b = stream * stream;
            t = sqrtf(sqrtf(a * a + b * b));
          }
          return t + (float)s * (float)M * (float)N * 8.f / 4e6f + extra;
        };
        // one tile row goes before two that bring the same lines; the time that others compare with stays the estimate's
        const float rank = estimate(dt == BF16 && tiles_m > 1 && !to_scratch ? 1.02f * step : step);
        if (rank < best_rank) {
          best_rank = rank;
          best_us = estimate(step);
          best.bm = bm; best.bn = bn; best.splits = s;
        }
      }
    };
    if (dt == BF16) {
#define LS_TILE(tm_, tn_, wm_, wn_, glu_) \
  if (epi != TILED_SWIGLU || glu_) consider(16 * wm_ * tm_, 16 * wn_ * tn_, 0.f, 0.f);
      LS_TILED_BF16(LS_TILE)
#undef LS_TILE
    } else {
      auto fp32 = [&](int bm, int bn) {
        const float area = (float)(bm * bn), mma = 64.f * area / (0.36e6f + 12.f * area) + 0.05f;
        const float step = 0.05f + 0.0024f * (float)(bm + bn);
        consider(bm, bn, mma > step ? mma : step, 0.f);
      };
#define LS_TILE(bm_, bn_, wm_, tm_, tn_, glu_) \
  if (epi != TILED_SWIGLU || glu_) fp32(bm_, bn_);
      LS_TILED_F32(LS_TILE)
#undef LS_TILE
#define LS_TILE(bm_, bn_) consider(bm_, bn_, 0.39f + 0.055f * (bm_ / 16) * (bn_ / 64) + (bn_ > 128 ? 0.2f : 0.f), 3.5f);
      if (gemm_split_parts_bytes(M, K) <= parts_bytes) { LS_SPLIT_TILES(LS_TILE) }
#undef LS_TILE
    }
  }
  if (us) *us = best_us;
  return best;
}

bool launch_gemm_tiled(uint32_t dt, int epi, const TiledPlan& p, const void* A, const void* W, int M, int N, int K, void* out,
                       const RopeAppend& rope, hipStream_t st, void* parts) {
  if (!p.splits) return false;
  if (!p.bm) return launch_gemm_rows_f32(epi, A, W, M, N, K, p.splits, out, st);
  if (dt != F32) return launch_gemm_tiled_bf16(epi, p, A, W, M, N, K, out, rope, st);
  return launch_gemm_tiled_f32(epi, p, A, W, M, N, K, out, rope, st) ||
         (parts && launch_gemm_split_f32(epi, p, A, parts, W, M, N, K, out, rope, st));
}

namespace {

// One workgroup per row; the row lives in registers (P 16-byte pieces per thread, P * NT * 4 columns at
// most).  This one pass stands for the separate load (or embedding gather), residual add, norm and
// store passes.  Many rows are bound by HBM: 256 threads, eight workgroups per CU.  With few rows it is the
// latency of a chain of loads: 1024 threads, and the partial tiles four at a time in flight
// (45..311 rows of 4096 columns, 4 to 8 splits: 8.5 us with 256 threads and one split after the other).
template <class T, int SRC, int NT, int P>
__global__ void __launch_bounds__(NT) k_rows(const void* in, float* x, const void* gamma, void* y, int rows, int d, int splits, RowsArgs a) {
  // what the first loads need comes in registers, ahead of the structure
  if (SRC == ROWS_RESID) a.part = (const float*)in;
  else a.in = in;
  a.x = x; a.gamma = gamma; a.y = y; a.rows = rows; a.d = d; a.splits = splits;
  typedef T T4 __attribute__((ext_vector_type(4)));
  __shared__ float wsum[NT / 64];
  const int r = blockIdx.x, nv = a.d >> 2;
  if constexpr (SRC != ROWS_RESID) {
    if (threadIdx.x == 0) {
      if (a.cu) {  // prompt pass: find b with cu[b] <= r < cu[b + 1]
        int lo = 0, hi = a.batch;
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (a.cu[mid] <= r) lo = mid; else hi = mid;
        }
        const int c0 = a.cu[lo], c1 = a.cu[lo + 1];
        a.row_seq[r] = lo;
        a.row_pos[r] = r - c0;
        if (r == c1 - 1) {
          a.last_rows[lo] = r;
          a.seq_lens[lo] = c1 - c0;
        }
      } else {  // generation step: a sequence without room is left alone and marked -1
        const int p = a.seq_lens[r];
        const bool ok = p >= 0 && p < a.max_seq;
        a.row_seq[r] = r;
        a.row_pos[r] = ok ? p : -1;
        a.last_rows[r] = r;
        if (ok) a.seq_lens[r] = p + 1;
      }
    }
  }
  auto widen = [](const T* p, bool vec) {
    f32x4 v;
    if (vec) {
      const T4 t = *reinterpret_cast<const T4*>(p);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = to_f(t[e]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = to_f(p[e]);
    }
    return v;
  };
  float* xr = a.x + (size_t)r * a.d;
  // few rows: the gain is asked for before the rows, so that it is there when they are; many rows have the registers
  // for it only behind them
  constexpr bool EARLY = P <= 2;
  T4 gain[P];
  auto load_gain = [&]() {
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const int idx = threadIdx.x + NT * i;
      gain[i] = reinterpret_cast<const T4*>(a.gamma)[idx < nv ? idx : 0];
    }
  };
  if (EARLY && a.gamma) load_gain();
  f32x4 v[P];
  if constexpr (SRC == ROWS_RESID) {
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const int idx = threadIdx.x + NT * i;
      v[i] = idx < nv ? reinterpret_cast<const f32x4*>(xr)[idx] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const size_t split = (size_t)a.rows * a.d;
    constexpr int U = P <= 2 ? 4 : 1;  // splits in flight
    for (int s = 0; s < a.splits; s += U) {
      f32x4 p[U][P];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const f32x4* pr = reinterpret_cast<const f32x4*>(a.part + (size_t)min(s + u, a.splits - 1) * split + (size_t)r * a.d);
#pragma unroll
        for (int i = 0; i < P; ++i) {
          const int idx = threadIdx.x + NT * i;
          p[u][i] = idx < nv ? pr[idx] : f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)  // in split order
        if (s + u < a.splits)
#pragma unroll
          for (int i = 0; i < P; ++i) v[i] += p[u][i];
    }
  } else {
    const T* src;
    if constexpr (SRC == ROWS_EMBED) {
      int id = ((const int32_t*)a.in)[r];
      id = id < 0 ? 0 : (id >= a.vocab ? a.vocab - 1 : id);  // an id outside the table is clamped
      src = (const T*)a.table + (size_t)id * a.d;
    } else {
      src = (const T*)a.in + (size_t)r * a.d;
    }
    const bool vec = (reinterpret_cast<uintptr_t>(src) & (sizeof(T4) - 1)) == 0;  // the caller's buffer may lie anywhere
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const int idx = threadIdx.x + NT * i;
      v[i] = idx < nv ? widen(src + idx * 4, vec) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  if (a.out) {  // the stage's output rows
    T* o = (T*)a.out + (size_t)r * a.d;
    const bool vec = (reinterpret_cast<uintptr_t>(o) & (sizeof(T4) - 1)) == 0;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const int idx = threadIdx.x + NT * i;
      if (idx < nv) {
        T4 t;
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = from_f<T>(v[i][e]);
        if (vec) *reinterpret_cast<T4*>(o + idx * 4) = t;
        else
#pragma unroll
          for (int e = 0; e < 4; ++e) o[idx * 4 + e] = t[e];
      }
    }
    return;
  }
  if (!a.norm_only)
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const int idx = threadIdx.x + NT * i;
      if (idx < nv) reinterpret_cast<f32x4*>(xr)[idx] = v[i];
    }
  if (!a.gamma) return;
  if (!EARLY) load_gain();
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < P; ++i) ss += v[i][0] * v[i][0] + v[i][1] * v[i][1] + v[i][2] * v[i][2] + v[i][3] * v[i][3];
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) tot += wsum[w];
  const float inv = 1.0f / sqrtf(tot / (float)a.d + a.eps);
  T* yr = (T*)a.y + (size_t)r * a.d;
#pragma unroll
  for (int i = 0; i < P; ++i) {
    const int idx = threadIdx.x + NT * i;
    if (idx < nv) {
      T4 t;
#pragma unroll
      for (int e = 0; e < 4; ++e) t[e] = from_f<T>(v[i][e] * inv * to_f(gain[i][e]));
      *reinterpret_cast<T4*>(yr + idx * 4) = t;
    }
  }
}

template <class T, int NT, int P>
void launch_rows_n(int src, const RowsArgs& a, hipStream_t st) {
  const void* in = src == ROWS_RESID ? a.part : a.in;
  if (src == ROWS_RESID) k_rows<T, ROWS_RESID, NT, P><<<a.rows, NT, 0, st>>>(in, a.x, a.gamma, a.y, a.rows, a.d, a.splits, a);
  else if (src == ROWS_HIDDEN) k_rows<T, ROWS_HIDDEN, NT, P><<<a.rows, NT, 0, st>>>(in, a.x, a.gamma, a.y, a.rows, a.d, a.splits, a);
  else k_rows<T, ROWS_EMBED, NT, P><<<a.rows, NT, 0, st>>>(in, a.x, a.gamma, a.y, a.rows, a.d, a.splits, a);
}

// up to 512 rows every one of them fits the chip at once with 1024 threads.  The choice depends on
// the call's rows only: a norm folded into a residual add and one launched on its own give the same bits.
template <class T>
void launch_rows_t(int src, const RowsArgs& a, hipStream_t st) {
  if (a.rows <= 512) launch_rows_n<T, 1024, 2>(src, a, st);
  else launch_rows_n<T, 256, 8>(src, a, st);
}

}  // namespace

bool rows_supported(int d) { return d % 4 == 0 && d <= 8192; }

void launch_rows(uint32_t dt, int src, const RowsArgs& a, hipStream_t st) {
  if (a.rows <= 0) return;
  if (dt == F32) launch_rows_t<float>(src, a, st);
  else launch_rows_t<bf16>(src, a, st);
}

}  // namespace ls

namespace {

// A launch with a chosen tile.  The split tiles bring their own room for the parts, which the callers have not.
bool launch_chosen(uint32_t dt, int epi, int bm, int bn, int splits, const void* A, const void* W, int M, int N, int K, void* out,
                   const ls::RopeAppend& rope, hipStream_t st) {
  using namespace ls;
  TiledPlan p;
  p.bm = bm; p.bn = bn; p.splits = splits;
  if (bm <= 0) return false;
  bool by_parts = false;
#define LS_TILE(bm_, bn_) by_parts |= dt == F32 && bm == bm_ && bn == bn_;
  LS_SPLIT_TILES(LS_TILE)
#undef LS_TILE
  if (!by_parts) return launch_gemm_tiled(dt, epi, p, A, W, M, N, K, out, rope, st);
  void* parts = nullptr;
  if (hipMallocAsync(&parts, gemm_split_parts_bytes(M, K), st) != hipSuccess) return false;
  const bool ok = launch_gemm_tiled(dt, epi, p, A, W, M, N, K, out, rope, st, parts);
  return hipFreeAsync(parts, st) == hipSuccess && ok;
}

}  // namespace

// For the tests, which choose a tile themselves to reach its edges; not declared in ls_stage.h.  All return 0
// where there is no plan, or where the launch would not be one that the kernels take.
extern "C" int ls_test_tiled_plan(uint32_t dt, int epi, int M, int N, int K, int to_scratch, size_t scratch_bytes, int* plan) {
  const ls::TiledPlan p = ls::gemm_tiled_plan(dt, epi, M, N, K, to_scratch != 0, scratch_bytes, nullptr);
  plan[0] = p.bm; plan[1] = p.bn; plan[2] = p.splits;
  return p.splits != 0;
}

// A [M,K], W [N,K] (SwiGLU: [2N,K]), out [M,N] in the storage type, TILED_PART: fp32 [splits][M][N].
extern "C" int ls_test_tiled_gemm(uint32_t dt, int epi, int bm, int bn, int splits, const void* A, const void* W, int M, int N,
                                  int K, void* out, void* hip_stream) {
  using namespace ls;
  const int nk = dt == F32 ? (K + 31) / 32 : (K + 63) / 64;
  if ((dt != F32 && dt != BF16) || epi < TILED_PART || epi > TILED_SWIGLU || !A || !W || !out) return 0;
  if (!gemm_tiled_supported(dt, epi, M, N, K) || splits < 1 || splits > 8) return 0;
  if (splits > 1 && (epi != TILED_PART || nk < 2 * splits)) return 0;
  return launch_chosen(dt, epi, bm, bn, splits, A, W, M, N, K, out, RopeAppend{}, (hipStream_t)hip_stream);
}

// The same with RoPE and the cache append: N = (hq + 2 hkv) hd, out [M,N], cs [max_seq][hd/2][2], caches [seq][hkv][max_seq][hd].
extern "C" int ls_test_tiled_rope(uint32_t dt, int bm, int bn, const void* A, const void* W, int M, int K, void* out, const float* cs,
                                  const int32_t* row_seq, const int32_t* row_pos, int hq, int hkv, int hd, int max_seq, void* kc,
                                  void* vc, void* hip_stream) {
  using namespace ls;
  if ((dt != F32 && dt != BF16) || !A || !W || !out || !cs || !row_seq || !row_pos || !kc || !vc) return 0;
  if (hq < 1 || hkv < 1 || hd < 16 || hd % 16 || max_seq < 1) return 0;
  const int N = (hq + 2 * hkv) * hd;
  if (!gemm_tiled_supported(dt, TILED_ROPE, M, N, K)) return 0;
  RopeAppend r;
  r.cs = cs; r.row_seq = row_seq; r.row_pos = row_pos;
  r.hq = hq; r.hkv = hkv; r.hd = hd; r.max_seq = max_seq;
  r.kc = (__bf16*)kc; r.vc = (__bf16*)vc;
  return launch_chosen(dt, TILED_ROPE, bm, bn, 1, A, W, M, N, K, out, r, (hipStream_t)hip_stream);
}
