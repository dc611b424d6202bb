// fp32 GEMM of 9 to 96 rows, and of matrices too small for gemm_split_f32.hip: C[M,N] = A[M,K] W[N,K]^T on
// v_mfma_f32_16x16x4_f32.
//
// A 512-thread workgroup (8 wavefronts, one workgroup per CU) owns a tile of 32..128 rows x 64 or 128 weight rows,
// chosen per launch (gemm_tiled_plan) so that the tiles, times the number of ways K is cut, fill the chip.
//
// Data path: both operands are K-contiguous; a k-step is 128 bytes of every row (32 floats).  Rows go from global
// memory straight into LDS (global_load_lds_dwordx4) into a ring of NS stages, 16-byte chunks XOR-swizzled by
// (row/2)&7, so that the 16 rows a quarter-wave reads fall into different banks.  One barrier per stage (one or two
// k-steps): behind it the stage of this k-step has landed for every wavefront (each waited for its own fills,
// counted) and the stage of the previous one has been read by all, so its slot takes the fills NS - 1 stages ahead.
//
// Bound by the matrix instructions from 64 rows on, by the fills below.  Counters, 321 rows of the 7B shape: 0.08
// PFLOP/s of the 0.154 a large fp32 matrix product reaches.
//
// A lane's 16-byte chunk holds four consecutive k, and element e of all four lane groups together is one
// instruction's k = 4: both operands agree on which k a lane's element e is, and a sum does not care in what
// order k is visited.
//
// Weight fragments are the A operand, activations the B operand: a lane of a result holds row
// m = lane%16 of its tile and four consecutive columns n = 4*(lane/16) .. +3.
#include "kernels.hpp"
#include "device_util.hpp"

namespace ls {

namespace {

constexpr int ROWB = 128;  // bytes of a row in one k-step
constexpr int WAVES = 8;
// Tile of 16 WM TM rows x 16 WN TN columns, wavefronts WM x WN, ring as deep as LDS allows (at most
// eight stages: no shape gained from more).
template <int WM_, int TM_, int TN_>
struct Tile {
  static constexpr int WM = WM_, WN = WAVES / WM_, TM = TM_, TN = TN_;
  static constexpr int BM = 16 * WM * TM, BN = 16 * WN * TN;
  static constexpr int SUB = (BM + BN) * ROWB;  // one k-step
  // k-steps per barrier: where a step is short the barrier and the LDS latency behind it are a good part of it
  // (64 x 64: 28 -> 24 us for 45 rows of the 7B QKV); larger tiles want the ring's finer steps (96 x 128: +30 %)
  static constexpr int KS = BM + BN <= 192 ? 2 : 1;
  static constexpr int STAGE = KS * SUB;
  static constexpr int FIT = 160 * 1024 / STAGE, NS = FIT > 8 ? 8 : FIT;
  static constexpr int SMEM = NS * STAGE;
  static constexpr int NFILL = (BM + BN) / 8;              // fill instructions of a k-step, eight rows each
  static constexpr int F = (NFILL + WAVES - 1) / WAVES;    // ... of a wavefront
};

// acc[i][j] += w[j] x[i]^T over half a k-step (16 bytes of a row per lane)
template <int TM, int TN>
__device__ __forceinline__ void mma(f32x4 (&acc)[TM][TN], const u32x4 (&w)[TN], const u32x4 (&x)[TM]) {
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(f32x4, w[j])[e], __builtin_bit_cast(f32x4, x[i])[e],
                                                         acc[i][j], 0, 0, 0);
}

// The operand fragments of a k-step: of each half, TM activation row blocks and TN weight row blocks, 16 rows
// (2048 bytes) apart.  The reads and the wait for them are ONE asm statement: the compiler, which
// takes an LDS-direct load for a possible writer of all LDS, would otherwise wait for every fill
// in flight before each read, and it must not see the registers before the data is there.
#define LS_R(o_, a_, off_) "ds_read_b128 %" #o_ ", %" #a_ " offset:" #off_ "\n\t"
#define LS_W "s_waitcnt lgkmcnt(0)"
#define LS_O(v_) "=&v"(v_)
template <int TM, int TN>
__device__ __forceinline__ void read_frags(unsigned xa0, unsigned wa0, unsigned xa1, unsigned wa1, u32x4 (&x0)[TM],
                                           u32x4 (&w0)[TN], u32x4 (&x1)[TM], u32x4 (&w1)[TN]) {
  if constexpr (TM == 1 && TN == 1)
    asm volatile(
        LS_R(0, 5, 0) LS_R(1, 4, 0) LS_R(2, 7, 0) LS_R(3, 6, 0) LS_W
        : LS_O(w0[0]), LS_O(x0[0]), LS_O(w1[0]), LS_O(x1[0])
        : "v"(xa0), "v"(wa0), "v"(xa1), "v"(wa1) : "memory");
  else if constexpr (TM == 1 && TN == 2)
    asm volatile(
        LS_R(0, 7, 0) LS_R(1, 7, 2048) LS_R(2, 6, 0) LS_R(3, 9, 0) LS_R(4, 9, 2048) LS_R(5, 8, 0) LS_W
        : LS_O(w0[0]), LS_O(w0[1]), LS_O(x0[0]), LS_O(w1[0]), LS_O(w1[1]), LS_O(x1[0])
        : "v"(xa0), "v"(wa0), "v"(xa1), "v"(wa1) : "memory");
  else if constexpr (TM == 2 && TN == 1)
    asm volatile(
        LS_R(0, 7, 0) LS_R(1, 6, 0) LS_R(2, 6, 2048) LS_R(3, 9, 0) LS_R(4, 8, 0) LS_R(5, 8, 2048) LS_W
        : LS_O(w0[0]), LS_O(x0[0]), LS_O(x0[1]), LS_O(w1[0]), LS_O(x1[0]), LS_O(x1[1])
        : "v"(xa0), "v"(wa0), "v"(xa1), "v"(wa1) : "memory");
  else if constexpr (TM == 2 && TN == 2)
    asm volatile(
        LS_R(0, 9, 0) LS_R(1, 9, 2048) LS_R(2, 8, 0) LS_R(3, 8, 2048) LS_R(4, 11, 0) LS_R(5, 11, 2048) LS_R(6, 10, 0)
        LS_R(7, 10, 2048) LS_W
        : LS_O(w0[0]), LS_O(w0[1]), LS_O(x0[0]), LS_O(x0[1]), LS_O(w1[0]), LS_O(w1[1]), LS_O(x1[0]), LS_O(x1[1])
        : "v"(xa0), "v"(wa0), "v"(xa1), "v"(wa1) : "memory");
  else if constexpr (TM == 4 && TN == 1)
    asm volatile(
        LS_R(0, 11, 0) LS_R(1, 10, 0) LS_R(2, 10, 2048) LS_R(3, 10, 4096) LS_R(4, 10, 6144) LS_R(5, 13, 0)
        LS_R(6, 12, 0) LS_R(7, 12, 2048) LS_R(8, 12, 4096) LS_R(9, 12, 6144) LS_W
        : LS_O(w0[0]), LS_O(x0[0]), LS_O(x0[1]), LS_O(x0[2]), LS_O(x0[3]), LS_O(w1[0]), LS_O(x1[0]), LS_O(x1[1]),
        LS_O(x1[2]), LS_O(x1[3])
        : "v"(xa0), "v"(wa0), "v"(xa1), "v"(wa1) : "memory");
}
#undef LS_R
#undef LS_W
#undef LS_O

// Tile order: groups of up to eight tile rows; inside a group, the tiles of one column of tiles
// (they share the weight panel) get workgroup ids that are 8 apart, i.e. the same XCD, next to
// each other in time, so that a weight line comes from memory once for them.
template <class TL, int EPI, bool ONCE>
__global__ void __launch_bounds__(WAVES * 64, 2)
k_gemm_tiled(const float* __restrict__ A, const float* __restrict__ W, int M, int N, int K, float* __restrict__ out, int tiles_m,
             int tiles_n, RopeAppend rp) {
  constexpr int NS = TL::NS, F = TL::F, KS = TL::KS, TM = TL::TM, TN = TL::TN, WN = TL::WN, BM = TL::BM, BN = TL::BN;
  constexpr bool GLU = EPI == TILED_SWIGLU;
  constexpr int NCOLS = GLU ? BN / 2 : BN;
  constexpr int KB = ROWB / 4;  // elements of a row in one k-step
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  typedef __attribute__((address_space(3))) void lds_void;
  const int panels = (tiles_n + 7) >> 3, q = blockIdx.x >> 3;
  const int g = q / (8 * panels), gm = min(8, tiles_m - 8 * g), qg = q - g * 8 * panels;
  const int tm = 8 * g + qg % gm, tn = qg / gm * 8 + (blockIdx.x & 7);
  if (tn >= tiles_n) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN, l16 = lane & 15, lq = lane >> 4;
  const int m0 = tm * BM, n0 = tn * NCOLS;
  const int nk = (K + KB - 1) / KB;
  const bool ragged = K % KB != 0;  // the last k-step is only half there (K is a multiple of KB / 2)
  const int t0 = (int)((long)blockIdx.y * nk / gridDim.y), t1 = (int)((long)(blockIdx.y + 1) * nk / gridDim.y);
  const int n = t1 - t0, ng = (n + KS - 1) / KS;  // k-steps, and groups of KS of them
  // ONCE: no other workgroup reads these weights.  Their fills are non-temporal, and the k-steps
  // are visited in cyclic order from a start of the tile's own: with rows a power of two apart
  // (hidden sizes 4096, 8192) workgroups in lock step would all ask the same memory channels.
  int kc = ONCE && !ragged ? t0 + tn % n : t0;
  auto next_k = [&]() {
    const int k = kc++;
    if (ONCE && kc == t1) kc = t0;
    return k;
  };

  auto weight_row = [&](int r) -> int {
    if constexpr (GLU) {  // a wavefront's fragments: TN / 2 of gate rows, then the up rows of the same columns
      const int jj = (r >> 4) % TN, f = n0 + r / (16 * TN) * (8 * TN) + (jj % (TN / 2)) * 16 + (r & 15);
      return (jj >= TN / 2 ? N : 0) + min(f, N - 1);
    } else {
      return min(n0 + r, N - 1);
    }
  };
  // This wavefront's fills: instructions wave, wave + 8, ... of a k-step's (activation rows first, eight
  // rows each).  Lane l supplies physical chunk l%8 of row l/8: byte offsets from the operand, both
  // below 4 GB.  Where their number is no multiple of the wavefronts', some have one less to wait
  // for; letting them fill the last rows once more instead stalls the CU's cache on lines that are
  // on their way already (32 x 64 tiles, 32 rows of the 13B QKV: 39 us against 32).
  unsigned off[F];
#pragma unroll
  for (int i = 0; i < F; ++i) {
    const int in = min(wave + WAVES * i, TL::NFILL - 1);
    const int row = in * 8 + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
    const int grow = in < BM / 8 ? min(m0 + row, M - 1) : weight_row(row - BM);
    off[i] = (unsigned)((size_t)grow * K * 4) + c * 16;
  }
  auto fill = [&](int sub, int kt) {
    const size_t kofs = (size_t)kt * ROWB;
    if (ragged && kt == nk - 1) {
      // the last fill of all; chunks 4..7 lie past the end of the row: the lanes that fill them
      // fetch chunks 0..3 instead (never read by a wavefront)
#pragma unroll
      for (int i = 0; i < F; ++i) {
        const int in = min(wave + WAVES * i, TL::NFILL - 1);
        off[i] -= ((((lane >> 2) & 1) ^ (in & 1)) != 0) ? 64u : 0u;
      }
    }
#pragma unroll
    for (int i = 0; i < F; ++i) {
      const int in = wave + WAVES * i;
      lds_void* to = (lds_void*)(smem + sub * TL::SUB + in * 1024);
      if ((i + 1) * WAVES <= BM / 8 || (i * WAVES < BM / 8 && in < BM / 8))
        __builtin_amdgcn_global_load_lds((const void*)((const char*)A + kofs + off[i]), to, 16, 0, 0);
      else if ((i + 1) * WAVES <= TL::NFILL || in < TL::NFILL)
        __builtin_amdgcn_global_load_lds((const void*)((const char*)W + kofs + off[i]), to, 16, 0, ONCE ? 2 : 0);
    }
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // this lane's fragment reads: row lane%16 of a 16-row block, chunk lane/16 (first half of the
  // k-step) or 4 + lane/16 (second)
  const unsigned lds0 = (unsigned)(size_t)(lds_void*)smem;
  const unsigned c0 = (unsigned)((lq ^ ((l16 >> 1) & 7)) << 4), c1 = c0 ^ 64;
  const unsigned xb = lds0 + (wm * 16 * TM + l16) * ROWB, wb = lds0 + BM * ROWB + (wn * 16 * TN + l16) * ROWB;

  // the fills of group g (of the last group only what there is: waits for it count nothing as young)
  auto fill_group = [&](int slot, int g) {
#pragma unroll
    for (int s = 0; s < KS; ++s)
      if (KS == 1 || g * KS + s < n) fill(slot * KS + s, next_k());
  };
#pragma unroll
  for (int p = 0; p < NS - 1; ++p)
    if (p < ng) fill_group(p, p);
  int slot = 0, fslot = NS - 1;
  for (int g = 0; g < ng; ++g) {
    asm volatile("" ::: "memory");
    // own fills of this group have landed: those of the NS - 2 groups after it may still be on their way
    if (g + NS - 1 < ng || (KS == 1 && g + NS - 1 == ng)) {
      if (TL::NFILL % WAVES == 0 || wave < TL::NFILL % WAVES) __builtin_amdgcn_s_waitcnt(waitcnt_vm((NS - 2) * KS * F));
      else __builtin_amdgcn_s_waitcnt(waitcnt_vm((NS - 2) * KS * (F - 1)));
    } else {
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int t = g * KS + s;
      if (KS > 1 && t >= n) break;
      const unsigned so = (slot * KS + s) * TL::SUB;
      u32x4 x0[TM], w0[TN], x1[TM], w1[TN];
      read_frags<TM, TN>(xb + so + c0, wb + so + c0, xb + so + c1, wb + so + c1, x0, w0, x1, w1);
      mma<TM, TN>(acc, w0, x0);
      if (s == 0 && g + NS - 1 < ng) fill_group(fslot, g + NS - 1);  // issued while the matrix pipe works on the first half
      if (!ragged || t0 + t != nk - 1) mma<TM, TN>(acc, w1, x1);  // see above
    }
    slot = slot + 1 == NS ? 0 : slot + 1;
    fslot = fslot + 1 == NS ? 0 : fslot + 1;
  }

  // ---- epilogue.  N is a multiple of 16: a 16-column fragment is inside the matrix or outside.
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + (wm * TM + i) * 16 + l16;
    if (m >= M) continue;
    if constexpr (EPI == TILED_SWIGLU) {
#pragma unroll
      for (int j = 0; j < TN / 2; ++j) {
        const int col = n0 + wn * 8 * TN + j * 16 + 4 * lq;
        f32x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = silu_f(acc[i][j][r]) * acc[i][j + TN / 2][r];
        if (col < N) *reinterpret_cast<f32x4*>(out + (size_t)m * N + col) = v;
      }
    } else if constexpr (EPI == TILED_ROPE) {
      const int pos = rp.row_pos[m], seq = rp.row_seq[m];
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int col = n0 + (wn * TN + j) * 16 + 4 * lq;
        if (col >= N) continue;
        const int head = col / rp.hd, dd = col - head * rp.hd;
        const bool is_q = head < rp.hq, is_v = head >= rp.hq + rp.hkv;
        f32x4 v = acc[i][j];
        if (!is_v && pos >= 0) {  // pairs (2p, 2p + 1)
          const f32x4 c = *reinterpret_cast<const f32x4*>(rp.cs + ((size_t)pos * (rp.hd >> 1) + (dd >> 1)) * 2);
          v = f32x4{v[0] * c[0] - v[1] * c[1], v[0] * c[1] + v[1] * c[0], v[2] * c[2] - v[3] * c[3], v[2] * c[3] + v[3] * c[2]};
        }
        if (is_q) {
          *reinterpret_cast<f32x4*>(out + (size_t)m * N + col) = v;
        } else if (pos >= 0) {  // a row whose sequence has no room left appends nothing
          float* cache = (float*)(is_v ? rp.vc : rp.kc);
          const int kh = is_v ? head - rp.hq - rp.hkv : head - rp.hq;
          *reinterpret_cast<f32x4*>(cache + (((size_t)seq * rp.hkv + kh) * rp.max_seq + pos) * rp.hd + dd) = v;
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int col = n0 + (wn * TN + j) * 16 + 4 * lq;
        if (col < N) *reinterpret_cast<f32x4*>(out + ((EPI == TILED_PART ? (size_t)blockIdx.y * M : 0) + m) * N + col) = acc[i][j];
      }
    }
  }
}

template <class TL, int EPI>
void launch_tile(const TiledPlan& p, const float* A, const float* W, int M, int N, int K, float* out, const RopeAppend& rp,
                 hipStream_t st) {
  const int ncols = EPI == TILED_SWIGLU ? TL::BN / 2 : TL::BN;
  const int tiles_m = (M + TL::BM - 1) / TL::BM, tiles_n = (N + ncols - 1) / ncols;
  const dim3 grid((unsigned)((tiles_n + 7) / 8 * 8 * tiles_m), (unsigned)p.splits);
  // partial tiles have their sums in another kernel: the operator is more than one launch, which
  // the runtime's start/stop events of one kernel cannot time
  auto launch = [&](auto kernel) {
    if (EPI == TILED_PART) hipLaunchKernelGGL(kernel, grid, dim3(WAVES * 64), TL::SMEM, st, A, W, M, N, K, out, tiles_m, tiles_n, rp);
    else launch_kernel(kernel, grid, dim3(WAVES * 64), TL::SMEM, st, A, W, M, N, K, out, tiles_m, tiles_n, rp);
  };
  if (tiles_m == 1) {  // nobody else reads these weights
    static std::atomic<uint64_t> lds_allowed{0};
    allow_dynamic_lds((const void*)k_gemm_tiled<TL, EPI, true>, TL::SMEM, lds_allowed);
    launch(k_gemm_tiled<TL, EPI, true>);
  } else {
    static std::atomic<uint64_t> lds_allowed{0};
    allow_dynamic_lds((const void*)k_gemm_tiled<TL, EPI, false>, TL::SMEM, lds_allowed);
    launch(k_gemm_tiled<TL, EPI, false>);
  }
}

template <int EPI>
bool launch_epi(const TiledPlan& p, const float* A, const float* W, int M, int N, int K, float* out, const RopeAppend& rp,
                hipStream_t st) {
#define LS_TILE(bm_, bn_, wm_, tm_, tn_, glu_)                                \
  if constexpr (EPI != TILED_SWIGLU || glu_)                                  \
    if (p.bm == bm_ && p.bn == bn_) {                                         \
      launch_tile<Tile<wm_, tm_, tn_>, EPI>(p, A, W, M, N, K, out, rp, st);   \
      return true;                                                            \
    }
  LS_TILED_F32(LS_TILE)
#undef LS_TILE
  return false;
}

}  // namespace

bool launch_gemm_tiled_f32(int epi, const TiledPlan& p, const void* A, const void* W, int M, int N, int K, void* out,
                           const RopeAppend& rope, hipStream_t st) {
  const float *a = (const float*)A, *w = (const float*)W;
  float* o = (float*)out;
  switch (epi) {
    case TILED_PART: return launch_epi<TILED_PART>(p, a, w, M, N, K, o, rope, st);
    case TILED_STORE: return launch_epi<TILED_STORE>(p, a, w, M, N, K, o, rope, st);
    case TILED_SWIGLU: return launch_epi<TILED_SWIGLU>(p, a, w, M, N, K, o, rope, st);
    case TILED_ROPE: return launch_epi<TILED_ROPE>(p, a, w, M, N, K, o, rope, st);
  }
  return false;
}

}  // namespace ls
