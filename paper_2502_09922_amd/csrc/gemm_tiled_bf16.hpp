// bf16 GEMM for some dozen to some thousand rows: C[M,N] = A[M,K] W[N,K]^T with fp32 accumulation.
//
// What it is for.  The 256 x 256 tiles of k_gemm_mfma leave most of the chip idle when the output has few of them
// (311 rows x 4096 columns: 32 tiles on 256 CUs), and the weight-streaming kernels hold all rows of the call in one
// fragment set.  Here a workgroup (one per CU) owns a tile of 32..256 rows x 48..256 weight rows, chosen per launch
// (gemm_tiled_plan) so that the tiles, times the number of ways K is cut, fill the chip.
//
// What bounds it: the lines a CU can have on their way.  A CU's cache holds 32 KB and keeps room there for every line
// that was asked for; lines come back in order, so lines that hit L2 wait behind those that do not, and all
// workgroups of an XCD ask for a line at the same time.  Measured with nothing but fills: 120 GB/s a CU if everything
// hits L2, 54 if it comes from memory, 48..60 in any mixture and however many bytes are asked for ahead.  So
// (1) a tile is chosen by the lines it brings in a k-step, rows plus weight rows, and rows past the end of the
// call are not asked for; (2) wavefronts that ask for more than there is room for stand still, therefore four
// wavefronts only fill and the others only multiply: before, eight did both, and a k-step took as long as its fills
// and its products one after the other.  Workgroups that only touch the weights' lines ahead of the others, an XCD's
// share each, raised the fills to 100 GB/s by themselves but gained 0..9 % here and cost far more where they drifted
// too far ahead; touching them from the same CU takes the room of the fills.
//
// Data path: both operands are K-contiguous; a k-step is 128 bytes of every row.  Rows go from global memory straight
// into LDS (global_load_lds_dwordx4) into a ring of NS stages, 16-byte chunks XOR-swizzled by (row/2)&7 as in
// k_gemm_mfma, so that the 16 rows a quarter-wave reads fall into different banks.  One barrier per k-step hands the
// stages over: behind barrier t k-step t is there and the slot of k-step t - 1 takes the fills of t + NS - 1.
// Multiplying wavefronts read half a k-step ahead of their products.
//
// Measured between events (4 us of each are the events'), cold weights, 7B layer, QKV / O / gate-up / down (the kernel
// before): 45 rows 22 / 12 / 33 / 21 us (26 / 12 / 38 / 21), 311 rows 44 / 24 / 62 / 41 (55 / 23 / 84 / 43), 1024 rows
// 88 / 40 / 166 / 83 (137 / 56 / 230 / 105; 1.1 PFLOP/s); 13B layer, 100 rows QKV 43 (49); 70B layer, 64 rows QKV and
// gate-up 40 and 143 (45 and 153).
//
// Weight fragments are the A operand, activations the B operand: a lane of a result holds row
// m = lane%16 of its tile and four consecutive columns n = 4*(lane/16) .. +3.
//
// One source file per epilogue includes this one: together they take a minute and a half to compile.
#pragma once
#include "kernels.hpp"
#include "device_util.hpp"

namespace ls {

namespace {

typedef __attribute__((address_space(3))) unsigned char lds_char;
typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(3))) u32x4* lds_vec;

constexpr int FILLERS = 4;  // wavefronts that fill (two: 4..10 % slower)

// Tile of 16 WM TM rows x 16 WN TN weight rows, multiplying wavefronts WM x WN, ring as deep as LDS allows (at most
// six stages: no tile gained from more).
template <int TM, int TN, int WM, int WN>
struct Tile {
  static constexpr int CONSUMERS = WM * WN, WAVES = CONSUMERS + FILLERS;
  static constexpr int BM = 16 * WM * TM, BN = 16 * WN * TN, SIZE = (BM + BN) * 128;
  static constexpr int FIT = 160 * 1024 / SIZE, NS = FIT > 6 ? 6 : FIT, SMEM = NS * SIZE;
  static constexpr int F = ((BM + BN) / 8 + FILLERS - 1) / FILLERS;  // fills of a wavefront in a k-step, eight rows each
  // Two k-steps are filled at a time, the two lines of a row that lie side by side one after the other, where six stages
  // are all that fits and what is on its way is enough with two stages less: 161..213 lines.  Two layers of a step: 13B,
  // 100 rows, whose QKV takes 128 x 64, 664 -> 658 us; 70B, 64 rows, whose O and down take 64 x 128, 725 -> 718.  With
  // fewer lines a k-step the two stages are missed, also with eight or ten of them (48 x 48 and 48 x 64, 45 rows: +2.5 %
  // of the pass); with more lines there is no sixth stage.
  static constexpr bool PAIRS = NS == 6 && FIT < 8;
  static_assert(NS >= 2 && (NS - 2) * F < 64, "");
};

// Tile order: groups of up to eight tile rows; inside a group, the tiles of one column of tiles
// (they share the weight panel) get workgroup ids that are 8 apart, i.e. the same XCD, next to
// each other in time, so that a weight line comes from memory once for them.
template <int TM, int TN, int WM, int WN, int EPI>
__global__ void __launch_bounds__(64 * (WM * WN + FILLERS), (WM * WN + FILLERS + 3) / 4)
k_gemm_tiled(const bf16* __restrict__ A, const bf16* __restrict__ W, int M, int N, int K, void* __restrict__ outv, int tiles_m,
             int tiles_n, RopeAppend rp) {
  typedef Tile<TM, TN, WM, WN> TL;
  constexpr bool GLU = EPI == TILED_SWIGLU;
  constexpr int NS = TL::NS, F = TL::F, BM = TL::BM, BN = TL::BN, NCOLS = GLU ? BN / 2 : BN;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int panels = (tiles_n + 7) >> 3, q = blockIdx.x >> 3;
  const int g = q / (8 * panels), gm = min(8, tiles_m - 8 * g), qg = q - g * 8 * panels;
  const int tm = 8 * g + qg % gm, tn = qg / gm * 8 + (blockIdx.x & 7);
  if (tn >= tiles_n) return;
  const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m0 = tm * BM, n0 = tn * NCOLS;
  const int nk = (K + 63) / 64;
  const bool ragged = K % 64 != 0;  // the last k-step is only half there (K is a multiple of 32)
  const int t0 = (int)((long)blockIdx.y * nk / gridDim.y), t1 = (int)((long)(blockIdx.y + 1) * nk / gridDim.y);
  const int n = t1 - t0;

  if (wave >= TL::CONSUMERS) {
    // ---- fills: instructions p, p + 4, ... of those that bring rows of the call and of the matrix
    const int p = wave - TL::CONSUMERS;
    const int la = (min(M - m0, BM) + 7) >> 3;  // of A's rows
    // ... of W's: SwiGLU takes them by blocks of 16 columns, gate and up rows of a block (two instructions each)
    const int lw = GLU ? 4 * (min(N - n0, NCOLS) >> 4) : min(N - n0, NCOLS) >> 3;
    const int f = (la + lw - p + FILLERS - 1) / FILLERS;  // of this wavefront
    // Lane l supplies physical chunk l%8 of row l/8: byte offsets from the operand, both below 4 GB.
    unsigned off[F];
    int dst[F];
#pragma unroll
    for (int i = 0; i < F; ++i) {
      const int v = p + FILLERS * i, u = v - la;
      int in;  // eight rows of the stage
      size_t row;
      if (u < 0) {
        in = v;
        row = (size_t)min(m0 + 8 * in + (lane >> 3), M - 1);
      } else if constexpr (GLU) {  // a wavefront's fragments: TN / 2 of gate rows, then the up rows of the same columns
        const int block = u >> 2, up = (u >> 1) & 1, half = u & 1;
        in = BM / 8 + 2 * (block / (TN / 2) * TN + block % (TN / 2) + up * (TN / 2)) + half;
        row = (size_t)(up ? N : 0) + min(n0 + 16 * block + 8 * half + (lane >> 3), N - 1);
      } else {
        in = BM / 8 + u;
        row = (size_t)min(n0 + 8 * u + (lane >> 3), N - 1);
      }
      const int r = 8 * in + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
      off[i] = (unsigned)(row * K * 2) + c * 16;
      dst[i] = in * 1024;
    }
    // ONCE (one tile row): no other workgroup reads these weights.  Their fills are non-temporal, and the k-steps are
    // visited in cyclic order from a start of the tile's own: with rows a power of two apart (hidden sizes 4096,
    // 8192) workgroups in lock step would all ask the same memory channels.  The tiles of an XCD, eight apart, start eight
    // k-steps from each other, or two where the call's rows take more than five sixths of the XCD's 4 MB of L2: what one of
    // them brought of the rows has to be there when the next one asks.  Eight k-steps apart / two, down projections: 13B, 104
    // rows (2.7 MB) 31.2 / 30.6 us, 128 (3.4) 34.2 / 32.9, 160 (4.2) 43.9 / 35.1, 250 rows 61 / 42; 7B, 128 rows (2.7) 23.6 / 23.7,
    // 250 rows (5.3) 40 / 32; 70B, 72 rows (3.9) 81.7 / 81.9, 120 (6.6) 107.7 / 90.9, 224 (12.3) 178 / 109.  Gate-up of 70B, 64 rows
    // (1.0) 139.3 / 139.9, 96 (1.5) 142.0 / 141.6, 192 (3.0) 231 / 237, 208 (3.25) 230 / 235, 224 (3.5) 234 / 230.
    auto run = [&](auto once_, auto count_) {
      constexpr bool ONCE = decltype(once_)::value;
      constexpr int C = decltype(count_)::value;  // f, or -1: not known
      const unsigned bytes = 2u * M * K;  // below 4 GB
      const int lag = bytes > (4u << 20) / 6 * 5 ? 2 : 8, start = ((tn >> 3) * lag + (tn & 7)) % n;
      int kc = ONCE && !ragged ? (TL::PAIRS ? start & ~1 : start) : 0, slot = 0;
      auto fill = [&]() {
        const size_t ko = (size_t)(t0 + kc) * 128;
        const char *a = (const char*)A + ko, *w = (const char*)W + ko;
        const bool half = ragged && t0 + kc == nk - 1;
        if (++kc == n) kc = 0;
        unsigned char* to = smem + slot * TL::SIZE;
#pragma unroll
        for (int i = 0; i < F; ++i) {
          if (C >= 0 ? i >= C : i >= f) continue;
          unsigned o = off[i];
          // chunks 4..7 of a last half k-step lie past the end of the row: the lanes that fill them fetch chunks
          // 0..3 instead (never used)
          if (half) o -= (((lane >> 2) & 1) ^ ((dst[i] >> 10) & 1)) != 0 ? 64u : 0u;
          if (p + FILLERS * i < la) __builtin_amdgcn_global_load_lds((const void*)(a + o), (lds_void*)(to + dst[i]), 16, 0, 0);
          else __builtin_amdgcn_global_load_lds((const void*)(w + o), (lds_void*)(to + dst[i]), 16, 0, ONCE ? 2 : 0);
        }
        slot = slot + 1 == NS ? 0 : slot + 1;
      };
      auto fill2 = [&](bool two) {  // the next k-step and the one behind it
        if (!two) {
          fill();
          return;
        }
        const int ka = t0 + kc;
        if (++kc == n) kc = 0;
        const int kb = t0 + kc;
        if (++kc == n) kc = 0;
        unsigned char* to = smem + slot * TL::SIZE;
        const bool ha = ragged && ka == nk - 1, hb = ragged && kb == nk - 1;
        auto line = [&](int i, int k, bool half, unsigned char* at) {
          unsigned o = off[i];
          if (half) o -= (((lane >> 2) & 1) ^ ((dst[i] >> 10) & 1)) != 0 ? 64u : 0u;
          const size_t ko = (size_t)k * 128;
          if (p + FILLERS * i < la) __builtin_amdgcn_global_load_lds((const void*)((const char*)A + ko + o), (lds_void*)(at + dst[i]), 16, 0, 0);
          else __builtin_amdgcn_global_load_lds((const void*)((const char*)W + ko + o), (lds_void*)(at + dst[i]), 16, 0, ONCE ? 2 : 0);
        };
#pragma unroll
        for (int i = 0; i < F; ++i) {
          if (C >= 0 ? i >= C : i >= f) continue;
          line(i, ka, ha, to);
          line(i, kb, hb, to + TL::SIZE);
        }
        slot = slot + 2 == NS ? 0 : slot + 2;
      };
      if constexpr (TL::PAIRS) {
        for (int s = 0; s < NS; s += 2)
          if (s < n) fill2(s + 1 < n);
        wait_vm((min(n, NS) - min(n, 2)) * f);
        __builtin_amdgcn_s_barrier();  // 0
        int t = 1;
        for (; t + NS < n; t += 2) {
          __builtin_amdgcn_s_barrier();  // t: came with t - 1
          if constexpr (C >= 0) __builtin_amdgcn_s_waitcnt(waitcnt_vm((NS - 4) * C));
          else wait_vm((NS - 4) * f);
          __builtin_amdgcn_s_barrier();  // t + 1
          fill2(true);                   // of k-steps t + NS - 1 and t + NS, into the slots of t - 1 and t
        }
        for (; t < n; ++t) {
          const bool even = !(t & 1);
          if (even) wait_vm((min(n, t - 2 + NS) - min(n, t + 2)) * f);
          __builtin_amdgcn_s_barrier();  // t
          if (even && t + NS - 2 < n) fill2(t + NS - 1 < n);
        }
      } else {
        for (int s = 0; s < NS; ++s)
          if (s < n) fill();
        wait_vm((min(n, NS) - 1) * f);
        __builtin_amdgcn_s_barrier();  // 0
        int t = 1;
        for (; t + NS - 1 < n; ++t) {
          if constexpr (C >= 0) __builtin_amdgcn_s_waitcnt(waitcnt_vm((NS - 2) * C));
          else wait_vm((NS - 2) * f);
          __builtin_amdgcn_s_barrier();  // t
          fill();                        // of k-step t + NS - 1, into the slot of t - 1
        }
        for (; t < n; ++t) {
          wait_vm((n - t - 1) * f);
          __builtin_amdgcn_s_barrier();  // t
        }
      }
      __builtin_amdgcn_s_barrier();  // n
    };
    const std::integral_constant<int, -1> any{};
    const std::integral_constant<int, F> most{};
    const std::integral_constant<int, F - 1> less{};
    const std::true_type yes{};
    const std::false_type no{};
    if (tiles_m == 1) {
      if (f == F) run(yes, most); else if (f == F - 1) run(yes, less); else run(yes, any);
    } else {
      if (f == F) run(no, most); else if (f == F - 1) run(no, less); else run(no, any);
    }
    return;
  }

  // ---- products
  const int wm = wave / WN, wn = wave % WN;
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // RoPE: sequence and position of this lane's rows, before the products where the registers last: 256 for a wavefront, with
  // more than eight wavefronts 168 (256 x 192, 8 + 4 of them: 40 registers spilled if loaded before)
  constexpr bool ROPE = EPI == TILED_ROPE, EARLY = 4 * TM * TN + 8 * (TM + TN) + 2 * TM <= (TL::WAVES > 8 ? 168 : 200);
  int pos[ROPE ? TM : 1], seq[ROPE ? TM : 1];
  auto positions = [&]() {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = min(m0 + (wm * TM + i) * 16 + l16, M - 1);
      pos[i] = rp.row_pos[m];
      seq[i] = rp.row_seq[m];
    }
  };
  if constexpr (ROPE && EARLY) positions();
  // this lane's fragment reads: row lane%16 of a 16-row block, chunk lane/16 (first half of the
  // k-step) or 4 + lane/16 (second)
  const unsigned lds0 = (unsigned)(size_t)(lds_char*)smem;
  const unsigned c0 = (unsigned)((lq ^ ((l16 >> 1) & 7)) << 4);
  const unsigned xa = lds0 + (wm * 16 * TM + l16) * 128 + c0, wa = lds0 + (BM + wn * 16 * TN + l16) * 128 + c0;
  const unsigned xb = xa ^ 64, wb = wa ^ 64;
  auto read = [&](unsigned xs, unsigned ws, u32x4 (&x)[TM], u32x4 (&w)[TN]) {
#pragma unroll
    for (int j = 0; j < TN; ++j) w[j] = ((lds_vec)(size_t)ws)[128 * j];
#pragma unroll
    for (int i = 0; i < TM; ++i) x[i] = ((lds_vec)(size_t)xs)[128 * i];
  };
  auto multiply = [&](const u32x4 (&x)[TM], const u32x4 (&w)[TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[j]), __builtin_bit_cast(bf16x8, x[i]),
                                                            acc[i][j], 0, 0, 0);
  };
  {
    const int full = n - (ragged && t1 == nk);  // whole k-steps
    u32x4 x0[TM], w0[TN], x1[TM], w1[TN];
    unsigned so = 0;
    slot_barrier<false>();  // 0
    read(xa, wa, x0, w0);
    for (int t = 0; t < full; ++t) {
      read(xb + so, wb + so, x1, w1);
      multiply(x0, w0);
      __builtin_amdgcn_sched_barrier(0);
      slot_barrier<true>();  // t + 1
      so = so + TL::SIZE == NS * TL::SIZE ? 0 : so + TL::SIZE;
      read(xa + so, wa + so, x0, w0);  // behind the last k-step: not used
      multiply(x1, w1);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (full < n) {
      multiply(x0, w0);
      slot_barrier<false>();
    }
  }

  // ---- epilogue.  N is a multiple of 16: a 16-column fragment is inside the matrix or outside.
  auto put = [](bf16* p, f32x4 v) {
    bf16x4 y;
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = from_f<bf16>(v[r]);
    *reinterpret_cast<bf16x4*>(p) = y;
  };
  // RoPE: a row block's (cos, sin) are on their way while the block before is stored; one after the other each block waits
  // for memory (7B, 311 rows, four row blocks and more: 2.4 us of 48).  256 x 192 has no registers for two blocks' (24 spilled).
  constexpr bool AHEAD = 4 * TM * TN + 10 * TN + 2 * TM <= (TL::WAVES > 8 ? 150 : 220);
  int head[ROPE ? TN : 1], dim[ROPE ? TN : 1];
  f32x4 cs[AHEAD ? 2 : 1][ROPE ? TN : 1];
  auto turns = [&](int i, f32x4 (&to)[ROPE ? TN : 1]) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
      to[j] = *reinterpret_cast<const f32x4*>(rp.cs + ((size_t)max(pos[i], 0) * (rp.hd >> 1) + (dim[j] >> 1)) * 2);
  };
  if constexpr (ROPE) {
    if (!EARLY) positions();
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = min(n0 + (wn * TN + j) * 16 + 4 * lq, N - 4);
      head[j] = col / rp.hd;
      dim[j] = col - head[j] * rp.hd;
    }
    turns(0, cs[0]);
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + (wm * TM + i) * 16 + l16;
    if (!ROPE && m >= M) continue;
    if constexpr (GLU) {
#pragma unroll
      for (int j = 0; j < TN / 2; ++j) {
        const int col = n0 + wn * 8 * TN + j * 16 + 4 * lq;
        f32x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = silu_f(acc[i][j][r]) * acc[i][j + TN / 2][r];
        if (col < N) put((bf16*)outv + (size_t)m * N + col, v);
      }
    } else if constexpr (EPI == TILED_ROPE) {
      if (!AHEAD && i) turns(i, cs[0]);
      if (AHEAD && i + 1 < TM) turns(i + 1, cs[(i + 1) & 1]);
      if (m >= M) continue;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int col = n0 + (wn * TN + j) * 16 + 4 * lq;
        if (col >= N) continue;
        const bool is_q = head[j] < rp.hq, is_v = head[j] >= rp.hq + rp.hkv;
        f32x4 v = acc[i][j];
        if (!is_v && pos[i] >= 0) {
          // the projection's output in storage type is what turns (pairs 2p, 2p + 1)
          const f32x4 c = cs[AHEAD ? i & 1 : 0][j];
          const float u0 = to_f(from_f<bf16>(v[0])), u1 = to_f(from_f<bf16>(v[1])), u2 = to_f(from_f<bf16>(v[2])), u3 = to_f(from_f<bf16>(v[3]));
          v = f32x4{u0 * c[0] - u1 * c[1], u0 * c[1] + u1 * c[0], u2 * c[2] - u3 * c[3], u2 * c[3] + u3 * c[2]};
        }
        if (is_q) {
          put((bf16*)outv + (size_t)m * N + col, v);
        } else if (pos[i] >= 0) {  // a row whose sequence has no room left appends nothing
          bf16* cache = is_v ? rp.vc : rp.kc;
          const int kh = is_v ? head[j] - rp.hq - rp.hkv : head[j] - rp.hq;
          put(cache + (((size_t)seq[i] * rp.hkv + kh) * rp.max_seq + pos[i]) * rp.hd + dim[j], v);
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int col = n0 + (wn * TN + j) * 16 + 4 * lq;
        if (col >= N) continue;
        if constexpr (EPI == TILED_PART)
          *reinterpret_cast<f32x4*>((float*)outv + ((size_t)blockIdx.y * M + m) * N + col) = acc[i][j];
        else
          put((bf16*)outv + (size_t)m * N + col, acc[i][j]);
      }
    }
  }
}

template <int TM, int TN, int WM, int WN, int EPI>
void launch_tile(const TiledPlan& p, const void* A, const void* W, int M, int N, int K, void* out, const RopeAppend& rp,
                 hipStream_t st) {
  typedef Tile<TM, TN, WM, WN> TL;
  const int ncols = EPI == TILED_SWIGLU ? TL::BN / 2 : TL::BN;
  const int tiles_m = (M + TL::BM - 1) / TL::BM, tiles_n = (N + ncols - 1) / ncols;
  const dim3 grid((unsigned)((tiles_n + 7) / 8 * 8 * tiles_m), (unsigned)p.splits), block(64 * TL::WAVES);
  static std::atomic<uint64_t> lds_allowed{0};
  allow_dynamic_lds((const void*)k_gemm_tiled<TM, TN, WM, WN, EPI>, TL::SMEM, lds_allowed);
  const bf16 *a = (const bf16*)A, *w = (const bf16*)W;
  // partial tiles have their sums in another kernel: the operator is more than one launch, which
  // the runtime's start/stop events of one kernel cannot time
  if (EPI == TILED_PART) hipLaunchKernelGGL((k_gemm_tiled<TM, TN, WM, WN, EPI>), grid, block, TL::SMEM, st, a, w, M, N, K, out, tiles_m, tiles_n, rp);
  else launch_kernel(k_gemm_tiled<TM, TN, WM, WN, EPI>, grid, block, TL::SMEM, st, a, w, M, N, K, out, tiles_m, tiles_n, rp);
}

template <int EPI>
bool launch_epi(const TiledPlan& p, const void* A, const void* W, int M, int N, int K, void* out, const RopeAppend& rp,
                hipStream_t st) {
#define LS_TILE(tm_, tn_, wm_, wn_, glu_)                                   \
  if constexpr (EPI != TILED_SWIGLU || glu_)                                \
    if (p.bm == 16 * wm_ * tm_ && p.bn == 16 * wn_ * tn_) {                 \
      launch_tile<tm_, tn_, wm_, wn_, EPI>(p, A, W, M, N, K, out, rp, st);  \
      return true;                                                          \
    }
  LS_TILED_BF16(LS_TILE)
#undef LS_TILE
  return false;
}

}  // namespace

}  // namespace ls
