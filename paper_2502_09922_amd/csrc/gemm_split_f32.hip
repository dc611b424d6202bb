// fp32 GEMM for some dozen rows and more: C[M,N] = A[M,K] W[N,K]^T as bf16 products of three-way split operands.
//
// Why: v_mfma_f32_16x16x4_f32 moves 4 k in 32 cycles; six bf16 instructions, which give the same 24 bits, move 32 k
// in 96.  What is left is the splitting (11 vector instructions per pair of values), and it is done where it
// is done once: the rows of A by a kernel of its own in front (k_parts, some microseconds), the rows of W by the one
// wavefront that multiplies with them.  Before, eight wavefronts of a 96 x 128 or 256 x 128 tile each split all the
// operands they read, 4 to 18 times the work, and a split by v_dot2 (7 instructions) takes the matrix unit's time:
// beside matrix instructions it runs at 24.6 cycles against 12 for any other vector instruction.
//
// Four wavefronts multiply, one per SIMD: all 16 TM rows of the tile times 16 TN weight rows of their own.  Four
// more only fill: LDS-direct loads into a ring of NS stages (parts of 16 TM rows, fp32 weights, of 32 k), because a
// wavefront that asks for more than the CU's cache has room for (about 32 KB on their way) stands still, and
// its matrix instructions with it.  One barrier a k-step hands the stages over.  The tile's rows are cut evenly
// (325 rows: 11 + 10 fragments of 16).  The parts lie in memory as LDS and the matrix instructions want them, 1 KB
// per fragment, part and k-step; weights lie in rows of 128 bytes, 16-byte chunks XOR-swizzled by (row/2)&7.
//
// Measured, 325 rows of the 7B shape, QKV / O / gate-up / down (before): 228 / 67 / 423 / 165 us (416 / 112 / 640 / 300);
// 512 rows of gate-up 534 (750), 100 rows 160 (258).  A k-step of a 176 x 128 tile takes 1.6 us, its matrix instructions
// 1.07; spreading the weights' splitting over more of them, and splitting the rows of A by wavefronts of the same
// workgroup instead of a kernel (1.8-2.4 us a k-step), gave nothing or less.
#include "kernels.hpp"
#include "device_util.hpp"

namespace ls {

namespace {

typedef __attribute__((address_space(3))) unsigned char lds_char;
typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(3))) u32x4* lds_vec;

constexpr int CONSUMERS = 4, FILLERS = 4;  // wavefronts
constexpr int CHUNK = 8;                    // k-steps of A that share a flag

// An fp32 value as the sum of three bf16 values, each the rest rounded to the nearest: of a value in [1, 2) the
// second is at most 2^-8, the third at most 2^-17 (a multiple of 2^-23), both of either sign.  (Henry, Tang,
// Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations",
// ARITH 2019.)  The sum is exact from 2^-102 on; of smaller values what lies below 2^-126 may be lost, as
// bf16 parts end there.  part[0..2][p]: the three parts of the pieces a and b of a row, two values per register.
__device__ __forceinline__ void split3(u32x4 a, u32x4 b, u32x4 (&part)[3]) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    float f0 = __uint_as_float(p < 2 ? a[2 * p] : b[2 * p - 4]), f1 = __uint_as_float(p < 2 ? a[2 * p + 1] : b[2 * p - 3]);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const unsigned h = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{f0, f1}), bf16x2));
      part[s][p] = h;
      f0 -= __uint_as_float(h << 16);
      f1 -= __uint_as_float(h & 0xffff0000u);
    }
    part[2][p] = __builtin_amdgcn_perm(__float_as_uint(f1), __float_as_uint(f0), 0x07060302);  // fits: the upper halves of both
  }
}

// Infinities, values that round to one and values whose products could overflow by their parts are multiplied in fp32.
constexpr float BIG = 0x1p63f;
__device__ __forceinline__ float largest(float big, u32x4 v) {
  const f32x4 f = __builtin_bit_cast(f32x4, v);
  big = fmaxf(fmaxf(fabsf(f[0]), fabsf(f[1])), big);
  return fmaxf(fmaxf(fabsf(f[2]), fabsf(f[3])), big);
}

// The parts of A: [k-step][fragment of 16 rows][part][lane][8].  Lane l holds of row l%16 the values 4 (l/16) .. +3 and
// 16 + 4 (l/16) .. +3 of the k-step; the weights are read alike, and a sum does not care in what order k
// is visited.  flags[fragment][k-step / CHUNK]: a value among them is BIG or more.
__global__ void __launch_bounds__(64 * CHUNK)
k_parts(const float* __restrict__ A, int M, int K, int frags, int chunks, unsigned char* __restrict__ parts,
        int* __restrict__ flags) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
  const int fr = blockIdx.x / chunks, kt = (blockIdx.x - fr * chunks) * CHUNK + (threadIdx.x >> 6), nk = (K + 31) / 32;
  float big = 0.f;
  if (kt < nk) {
    const float* r = A + (size_t)min(16 * fr + l16, M - 1) * K + kt * 32 + 4 * lq;  // rows past the end are never stored
    const u32x4 a = *reinterpret_cast<const u32x4*>(r);
    const u32x4 b = kt == nk - 1 && K % 32 ? u32x4{0, 0, 0, 0} : *reinterpret_cast<const u32x4*>(r + 16);
    big = largest(largest(0.f, a), b);
    u32x4 p[3];
    split3(a, b, p);
    unsigned char* o = parts + ((size_t)kt * frags + fr) * 3072 + lane * 16;
#pragma unroll
    for (int s = 0; s < 3; ++s) *reinterpret_cast<u32x4*>(o + s * 1024) = p[s];
  }
  const int any = __syncthreads_or(big >= BIG);
  if (threadIdx.x == 0) flags[blockIdx.x] = any;
}

// Tile of at most 16 TM rows x 64 TN weight rows; ring as deep as LDS allows (at most four stages).
template <int TM, int TN>
struct Stage {
  static constexpr int BN = 16 * CONSUMERS * TN;
  static constexpr int X = TM * 3 * 1024, SIZE = X + BN * 128, FIT = 160 * 1024 / SIZE, NS = FIT > 4 ? 4 : FIT, SMEM = NS * SIZE;
  static_assert(NS >= 3, "a stage being read and two on their way");
};

template <int TM, int TN, int EPI>
__global__ void __launch_bounds__(64 * (CONSUMERS + FILLERS), 2)
k_gemm_split(const float* __restrict__ A, const unsigned char* __restrict__ parts, const int* __restrict__ flags,
             const float* __restrict__ W, int M, int N, int K, float* __restrict__ out, int tiles_m, int tiles_n, int nf,
             RopeAppend rp) {
  typedef Stage<TM, TN> S;
  constexpr bool GLU = EPI == TILED_SWIGLU;
  constexpr int NS = S::NS, NCOLS = GLU ? S::BN / 2 : S::BN;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  // The tiles of one column of tiles, which share the weights, get workgroup ids that are 8 apart: the same XCD.
  const int q = blockIdx.x >> 3, tm = q % tiles_m, tn = q / tiles_m * 8 + (blockIdx.x & 7);
  if (tn >= tiles_n) return;
  const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int f0 = tm * nf, frags = (M + 15) >> 4, nfh = min(nf, frags - f0);  // fragments of this tile
  const int m0 = 16 * f0, n0 = tn * NCOLS;
  const int nk = (K + 31) / 32;
  const bool ragged = K % 32 != 0;  // the last k-step is only half there (K is a multiple of 16)
  const int t0 = (int)((long)blockIdx.y * nk / gridDim.y), t1 = (int)((long)(blockIdx.y + 1) * nk / gridDim.y);
  const int n = t1 - t0;
  auto weight_row = [&](int r) -> int {  // row r of the tile; SwiGLU: a fragment holds eight gate rows and the up rows of their columns
    if constexpr (GLU) return ((r & 8) ? N : 0) + min(n0 + (r >> 4) * 8 + (r & 7), N - 1);
    else return min(n0 + r, N - 1);
  };

  if (wave >= CONSUMERS) {
    // ---- fills: instructions p, p + FILLERS, ... of the stage's, 1 KB each
    const int p = wave - CONSUMERS;
    constexpr int FX = (3 * TM + FILLERS - 1) / FILLERS, FW = S::BN / 8 / FILLERS;
    unsigned wo[FW];  // byte offsets from W, below 4 GB: eight rows an instruction, lane l chunk l%8 of row l/8
#pragma unroll
    for (int i = 0; i < FW; ++i) {
      const int row = 8 * (p + FILLERS * i) + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
      wo[i] = (unsigned)((size_t)weight_row(row) * K * 4) + c * 16;
    }
    // chunks 4..7 of a last half k-step lie past the end of the row: the lanes that fill them fetch chunks 0..3
    // instead (never used)
    const unsigned back = (((lane >> 2) & 1) ^ (p & 1)) != 0 ? 64u : 0u;
    const int nx = (3 * nfh - p + FILLERS - 1) / FILLERS;  // of the parts: only the fragments there are
    int kt = t0, slot = 0;
    auto fill = [&]() {
      const unsigned char* x = parts + ((size_t)kt * frags + f0) * 3072 + p * 1024 + lane * 16;
      const char* w = (const char*)W + (size_t)kt * 128;
      const unsigned less = ragged && kt == nk - 1 ? back : 0u;
      unsigned char* to = smem + slot * S::SIZE + p * 1024;
#pragma unroll
      for (int i = 0; i < FW; ++i)
        __builtin_amdgcn_global_load_lds((const void*)(w + (wo[i] - less)), (lds_void*)(to + S::X + FILLERS * i * 1024), 16, 0, 0);
#pragma unroll
      for (int i = 0; i < FX; ++i)
        if (i < nx) __builtin_amdgcn_global_load_lds((const void*)(x + FILLERS * i * 1024), (lds_void*)(to + FILLERS * i * 1024), 16, 0, 0);
      ++kt;
      slot = slot + 1 == NS ? 0 : slot + 1;
    };
    for (int s = 0; s < NS; ++s)
      if (s < n) fill();
    for (int t = 0; t < n; ++t) {
      const int issued = min(n, t == 0 ? NS : NS + t - 1);
      wait_vm((issued - t - 1) * (FW + nx));
      __builtin_amdgcn_s_barrier();         // k-step t is there, k-step t - 1 has been read
      if (t > 0 && t + NS - 1 < n) fill();  // into the slot of t - 1
    }
    __builtin_amdgcn_s_barrier();
    return;
  }

  // ---- products
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const unsigned lds0 = (unsigned)(size_t)(lds_char*)smem;
  // a lane's raw pieces of a 16-row block of weights: row l16, chunk lq and 4 + lq
  const unsigned c0 = (unsigned)((lq ^ ((l16 >> 1) & 7)) << 4), wb = S::X + (wave * 16 * TN + l16) * 128;
  u32x4 wp[TN][3], ra[TN], rb[TN];
  float big = 0.f;
  auto read_weights = [&](unsigned stage) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      ra[j] = ((lds_vec)(size_t)(stage + wb + c0))[128 * j];
      rb[j] = ((lds_vec)(size_t)(stage + wb + (c0 ^ 64)))[128 * j];
    }
  };
  auto split_weights = [&](int t, u32x4 (&dst)[TN][3]) {
    big = 0.f;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      if (ragged && t0 + t == nk - 1) rb[j] = u32x4{0, 0, 0, 0};
      big = largest(largest(big, ra[j]), rb[j]);
      split3(ra[j], rb[j], dst[j]);
    }
  };
  constexpr int NP = (TM + 1) / 2;  // fragments are taken in pairs: 2 TN sums side by side hide an instruction's latency
  auto read_parts = [&](unsigned stage, int i, u32x4 (&x)[2][3]) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (2 * i + u < TM)
#pragma unroll
        for (int s = 0; s < 3; ++s) x[u][s] = ((lds_vec)(size_t)(stage + lane * 16))[(2 * i + u) * 192 + s * 64];
  };
  // All products but mid * lo, lo * mid and lo * lo, together at most 2^-24 of a product and of either sign, so that
  // sums of them do not drift.  (Parts cut off instead of rounded have the sign of their value: up to 7.8 x
  // 2^-24 of a product left out, all towards zero, and small products of one sign that a large sum swallows one by
  // one.)  Relative error against float64 at K = 11008, as here / fp32 instructions: 1.7e-6 / 1.9e-6 for
  // Gaussian operands, 0.9e-6 / 1.5e-6 for positive ones.  The bf16 instruction rounds to nearest like the fp32 one,
  // except that an accumulator smaller than the product loses what lies below the result's last bit, towards
  // minus infinity: results lie 0.7e-6 of their mean magnitude low.
  auto multiply = [&](int i, const u32x4 (&x)[2][3]) {
    constexpr int PW[6] = {2, 0, 1, 1, 0, 0}, PX[6] = {0, 2, 1, 0, 1, 0};  // smallest products first
#pragma unroll
    for (int p = 0; p < 6; ++p)
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (2 * i + u < TM)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[2 * i + u][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wp[j][PW[p]]),
                                                                        __builtin_bit_cast(bf16x8, x[u][PX[p]]), acc[2 * i + u][j], 0, 0, 0);
  };
  auto multiply_fp32 = [&](int t, int i) {  // from memory
    const int kt = t0 + t;
    const float* xr = A + (size_t)min(m0 + 16 * i + l16, M - 1) * K + kt * 32 + 4 * lq;
#pragma unroll 1
    for (int h = 0; h < (ragged && kt == nk - 1 ? 1 : 2); ++h) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(xr + 16 * h);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const f32x4 w = *reinterpret_cast<const f32x4*>(W + (size_t)weight_row((wave * TN + j) * 16 + l16) * K + kt * 32 + 4 * lq + 16 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[e], x[e], acc[i][j], 0, 0, 0);
      }
    }
  };
  bool odd;  // rows with values that the parts cannot hold: the whole tile in fp32
  {
    const int chunks = (nk + CHUNK - 1) / CHUNK;
    int any = 0;
    for (int i = lane; i < nfh * chunks; i += 64) any |= flags[f0 * chunks + i];
    odd = __builtin_amdgcn_ballot_w64(any != 0) != 0;
  }

  slot_barrier<false>();  // k-step 0 is there
  read_weights(lds0);
  split_weights(0, wp);
  u32x4 x[2][2][3];
  read_parts(lds0, 0, x[0]);
  int slot = 0, t = 0;
  for (; t < n; ++t) {
    if (odd || __builtin_amdgcn_ballot_w64(big >= BIG) != 0) break;
    const unsigned stage = lds0 + slot * S::SIZE;
    slot = slot + 1 == NS ? 0 : slot + 1;
    const unsigned next = lds0 + slot * S::SIZE;
    u32x4 wn[TN][3];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      // the reads of the next pair run under the products of this one
      if (i + 1 < NP) read_parts(stage, i + 1, x[(i + 1) & 1]);
      if (i == NP - 2) {
        slot_barrier<true>();  // this k-step is in registers; the next one is there (behind the last: not used)
        read_weights(next);
      }
      if (i == NP - 1) read_parts(next, 0, x[NP & 1]);
      __builtin_amdgcn_sched_barrier(0);
      multiply(i, x[i & 1]);
      if (i == NP - 1) split_weights(t + 1, wn);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr ((NP & 1) != 0)
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int s = 0; s < 3; ++s) x[0][u][s] = x[1][u][s];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int s = 0; s < 3; ++s) wp[j][s] = wn[j][s];
  }
  // From the first k-step with such a value on (weights), or throughout (rows).  A loop of its own behind the other: as a
  // branch inside it the registers of both would not fit (3 us a k-step instead of 1.7).  So the last bits of a row
  // may depend on the rows beside it.
  for (; t < n; ++t) {
#pragma unroll
    for (int i = 0; i < TM; ++i) multiply_fp32(t, i);
    slot_barrier<false>();
  }

  // ---- epilogue: a lane holds row m = lane%16 of a fragment and four consecutive columns 4*(lane/16) .. +3.
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + 16 * i + l16;
    if (i >= nfh || m >= M) continue;
    if constexpr (GLU) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {  // lanes 0..31 hold gate columns, lanes 32..63 the up columns of the same place
        f32x4 v = acc[i][j], u;
#pragma unroll
        for (int r = 0; r < 4; ++r) u[r] = __shfl_xor(v[r], 32);
        const int col = n0 + (wave * TN + j) * 8 + 4 * lq;
        if (lq < 2 && col < N) {
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = silu_f(v[r]) * u[r];
          *reinterpret_cast<f32x4*>(out + (size_t)m * N + col) = v;
        }
      }
    } else if constexpr (EPI == TILED_ROPE) {
      const int pos = rp.row_pos[m], seq = rp.row_seq[m];
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int col = n0 + (wave * TN + j) * 16 + 4 * lq;
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
        const int col = n0 + (wave * TN + j) * 16 + 4 * lq;
        if (col < N) *reinterpret_cast<f32x4*>(out + ((EPI == TILED_PART ? (size_t)blockIdx.y * M : 0) + m) * N + col) = acc[i][j];
      }
    }
  }
}

template <int TM, int TN, int EPI>
void launch_tile(const float* A, void* parts, const float* W, int M, int N, int K, int splits, float* out, const RopeAppend& rp,
                 hipStream_t st) {
  constexpr int ncols = EPI == TILED_SWIGLU ? Stage<TM, TN>::BN / 2 : Stage<TM, TN>::BN, smem = Stage<TM, TN>::SMEM;
  const int frags = (M + 15) / 16, tiles_m = (frags + TM - 1) / TM, nf = (frags + tiles_m - 1) / tiles_m;
  const int tiles_n = (N + ncols - 1) / ncols, nk = (K + 31) / 32, chunks = (nk + CHUNK - 1) / CHUNK;
  int* flags = (int*)((char*)parts + (size_t)frags * nk * 3072);
  hipLaunchKernelGGL(k_parts, dim3((unsigned)chunks * (unsigned)frags), dim3(64 * CHUNK), 0, st, A, M, K, frags, chunks,
                     (unsigned char*)parts, flags);
  static std::atomic<uint64_t> lds_allowed{0};
  allow_dynamic_lds((const void*)k_gemm_split<TM, TN, EPI>, smem, lds_allowed);
  hipLaunchKernelGGL((k_gemm_split<TM, TN, EPI>), dim3((unsigned)((tiles_n + 7) / 8 * 8 * tiles_m), (unsigned)splits),
                     dim3(64 * (CONSUMERS + FILLERS)), smem, st, A, (const unsigned char*)parts, flags, W, M, N, K, out, tiles_m,
                     tiles_n, nf, rp);
}

template <int TM, int TN>
bool launch_epi(int epi, const float* A, void* parts, const float* W, int M, int N, int K, int splits, float* out,
                const RopeAppend& rp, hipStream_t st) {
  switch (epi) {
    case TILED_PART: launch_tile<TM, TN, TILED_PART>(A, parts, W, M, N, K, splits, out, rp, st); return true;
    case TILED_STORE: launch_tile<TM, TN, TILED_STORE>(A, parts, W, M, N, K, splits, out, rp, st); return true;
    case TILED_SWIGLU: launch_tile<TM, TN, TILED_SWIGLU>(A, parts, W, M, N, K, splits, out, rp, st); return true;
    case TILED_ROPE: launch_tile<TM, TN, TILED_ROPE>(A, parts, W, M, N, K, splits, out, rp, st); return true;
  }
  return false;
}

}  // namespace

size_t gemm_split_parts_bytes(int M, int K) {
  const size_t frags = ((size_t)M + 15) / 16, nk = ((size_t)K + 31) / 32;
  return frags * nk * 3072 + frags * ((nk + CHUNK - 1) / CHUNK) * sizeof(int);
}

bool launch_gemm_split_f32(int epi, const TiledPlan& p, const void* A, void* parts, const void* W, int M, int N, int K, void* out,
                           const RopeAppend& rope, hipStream_t st) {
  const float *a = (const float*)A, *w = (const float*)W;
  float* o = (float*)out;
#define LS_TILE(bm_, bn_) \
  if (p.bm == bm_ && p.bn == bn_) return launch_epi<bm_ / 16, bn_ / 64>(epi, a, parts, w, M, N, K, p.splits, o, rope, st);
  LS_SPLIT_TILES(LS_TILE)
#undef LS_TILE
  return false;
}

}  // namespace ls
