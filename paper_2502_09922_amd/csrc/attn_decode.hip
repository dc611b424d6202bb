// Decode attention (bf16 and fp32), fused with RoPE and the KV-cache append of the new row: one
// query row per sequence against its KV cache (GQA aware).
//
// The step's q, k, v are read un-rotated from the projection output.  q is rotated in
// registers; the new key is rotated, rounded to storage type and written to the cache row `pos`
// together with the new value by wave 0, which also feeds them to its own softmax state
// straight from registers -- no wavefront of this kernel reads cache row `pos`, so there is
// no ordering problem between that store and the streaming loads.
//
// Bound by streaming the cache out of HBM once per step, so: one workgroup per (sequence,
// kv head) reads that head's keys and values exactly once for all G = Hq/Hkv query heads
// that share it.  Its NW wavefronts split the context into contiguous ranges (split-KV
// inside the workgroup).  A 16-byte-per-lane load instruction fetches 64/LPK consecutive
// cache rows (LPK = head_dim/8 lanes per key, whole rows, 1 KB contiguous).  Each lane
// keeps the partial dot product of its 8 dimensions, a butterfly over the LPK lanes of a key
// completes the score, and every key slot runs its own online softmax (running max and sum)
// so that no cross-slot traffic is needed inside the loop.  Slots are merged by shuffles,
// wavefronts through LDS in wave order: the result does not depend on timing.
//
// One sequence of 3000 keys on 32 heads is 32 workgroups on 256 CUs; there contexts are also cut into
// chunks that are workgroups of their own, merged in chunk order by a second kernel (see
// chunks_for).
#include "kernels.hpp"
#include "device_util.hpp"

#include <algorithm>

namespace ls {

namespace {

// wavefronts per workgroup = context splits.  With one query head per kv head the kernel
// needs few registers and 16 wavefronts with one load per operand in flight stream best
// (measured inside the stage, 7B and 13B shapes); wider groups keep 8 wavefronts.
#ifndef LS_ATTN_NW
#define LS_ATTN_NW 8
#endif
#ifndef LS_ATTN_NW1
#define LS_ATTN_NW1 16
#endif
#ifndef LS_ATTN_U
#define LS_ATTN_U 1
#endif
// fp32 rows are twice as wide per lane: 8 wavefronts
template <class T> constexpr int waves_for(int g) { return g == 1 && sizeof(T) == 2 ? LS_ATTN_NW1 : LS_ATTN_NW; }

constexpr int PART_HDR = 4;  // floats in front of a chunk's partial result: maximum, sum

template <class T> struct Vec8;
template <> struct Vec8<bf16> { typedef bf16x8 type; };
template <> struct Vec8<float> { typedef float type __attribute__((ext_vector_type(8))); };

template <class T, int HD, int G>
// with one query head per kv head the kernel fits 64 registers: eight wavefronts per SIMD, two
// 16-wavefront workgroups per CU
__global__ void __launch_bounds__(waves_for<T>(G) * 64, (G == 1 && sizeof(T) == 2 ? 8 : 1))
k_attn_decode(const int32_t* __restrict__ row_pos, const int32_t* __restrict__ row_seq, int heads_first, int qkv_stride,
              const T* __restrict__ qkv, const float2* __restrict__ cs, T* __restrict__ kc, T* __restrict__ vc, int hq, int hkv, int max_seq,
              T* __restrict__ out, float* __restrict__ part, int nchunk, int chunk_keys) {
  typedef typename Vec8<T>::type T8;
  constexpr int NW = waves_for<T>(G);
  constexpr int LPK = HD / 8;     // lanes per key
  constexpr int KPI = 64 / LPK;   // keys per load instruction
  constexpr int U = (G >= 4 && sizeof(T) == 2) ? 2 : LS_ATTN_U;  // load instructions in flight per operand
  __shared__ float sm_m[NW][G], sm_l[NW][G];
  __shared__ float sm_acc[NW][G][HD];
  const int r = heads_first ? blockIdx.y : blockIdx.x, kh = heads_first ? blockIdx.x : blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int pos = row_pos[r];
  if (pos < 0) return;  // a sequence with no room left: whole workgroup leaves together
  const int seq = row_seq[r];
  // keys 0..pos-1 come from the cache, key `pos` from this step's row; this workgroup's chunk of the
  // former (the last chunk is open-ended), the latter goes with chunk 0
  const int c0 = blockIdx.z * chunk_keys, ctx = (int)blockIdx.z == nchunk - 1 ? pos : min(c0 + chunk_keys, pos);
  if (c0 >= pos && blockIdx.z) return;
  const int slot = lane / LPK, dl = lane % LPK;
  T* kb = kc + ((size_t)seq * hkv + kh) * max_seq * HD;
  T* vb = vc + ((size_t)seq * hkv + kh) * max_seq * HD;
  const T* row = qkv + (size_t)r * qkv_stride;

  // cos/sin of this lane's four pairs (dims 8 dl + 2i, 8 dl + 2i + 1) at position pos
  float2 rot[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) rot[i] = cs[(size_t)pos * (HD / 2) + dl * 4 + i];

  // this lane's 8 dimensions of every query head of the group: rotated, pre-scaled
  const float scale = 1.0f / sqrtf((float)HD);
  float q[G][8];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const T8 qv = *reinterpret_cast<const T8*>(row + (size_t)(kh * G + g) * HD + dl * 8);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float u0 = to_f(qv[2 * i]), u1 = to_f(qv[2 * i + 1]);
      q[g][2 * i] = (sizeof(T) == 4 ? turn0(u0, u1, rot[i]) : u0 * rot[i].x - u1 * rot[i].y) * scale;
      q[g][2 * i + 1] = (sizeof(T) == 4 ? turn1(u0, u1, rot[i]) : u0 * rot[i].y + u1 * rot[i].x) * scale;
    }
  }

  // contiguous key range of this wave, a multiple of KPI keys
  const int chunk = ((ctx - c0 + NW * KPI - 1) / (NW * KPI)) * KPI;
  const int k_begin = c0 + wave * chunk, k_end = min(k_begin + chunk, ctx);

  float m[G], l[G], acc[G][8];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m[g] = -INFINITY;
    l[g] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[g][e] = 0.f;
  }

  // fp32: which of two products is rounded is written down, as k_step_small_f32 does the same sums
#define LS_WEIGH(p, v, s) (sizeof(T) == 4 ? fmaf(p, v, s) : (s) + (p) * (v))
  // one key per slot: scores of the G heads, then the slot's online-softmax update
#define LS_KEY_UPDATE(kx, vx, valid)                                                         \
  _Pragma("unroll") for (int g = 0; g < G; ++g) {                                            \
    float s_ = 0.f;                                                                          \
    _Pragma("unroll") for (int e = 0; e < 8; ++e) s_ = fmaf(q[g][e], kx[e], s_);             \
    _Pragma("unroll") for (int off = LPK / 2; off; off >>= 1) s_ += __shfl_xor(s_, off);     \
    s_ = (valid) ? s_ : -INFINITY;                                                           \
    const float mn_ = fmaxf(m[g], s_);                                                       \
    /* mn_ == -inf only while this slot has seen no valid key: keep everything at zero (a     \
       NaN score, which no maximum shows, must not count as none) */                         \
    const float corr_ = (mn_ == -INFINITY) ? 1.f : __expf(m[g] - mn_);                       \
    const float p_ = (s_ == -INFINITY) ? 0.f : __expf(s_ - mn_);                             \
    l[g] = l[g] * corr_ + p_;                                                                \
    _Pragma("unroll") for (int e = 0; e < 8; ++e) acc[g][e] = LS_WEIGH(p_, vx[e], acc[g][e] * corr_); \
    m[g] = mn_;                                                                              \
  }

  // fp32: a slot without a key takes zeros for its values, as zero times an infinite one is NaN.  (bf16,
  // whose registers are full, multiplies what it loaded: NaN instead of an infinity there.)
#define LS_SEEN(v) (sizeof(T) == 4 && !valid ? 0.f : (v))

  // the new row first (wave 0): rotate k, round both to storage type, append to the cache, attend to
  // it.  Done before the cache stream so that the rotation table is dead inside the loop.
  if (wave == 0 && blockIdx.z == 0) {
    const T8 kn = *reinterpret_cast<const T8*>(row + (size_t)(hq + kh) * HD + dl * 8);
    const T8 vn = *reinterpret_cast<const T8*>(row + (size_t)(hq + hkv + kh) * HD + dl * 8);
    T8 kr;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float u0 = to_f(kn[2 * i]), u1 = to_f(kn[2 * i + 1]);
      kr[2 * i] = from_f<T>(sizeof(T) == 4 ? turn0(u0, u1, rot[i]) : u0 * rot[i].x - u1 * rot[i].y);
      kr[2 * i + 1] = from_f<T>(sizeof(T) == 4 ? turn1(u0, u1, rot[i]) : u0 * rot[i].y + u1 * rot[i].x);
    }
    if (slot == 0) {
      *reinterpret_cast<T8*>(kb + (size_t)pos * HD + dl * 8) = kr;
      *reinterpret_cast<T8*>(vb + (size_t)pos * HD + dl * 8) = vn;
    }
    const bool valid = slot == 0;
    float kx[8], vx[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) { kx[e] = to_f(kr[e]); vx[e] = LS_SEEN(to_f(vn[e])); }
    LS_KEY_UPDATE(kx, vx, valid)
  }
  // the cache is read once per step: non-temporal loads.  The cache stream is software pipelined: the loads of the next group of U*KPI keys are
  // in flight while the current group is folded into the softmax state; a load whose keys
  // all lie past the wave's range is not issued at all
#define LS_LOAD_GROUP(buf, j0_)                                                               \
  _Pragma("unroll") for (int u = 0; u < U; ++u) {                                             \
    if ((j0_) + u * KPI < k_end) {                                                            \
      const int key_ = min((j0_) + u * KPI + slot, ctx - 1); /* clamped: a valid cache row */ \
      kf[buf][u] = __builtin_nontemporal_load(reinterpret_cast<const T8*>(kb + (size_t)key_ * HD + dl * 8)); \
      vf[buf][u] = __builtin_nontemporal_load(reinterpret_cast<const T8*>(vb + (size_t)key_ * HD + dl * 8)); \
    }                                                                                         \
  }
#define LS_FOLD_GROUP(buf, j0_)                                                               \
  _Pragma("unroll") for (int u = 0; u < U; ++u) {                                             \
    if ((j0_) + u * KPI < k_end) {                                                            \
      const bool valid = ((j0_) + u * KPI + slot) < k_end;                                    \
      float kx[8], vx[8];                                                                     \
      _Pragma("unroll") for (int e = 0; e < 8; ++e) {                                         \
        kx[e] = to_f(kf[buf][u][e]);                                                          \
        vx[e] = LS_SEEN(to_f(vf[buf][u][e]));                                                 \
      }                                                                                       \
      LS_KEY_UPDATE(kx, vx, valid)                                                            \
    }                                                                                         \
  }
  {
    constexpr int STEP = KPI * U;
    T8 kf[2][U], vf[2][U];
    LS_LOAD_GROUP(0, k_begin)
    for (int j0 = k_begin; j0 < k_end; j0 += 2 * STEP) {
      LS_LOAD_GROUP(1, j0 + STEP)
      LS_FOLD_GROUP(0, j0)
      LS_LOAD_GROUP(0, j0 + 2 * STEP)
      LS_FOLD_GROUP(1, j0 + STEP)
    }
  }
#undef LS_LOAD_GROUP
#undef LS_FOLD_GROUP

#undef LS_SEEN
#undef LS_KEY_UPDATE
#undef LS_WEIGH

  // merge the key slots of the wave (lanes that hold the same dimensions)
#pragma unroll
  for (int g = 0; g < G; ++g) {
    float mw = m[g];
#pragma unroll
    for (int off = LPK; off < 64; off <<= 1) mw = fmaxf(mw, __shfl_xor(mw, off));
    const float w = (m[g] == -INFINITY) ? 0.f : __expf(m[g] - mw);
    float lw = l[g] * w;
#pragma unroll
    for (int off = LPK; off < 64; off <<= 1) lw += __shfl_xor(lw, off);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float a = acc[g][e] * w;
#pragma unroll
      for (int off = LPK; off < 64; off <<= 1) a += __shfl_xor(a, off);
      acc[g][e] = a;
    }
    if (lane < LPK) {
      if (dl == 0) { sm_m[wave][g] = mw; sm_l[wave][g] = lw; }
#pragma unroll
      for (int e = 0; e < 8; ++e) sm_acc[wave][g][dl * 8 + e] = acc[g][e];
    }
  }
  __syncthreads();

  // merge the waves in wave order and write the output row
  for (int i = threadIdx.x; i < G * HD; i += NW * 64) {
    const int g = i / HD, d = i % HD;
    float mm = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) mm = fmaxf(mm, sm_m[w][g]);
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float wt = (sm_m[w][g] == -INFINITY) ? 0.f : __expf(sm_m[w][g] - mm);
      num += sm_acc[w][g][d] * wt;
      den += sm_l[w][g] * wt;
    }
    if (nchunk == 1 || pos <= chunk_keys) {  // the sequence is this one chunk
      out[(size_t)r * (hkv * G * HD) + (size_t)(kh * G + g) * HD + d] = from_f<T>(num / den);
    } else {
      float* pp = part + ((((size_t)r * hkv + kh) * G + g) * nchunk + blockIdx.z) * (HD + PART_HDR);
      pp[PART_HDR + d] = num;
      if (d == 0) { pp[0] = mm; pp[1] = den; }
    }
  }
}

// Second pass for sequences longer than one chunk: the chunks' partial results in chunk order.
template <class T, int HD>
__global__ void __launch_bounds__(HD)
k_attn_decode_merge(const float* __restrict__ part, const int32_t* __restrict__ row_pos, int hq, int nchunk, int chunk_keys,
                    T* __restrict__ out) {
  const int r = blockIdx.x, h = blockIdx.y, d = threadIdx.x;
  const int pos = row_pos[r];
  if (pos <= chunk_keys) return;  // no room left, or the first pass wrote this row
  const int nch = min((pos + chunk_keys - 1) / chunk_keys, nchunk);
  const float* p0 = part + ((size_t)r * hq + h) * nchunk * (HD + PART_HDR);
  float mm = -INFINITY;
#pragma unroll 8
  for (int c = 0; c < nch; ++c) mm = fmaxf(mm, p0[c * (HD + PART_HDR)]);
  float num = 0.f, den = 0.f;
#pragma unroll 8
  for (int c = 0; c < nch; ++c) {
    const float* p = p0 + c * (HD + PART_HDR);
    const float wt = __expf(p[0] - mm);  // every chunk holds a visible key: finite
    num += p[PART_HDR + d] * wt;
    den += p[1] * wt;
  }
  out[((size_t)r * hq + h) * HD + d] = from_f<T>(num / den);
}

// Chunks per sequence.  One workgroup per (sequence, kv head) reads its cache at about 50 GB/s, 10 us
// for 1000 keys of 128 bf16 dimensions, so 128 of them saturate HBM and contexts are cut only
// below that, up to WG_TARGET workgroups in all.  The chunks' start and the merge kernel cost about
// 5 us: below CHUNK_FROM keys nothing is gained (8 x 32 heads, 600 keys: two chunks 20 us, one 15.4;
// 32 heads, 3000 keys: 35 us whole, 11 + 4.7 in 16 chunks; a target of 256 workgroups does the same).
constexpr int WG_TARGET = 512, CHUNK_MIN = 128, CHUNK_FROM = 640;
int chunks_for(int rows, int hkv, int max_keys) {
  const int base = rows * hkv;
  if (base >= 128 || max_keys < CHUNK_FROM) return 1;
  return std::max(1, std::min((WG_TARGET + base - 1) / base, max_keys / CHUNK_MIN));
}

struct Args {
  const void* qkv;
  int qkv_stride;
  const float* cs;
  void *kc, *vc;
  const int32_t *row_seq, *row_pos;
  int rows, hkv, max_seq;
  void* out;
  float* part;
  int nchunk, chunk_keys;
};

template <class T, int HD, int G>
void launch_g(const Args& a, hipStream_t st) {
  const AttnGrid g = attn_decode_grid(a.rows, a.hkv, a.nchunk);
  k_attn_decode<T, HD, G><<<dim3(g.x, g.y, g.z), waves_for<T>(G) * 64, 0, st>>>(
      a.row_pos, a.row_seq, g.heads_first, a.qkv_stride, (const T*)a.qkv, (const float2*)a.cs, (T*)a.kc, (T*)a.vc, a.hkv * G, a.hkv, a.max_seq,
      (T*)a.out, a.part, a.nchunk, a.chunk_keys);
  if (a.nchunk > 1)
    k_attn_decode_merge<T, HD><<<dim3(a.rows, a.hkv * G), HD, 0, st>>>(a.part, a.row_pos, a.hkv * G, a.nchunk, a.chunk_keys, (T*)a.out);
}

template <class T, int HD>
void launch_hd(int g, const Args& a, hipStream_t st) {
  switch (g) {
    case 1: launch_g<T, HD, 1>(a, st); break;
    case 2: launch_g<T, HD, 2>(a, st); break;
    case 4: launch_g<T, HD, 4>(a, st); break;
    case 8: launch_g<T, HD, 8>(a, st); break;
  }
}

}  // namespace

bool attn_decode_supported(int hq, int hkv, int hd) {
  const int g = hq / hkv;
  return (hd == 128 || hd == 64) && (g == 1 || g == 2 || g == 4 || g == 8);
}

int attn_decode_chunks(int rows, int hkv, int max_keys) { return chunks_for(rows, hkv, max_keys); }

// covers every launch of at most `rows` sequences: rows * hkv * chunks stays below WG_TARGET + 128
size_t attn_decode_scratch_bytes(int hq, int hkv, int hd, int max_keys) {
  if (!attn_decode_supported(hq, hkv, hd) || max_keys < CHUNK_FROM) return 0;
  return (size_t)(WG_TARGET + 128) * (hq / hkv) * (hd + PART_HDR) * sizeof(float);
}

void launch_attn_decode(uint32_t dt, const void* qkv, int qkv_stride, const float* cs_table, void* kc, void* vc,
                        const int32_t* row_seq, const int32_t* row_pos, int rows, int hq, int hkv, int hd,
                        int max_seq, void* out, hipStream_t st, int max_keys, float* scratch, size_t scratch_bytes) {
  if (rows <= 0) return;
  const int g = hq / hkv, keys = std::min(std::max(max_keys, 1), max_seq);
  int nchunk = chunks_for(rows, hkv, keys);
  int chunk_keys = (keys + nchunk - 1) / nchunk;
  if (nchunk > 1 && (!scratch || (size_t)rows * hq * nchunk * (hd + PART_HDR) * sizeof(float) > scratch_bytes)) nchunk = 1;
  if (nchunk == 1) chunk_keys = max_seq;
  const Args a = {qkv, qkv_stride, cs_table, kc, vc, row_seq, row_pos, rows, hkv, max_seq, out, scratch, nchunk, chunk_keys};
  if (dt == F32) {
    if (hd == 128) launch_hd<float, 128>(g, a, st);
    else launch_hd<float, 64>(g, a, st);
  } else {
    if (hd == 128) launch_hd<bf16, 128>(g, a, st);
    else launch_hd<bf16, 64>(g, a, st);
  }
}

}  // namespace ls
