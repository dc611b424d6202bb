// fp32 causal attention for the prompt pass, on v_mfma_f32_16x16x4_f32 (head_dim 64 or 128).
//
// One 256-thread workgroup handles 64 query rows of one (sequence, query head), 16 per wavefront,
// and walks the keys in tiles of 32 that pass through LDS; the next tile is on its way in registers
// while the current one is worked on.  As in the bf16 kernel both products are computed transposed, so
// that softmax state is per lane: S^T[key][q] = K Q^T leaves lane (q = lane%16, group lane/16) with keys
// 4*(lane/16) .. +3 of a 16-key block, and those four probabilities are, one by one, the B operands of
// four O^T[d][q] += V^T P^T instructions whose k index runs over the keys {e, 4 + e, 8 + e, 12 + e}.
// For the score product a lane's 16-byte piece of a row holds four dimensions, one per instruction
// (both operands agree which; a sum does not care in what order it is taken).
//
// Rows lie 132 (or 68) floats apart in LDS: rows of a 16-row operand read start 4 banks apart and rows
// 4 apart, which the transposed V reads touch together, 16 banks apart (counters: a fifth of the LDS cycles
// are conflicts, at 13 % of the time in LDS).
//
// Bound by latency at the lengths fp32 is used for (two sequences of 131..190 tokens, 32 heads: 192
// workgroups).  One wavefront per (row, head) that visited the keys one after the other took 300 us
// there.
//
// A masked key's probability is zero, but zero times an infinite or NaN value is NaN: where a tile that
// some row of the workgroup sees in part holds such a value, its value product is done on vector FMAs
// over the visible keys only, so that no row is touched by keys behind it.
#include "kernels.hpp"
#include "device_util.hpp"

namespace ls {

namespace {

constexpr int BQ = 64, BKV = 32;

template <int HD>
__global__ void __launch_bounds__(256)
k_attn_prefill_f32(const float* __restrict__ qkv, int qkv_stride, const float* __restrict__ kc, const float* __restrict__ vc,
                   const int32_t* __restrict__ cu, int hq, int hkv, int max_seq, float* __restrict__ out, int nq) {
  constexpr int ROW = HD + 4;                // floats between two rows in LDS
  constexpr int PIECES = BKV * HD / 4 / 256;  // 16-byte pieces of a tile per thread and operand
  constexpr int C = HD / 16;
  __shared__ __attribute__((aligned(16))) float ks[BKV * ROW], vs[BKV * ROW];
  __shared__ int odd[4];  // wavefront w loaded an infinite or NaN value of the tile
  const int qi = blockIdx.x % nq, h = (blockIdx.x / nq) % hq, b = blockIdx.x / (nq * hq), kh = h / (hq / hkv);
  const int row0 = cu[b], len = cu[b + 1] - row0;
  const int qt = (len + BQ - 1) / BQ - 1 - qi;  // longest tiles first
  if (qt < 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, lq = lane >> 4;
  const int q0 = qt * BQ + wave * 16, qpos = q0 + l16;
  const float* kb = kc + ((size_t)b * hkv + kh) * max_seq * HD;
  const float* vb = vc + ((size_t)b * hkv + kh) * max_seq * HD;
  const float* qr = qkv + (size_t)(row0 + min(qpos, len - 1)) * qkv_stride + (size_t)h * HD;  // rows past the end are discarded
  f32x4 qf[C];
#pragma unroll
  for (int c = 0; c < C; ++c) qf[c] = *reinterpret_cast<const f32x4*>(qr + c * 16 + lq * 4);

  f32x4 o[C];
#pragma unroll
  for (int c = 0; c < C; ++c) o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;                    // l_run: this lane's share of the row sum
  const float cexp = 1.4426950408889634f / sqrtf((float)HD);  // score -> exponent of 2

  f32x4 kr[PIECES], vr[PIECES];
  auto load = [&](int t0) {
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
      const int p = tid + 256 * i, key = min(t0 + p / (HD / 4), len - 1);  // rows at or past the end are never read
      kr[i] = *reinterpret_cast<const f32x4*>(kb + (size_t)key * HD + (p % (HD / 4)) * 4);
      vr[i] = *reinterpret_cast<const f32x4*>(vb + (size_t)key * HD + (p % (HD / 4)) * 4);
    }
  };
  const int ntk = (min(qt * BQ + BQ, len) + BKV - 1) / BKV;
  load(0);
  for (int t = 0; t < ntk; ++t) {
    const int t0 = t * BKV;
    __syncthreads();  // everyone is done with the previous tile
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
      const int p = tid + 256 * i, at = p / (HD / 4) * ROW + (p % (HD / 4)) * 4;
      *reinterpret_cast<f32x4*>(ks + at) = kr[i];
      *reinterpret_cast<f32x4*>(vs + at) = vr[i];
    }
    const bool part_seen = t0 + BKV - 1 > qt * BQ;  // workgroup-uniform
    if (part_seen) {
      float nul = 0.f;  // NaN from an infinity or NaN on
#pragma unroll
      for (int i = 0; i < PIECES; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) nul = fmaf(vr[i][e], 0.f, nul);
      const bool any = __builtin_amdgcn_ballot_w64(!(nul == 0.f)) != 0;
      if (lane == 0) odd[wave] = any;
    }
    __syncthreads();
    const bool by_key = part_seen && (odd[0] | odd[1] | odd[2] | odd[3]);
    if (t + 1 < ntk) load(t0 + BKV);
    if (t0 > q0 + 15) continue;  // above all rows of this wavefront
    f32x4 s[2];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      s[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const f32x4 kf = *reinterpret_cast<const f32x4*>(ks + (kt * 16 + l16) * ROW + c * 16 + lq * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[kt] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[e], qf[c][e], s[kt], 0, 0, 0);
      }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int key = t0 + kt * 16 + 4 * lq + e;
        s[kt][e] = key > qpos ? -INFINITY : s[kt][e];
        mx = fmaxf(mx, s[kt][e]);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m_run, mx);  // finite from the first tile on: key 0 is visible
    const float corr = __builtin_amdgcn_exp2f((m_run - m_new) * cexp);
    l_run *= corr;
#pragma unroll
    for (int c = 0; c < C; ++c) o[c] *= corr;
    m_run = m_new;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s[kt][e] = __builtin_amdgcn_exp2f((s[kt][e] - m_new) * cexp);
        l_run += s[kt][e];
      }
    if (by_key) {
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          for (int g = 0; g < 4; ++g) {
            const int key = kt * 16 + 4 * g + e;
            const float p = __shfl(s[kt][e], 16 * g + l16);
            if (t0 + key <= qpos) {
#pragma unroll
              for (int c = 0; c < C; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) o[c][r] = fmaf(p, vs[key * ROW + c * 16 + 4 * lq + r], o[c][r]);
            }
          }
      continue;
    }
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int c = 0; c < C; ++c)
          o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vs[(kt * 16 + 4 * lq + e) * ROW + c * 16 + l16], s[kt][e], o[c], 0, 0, 0);
  }
  float l = l_run + __shfl_xor(l_run, 16);
  l += __shfl_xor(l, 32);
  const float inv = 1.0f / l;
  if (qpos < len) {
    float* orow = out + (size_t)(row0 + qpos) * ((size_t)hq * HD) + (size_t)h * HD;
#pragma unroll
    for (int c = 0; c < C; ++c) *reinterpret_cast<f32x4*>(orow + c * 16 + 4 * lq) = o[c] * inv;
  }
}

}  // namespace

bool attn_prefill_f32_supported(int hq, int hkv, int hd) { return (hd == 128 || hd == 64) && hq % hkv == 0; }

void launch_attn_prefill_f32(const void* qkv, int qkv_stride, const void* kc, const void* vc, const int32_t* cu_seqlens,
                             int batch, int max_len, int hq, int hkv, int hd, int max_seq, void* out, hipStream_t st) {
  if (batch <= 0 || max_len <= 0) return;
  const int nq = (max_len + BQ - 1) / BQ;
  const dim3 grid((unsigned)nq * hq * batch);
  if (hd == 128)
    k_attn_prefill_f32<128><<<grid, 256, 0, st>>>((const float*)qkv, qkv_stride, (const float*)kc, (const float*)vc, cu_seqlens,
                                                  hq, hkv, max_seq, (float*)out, nq);
  else
    k_attn_prefill_f32<64><<<grid, 256, 0, st>>>((const float*)qkv, qkv_stride, (const float*)kc, (const float*)vc, cu_seqlens,
                                                 hq, hkv, max_seq, (float*)out, nq);
}

}  // namespace ls
