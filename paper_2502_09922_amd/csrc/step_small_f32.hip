// A whole generation step of a small fp32 model in one launch: every layer, the LM head and the argmax.
//
// Such a step is a chain of a dozen kernels that each read a few hundred KB and take what a launch takes, 3 us on the device and
// as much on the host.  Here sixteen workgroups stay for the whole step and hand the activations over through memory: a value
// goes out as one 8-byte store, its upper half a tag that no earlier value of the place has carried, and every workgroup polls
// for the values it needs until they carry the tag.  No flag, no fence and no wait for a store stands between producer and
// consumer: 1.2 us from one phase to the next (256 values; with flags 1.8, with a counter that all add to and fences 5 to 9).
// What a phase multiplies with is asked for before its values are.  The tiny model (2 layers of 256 columns, one row, 40 keys):
// a step 43 -> 27 us on the device, the generation of 8 tokens behind a 32-token prompt 491 -> 317 us.  What bounds it now: of
// the 27 us eleven exchanges take 13, the attention's softmax and merges 1.3 a layer, a projection's sums 0.7 to 1.8.
//
// Sixteen: with 32 workgroups a step takes 23.5 us, with 16 of them 27.3, but all of a launch have to be on the chip together.
// A CU holds two (512 threads, at most 128 registers, at most 64 KB of LDS), the chip 512, which is 32 such launches at once,
// more than the device has hardware queues (24); what else runs there ends by itself.  A stream that may use fewer CUs than
// those of 24 launches gets the separate launches (small_step_room).  A poll is bounded all the same (POLLS, many seconds): a value
// that has not come by then reads as NaN.
//
// Where the places are.  They and the last step's tag have to outlast the step, which a workspace need not: each stage has a
// part of a static array of its device for as long as it lives (take_small_step_places), and no other stage's calls write there.
//
// Who writes a place again.  Every phase has places of its own, written again a layer later.  Every workgroup has columns of
// the projections (small_step_shape), so whoever has gathered a phase's values knows that every workgroup is past the phases
// before it; a launch ends before the next begins, which goes on with tags behind the last one's.
//
// Sums are those of k_gemm_rows_f32, k_rows, k_attn_decode and k_argmax in their order: a step gives the same bits either way.
#include "kernels.hpp"
#include "device_util.hpp"

#include <algorithm>
#include <atomic>
#include <mutex>

namespace ls {

namespace {

typedef unsigned long long u64;

constexpr int NT = 512, NW = NT / 64, WGS = 16, GW = WGS * NW;
constexpr int POLLS = 1 << 25;
constexpr int ATTN_NW = NW;  // ranges a context is cut into, as in k_attn_decode<float>
constexpr int AMAX_NW = 16;  // ... wavefronts of k_argmax

__device__ __forceinline__ void put(u64* p, unsigned tag, float v) {
  __hip_atomic_store(p, (u64)tag << 32 | __builtin_bit_cast(unsigned, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// dst[e] = the value at place(e), e < n, as soon as it carries `tag`, U of them to a thread at a time.  For all threads of the
// workgroup; a barrier has to follow.
template <int U, class Place>
__device__ __forceinline__ void gather(int n, unsigned tag, float* dst, Place place) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  for (int e0 = 0; e0 < n; e0 += NT * U) {
    u64 v[U];
    bool all = false;
    for (int spin = 0; spin < POLLS && !all; ++spin) {
      bool have = true;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * NT + tid;
        v[u] = e < n ? __hip_atomic_load(place(e), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : (u64)tag << 32;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) have = have && (unsigned)(v[u] >> 32) == tag;
      all = __all(have);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * NT + tid;
      if (e < n) dst[e] = (unsigned)(v[u] >> 32) == tag ? __builtin_bit_cast(float, (unsigned)v[u]) : __builtin_nanf("");
    }
  }
}
__device__ __forceinline__ void gather(const u64* src, int n, unsigned tag, float* dst) {
  gather<2>(n, tag, dst, [&](int e) { return src + e; });
}

// One projection: this wavefront's columns n = first, first + GW, ..., S of them (GLU: S gate rows and the up rows of the same
// columns) at a time, U pieces of 256 of their weights in flight.  `ready` makes the R rows of xs (LDS, K floats each), behind
// the request for the first weights.  NORM: the rows' norm is what is multiplied.  SPLIT: K is summed in 2^cut parts.
// emit(m, n, base(m, n) and the parts' sums in order; GLU: gate, up).
template <int R, int S, int U, bool GLU, bool NORM, bool SPLIT, class Ready, class Base, class Emit>
__device__ __forceinline__ void project(const float* W, int N, int K, int cut, const float* gain, float eps, const float* xs, Ready ready,
                                        Base base, Emit emit) {
  constexpr int C = GLU ? 2 : 1;
  // what is derived from these is worked out here: kept over the layers, the addresses of all phases take the registers
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid), "+s"(W), "+s"(N), "+s"(K));
  const int lane = tid & 63;
  const int first = __builtin_amdgcn_readfirstlane(tid >> 6) * WGS + blockIdx.x;
  const int nv = K >> 2, nb = (nv + 63) >> 6;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 w[U][S][C], g[NORM ? U : 1];
  auto load = [&](int n0, int b, int be) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = (b + u) * 64 + lane;
      const bool live = b + u < be && i < nv;
#pragma unroll
      for (int s = 0; s < S; ++s)
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const int n = n0 + s * GW;
          w[u][s][c] = live && n < N ? reinterpret_cast<const f32x4*>(W + (size_t)(n + c * N) * K)[i] : zero;
        }
      if constexpr (NORM) g[u] = i < nv ? reinterpret_cast<const f32x4*>(gain)[i] : zero;
    }
  };
  load(first, 0, SPLIT ? nb >> cut : nb);
  ready();
  auto row = [&](int m, int b) {
    const int i = b * 64 + lane;
    return i < nv ? reinterpret_cast<const f32x4*>(xs + (size_t)m * K)[i] : zero;
  };
  float inv[R];
  if constexpr (NORM)
#pragma unroll
    for (int m = 0; m < R; ++m) {
      float tot = 0.f;
      for (int b = 0; b < nb; ++b) {
        const f32x4 v = row(m, b);
        float ss = 0.f;
        ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
        tot += wave_sum(ss);
      }
      inv[m] = 1.0f / sqrtf(tot / (float)K + eps);
    }
  for (int n0 = first; n0 < N; n0 += S * GW) {
    float sum[SPLIT ? S : 1];
    for (int sp = 0; sp < (SPLIT ? 1 << cut : 1); ++sp) {
      const int b0 = SPLIT ? sp * nb >> cut : 0, b1 = SPLIT ? (sp + 1) * nb >> cut : nb;
      float acc[S][C][R];
#pragma unroll
      for (int s = 0; s < S; ++s)
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int m = 0; m < R; ++m) acc[s][c][m] = 0.f;
      for (int b = b0; b < b1; b += U) {
        if (n0 != first || b) load(n0, b, b1);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          __builtin_amdgcn_sched_barrier(0);  // one piece of the rows in registers, not all
#pragma unroll
          for (int m = 0; m < R; ++m) {
            f32x4 x = row(m, b + u);  // behind the part's end: times no weights
            if constexpr (NORM)
#pragma unroll
              for (int e = 0; e < 4; ++e) x[e] = x[e] * inv[m] * g[u][e];
            else if (SPLIT && b + u >= b1) x = zero;
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
              for (int c = 0; c < C; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[s][c][m] = fmaf(w[u][s][c][e], x[e], acc[s][c][m]);
          }
        }
      }
      // lane m keeps row m's sums
#pragma unroll
      for (int s = 0; s < S; ++s) {
        float v[C];
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int m = 0; m < R; ++m) {
            const float t = exchange<16, 32>(row16_sum(acc[s][c][m]), Add{});
            v[c] = m == 0 || lane == m ? t : v[c];
          }
        const int n = n0 + s * GW;
        if (n < N && lane < R) {
          if constexpr (SPLIT) sum[s] = (sp ? sum[s] : base(lane, n)) + v[0];
          else emit(lane, n, v[0], v[C - 1]);
        }
      }
    }
    if constexpr (SPLIT)
#pragma unroll
      for (int s = 0; s < S; ++s)
        if (n0 + s * GW < N && lane < R) emit(lane, n0 + s * GW, sum[s], 0.f);
  }
}

template <int R, int HD>
__global__ void __launch_bounds__(NT, 4) k_step_small_f32(SmallStep a) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  __shared__ float am[ATTN_NW], al[ATTN_NW], aacc[ATTN_NW][HD], bv[AMAX_NW];
  __shared__ int bi[AMAX_NW], spos[R];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int d = a.d, F = a.F, qd = a.hq * HD, nq = qd + 2 * a.hkv * HD;
  float *xs = sm, *x2s = xs + R * d, *as = x2s + R * d, *hs = as + R * qd;  // rows, rows behind O, attention (q, k, v first), SwiGLU
  u64 *lx = a.xch, *lq = lx + R * d, *la = lq + R * nq, *lx2 = la + R * qd, *lh = lx2 + R * d, *ll = lh + R * F;
  const unsigned tag0 = __hip_atomic_load(a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
  if ((int)threadIdx.x < R) {
    const int p = a.seq_lens[threadIdx.x];
    spos[threadIdx.x] = p >= 0 && p < a.max_seq ? p : -1;
  }
  auto none = [](int, int) { return 0.f; };
  const float* w = a.w;
  for (int li = 0; li < a.layers; ++li, w += a.layer_stride) {
    const unsigned tag = tag0 + li;
    const bool keep = li + 1 == a.layers;  // what ls_stage_workspace_region shows
    // ---- QKV
    project<R, R <= 2 ? 6 : 4, 1, false, true, false>(w + a.o_qkv, nq, d, 0, w, a.eps, xs, [&]() {
      if (li) {
        gather(lx, R * d, tag, xs);
      } else {
        for (int i = threadIdx.x; i < R * d; i += NT) {
          const int r = i / d;
          const float* src = a.in + (size_t)r * d;
          if (a.table) {
            int id = ((const int32_t*)a.in)[r];
            id = id < 0 ? 0 : (id >= a.vocab ? a.vocab - 1 : id);  // an id outside the table is clamped
            src = a.table + (size_t)id * d;
          }
          xs[i] = src[i - r * d];
        }
      }
      __syncthreads();
    }, none, [&](int m, int n, float v, float) {
      put(lq + m * nq + n, tag, v);
      if (keep) a.qkv[m * nq + n] = v;
    });

    // ---- attention: a query head of a row at a time, the context in ranges as in k_attn_decode
    constexpr int LPK = HD / 8, KPI = 64 / LPK;
    typedef float f32x8 __attribute__((ext_vector_type(8)));
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, slot = lane / LPK, dl = lane % LPK;
    for (int unit = blockIdx.x; unit < R * a.hq; unit += WGS) {
      int r = 0, h = unit;  // no division on the way
      for (; h >= a.hq; h -= a.hq) ++r;
      const int kh = h >> a.group;
      const int pos = spos[r];
      if (pos < 0) {  // a sequence with no room left: its rows are nobody's, but the other workgroups wait for them
        if ((int)threadIdx.x < HD) put(la + r * qd + h * HD + threadIdx.x, tag, 0.f);
        continue;
      }
      float* kb = a.kc + li * a.kv_layer + ((size_t)r * a.hkv + kh) * a.max_seq * HD;
      float* vb = a.vc + li * a.kv_layer + ((size_t)r * a.hkv + kh) * a.max_seq * HD;
      const int chunk = ((pos + ATTN_NW * KPI - 1) / (ATTN_NW * KPI)) * KPI;
      const int begin = wave * chunk, end = min(begin + chunk, pos);
      auto fetch = [&](int j, f32x8& k, f32x8& v) {
        if (j < end) {
          const int key = min(j + slot, pos - 1);
          k = *reinterpret_cast<const f32x8*>(kb + (size_t)key * HD + dl * 8);
          v = *reinterpret_cast<const f32x8*>(vb + (size_t)key * HD + dl * 8);
        }
      };
      f32x8 kf, vf, kn, vn;
      float2 rot[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) rot[i] = a.cs[(size_t)pos * (HD / 2) + dl * 4 + i];
      fetch(begin, kf, vf);
      // q, k and v of this head
      __syncthreads();  // the unit before is done with as and the partial results
      gather<1>(3 * HD, tag, as, [&](int e) {
        const int part = e / HD;  // q, k, v
        return lq + r * nq + (part == 0 ? h : part == 1 ? a.hq + kh : a.hq + a.hkv + kh) * HD + e % HD;
      });
      __syncthreads();
      const float scale = 1.0f / sqrtf((float)HD);
      float q[8];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float u0 = as[dl * 8 + 2 * i], u1 = as[dl * 8 + 2 * i + 1];
        q[2 * i] = turn0(u0, u1, rot[i]) * scale;
        q[2 * i + 1] = turn1(u0, u1, rot[i]) * scale;
      }
      float m = -INFINITY, l = 0.f, acc[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.f;
      auto key = [&](const f32x8& k, const f32x8& v, bool valid) {
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) s = fmaf(q[e], k[e], s);
        s = exchange<LPK / 2, 1>(s, Add{});
        s = valid ? s : -INFINITY;
        const float mn = fmaxf(m, s);
        const float corr = mn == -INFINITY ? 1.f : __expf(m - mn);
        const float p = s == -INFINITY ? 0.f : __expf(s - mn);
        l = l * corr + p;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = fmaf(p, valid ? v[e] : 0.f, acc[e] * corr);
        m = mn;
      };
      if (wave == 0) {  // the new row
        f32x8 kr, vr;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const float u0 = as[HD + dl * 8 + 2 * p], u1 = as[HD + dl * 8 + 2 * p + 1];
          kr[2 * p] = turn0(u0, u1, rot[p]);
          kr[2 * p + 1] = turn1(u0, u1, rot[p]);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) vr[e] = as[2 * HD + dl * 8 + e];
        if (slot == 0 && (kh << a.group) == h) {
          *reinterpret_cast<f32x8*>(kb + (size_t)pos * HD + dl * 8) = kr;
          *reinterpret_cast<f32x8*>(vb + (size_t)pos * HD + dl * 8) = vr;
        }
        key(kr, vr, slot == 0);
      }
      for (int j = begin; j < end; j += 2 * KPI) {
        fetch(j + KPI, kn, vn);
        key(kf, vf, j + slot < end);
        fetch(j + 2 * KPI, kf, vf);
        if (j + KPI < end) key(kn, vn, j + KPI + slot < end);
      }
      const float mw = exchange<LPK, 32>(m, Max{});
      const float wt = m == -INFINITY ? 0.f : __expf(m - mw);
      // as there, the weighted value itself is added to its neighbour's rounded one
      auto total = [&](float v) { return exchange<2 * LPK, 32>(fmaf(v, wt, __shfl_xor(v * wt, LPK)), Add{}); };
      const float lw = total(l);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = total(acc[e]);
      if (lane < LPK) {
        if (dl == 0) { am[wave] = mw; al[wave] = lw; }
#pragma unroll
        for (int e = 0; e < 8; ++e) aacc[wave][dl * 8 + e] = acc[e];
      }
      __syncthreads();
      if ((int)threadIdx.x < HD) {
        float mm = -INFINITY;
#pragma unroll
        for (int v = 0; v < ATTN_NW; ++v) mm = fmaxf(mm, am[v]);
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int v = 0; v < ATTN_NW; ++v) {
          const float t = am[v] == -INFINITY ? 0.f : __expf(am[v] - mm);
          num += aacc[v][threadIdx.x] * t;
          den += al[v] * t;
        }
        put(la + r * qd + h * HD + threadIdx.x, tag, num / den);
        if (keep) a.attn[r * qd + h * HD + threadIdx.x] = num / den;
      }
    }

    // ---- O, added to the rows
    project<R, 2, R == 1 ? 4 : R == 2 ? 3 : 1, false, false, true>(w + a.o_o, d, qd, a.cut_o, nullptr, 0.f, as, [&]() {
      __syncthreads();  // the last unit is done with as
      gather(la, R * qd, tag, as);
      __syncthreads();
    }, [&](int m, int n) { return xs[m * d + n]; }, [&](int m, int n, float v, float) { put(lx2 + m * d + n, tag, v); });

    // ---- gate-up
    project<R, R <= 2 ? 3 : 2, 1, true, true, false>(w + a.o_gu, F, d, 0, w + a.o_g2, a.eps, x2s, [&]() {
      gather(lx2, R * d, tag, x2s);
      __syncthreads();
    }, none, [&](int m, int n, float g, float u) {
      const float v = silu_f(g) * u;
      put(lh + m * F + n, tag, v);
      if (keep) a.h[m * F + n] = v;
    });

    // ---- down, added to the rows: the next layer's, the head's or the stage's output
    const bool to_out = li + 1 == a.layers && !a.head_w;
    project<R, 2, R == 1 ? 4 : R == 2 ? 3 : 1, false, false, true>(w + a.o_d, d, F, a.cut_d, nullptr, 0.f, hs, [&]() {
      gather(lh, R * F, tag, hs);
      __syncthreads();
    }, [&](int m, int n) { return x2s[m * d + n]; }, [&](int m, int n, float v, float) {
      if (to_out) a.out[(size_t)m * d + n] = v;
      else put(lx + m * d + n, tag + 1, v);
    });
  }

  // ---- head: logits, then the workgroup of a row takes their largest as k_argmax does, whose threads are two of this one's
  if (a.head_w) {
    const unsigned tag = tag0 + a.layers;
    project<R, 4, 1, false, true, false>(a.head_w, a.vocab, d, 0, a.head_gain, a.eps, xs, [&]() {
      gather(lx, R * d, tag, xs);
      __syncthreads();
    }, none, [&](int m, int n, float v, float) {
      a.logits[(size_t)m * a.vocab + n] = v;
      put(ll + m * a.vocab + n, tag, v);
    });
    if ((int)blockIdx.x < R) {
      const int r = blockIdx.x;
      __syncthreads();
      gather(ll + r * a.vocab, a.vocab, tag, sm);
      __syncthreads();
#pragma unroll
      for (int half = 0; half < AMAX_NW / NW; ++half) {
        float best = -INFINITY;
        int idx = 0x7fffffff;
        for (int i = threadIdx.x + half * NT; i < a.vocab; i += AMAX_NW * 64)
          if (sm[i] > best || idx == 0x7fffffff) { best = sm[i]; idx = i; }
        auto better = [&](float ov, int oi) {
          if (ov > best || (ov == best && oi < idx)) { best = ov; idx = oi; }
        };
#define LS_OTHER(off) better(lane_xor<off>(best), __float_as_int(lane_xor<off>(__int_as_float(idx))));
        LS_OTHER(32) LS_OTHER(16) LS_OTHER(8) LS_OTHER(4) LS_OTHER(2) LS_OTHER(1)
#undef LS_OTHER
        if (lane == 0) { bv[wave + half * NW] = best; bi[wave + half * NW] = idx; }
      }
      __syncthreads();
      if (wave == 0) {  // the sixteen in order, from registers
        const float tv = bv[lane & 15];
        const int ti = bi[lane & 15];
        float best = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, tv), 0));
        int idx = __builtin_amdgcn_readlane(ti, 0);
#pragma unroll
        for (int v = 1; v < AMAX_NW; ++v) {
          const float ov = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, tv), v));
          const int oi = __builtin_amdgcn_readlane(ti, v);
          if (ov > best || (ov == best && oi < idx)) { best = ov; idx = oi; }
        }
        if (lane == 0) ((int32_t*)a.out)[r] = idx;
      }
    }
  }
  // Workgroup 0 has seen values of all others that they sent behind their reads of the tag and of the lengths.
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) *a.epoch = tag0 + a.layers;
    if ((int)threadIdx.x < R && spos[threadIdx.x] >= 0) a.seq_lens[threadIdx.x] = spos[threadIdx.x] + 1;
  }
}

constexpr int ROWS = 4;
std::atomic<long> launches{0};

// Parts of the static array, one to a stage: HEAD words for the last step's tag, then the places.  A stage that finds all of them taken takes the separate launches.
constexpr int PARTS = 64, HEAD = 32, PART_WORDS = 18 * 1024, MAX_DEVICES = 64;
__device__ __align__(256) u64 places[PARTS][PART_WORDS];

struct Pool {
  u64* base = nullptr;  // this device's copy of the array
  u64 taken = 0;        // bit i: part i
};
std::mutex pool_mutex;
Pool pools[MAX_DEVICES];

// The shapes that are taken (small_step_shape, small_step_rows).
constexpr int COLUMNS = 256, QUERY = 1024, FFN = 2048, VOCAB = 1024, UNITS = WGS, FFN_ROWS = 3072, HD_MOST = 128;
static_assert(HEAD + 2 * ROWS * COLUMNS + 4 * UNITS * HD_MOST + FFN_ROWS + ROWS * VOCAB <= PART_WORDS, "places of the largest step");
static_assert((2 * ROWS * COLUMNS + UNITS * HD_MOST + FFN_ROWS) * sizeof(float) <= 60 * 1024, "two workgroups and what they hold besides to a CU's 160 KB");

size_t lds_bytes(const SmallStep& a, int rows) {
  const size_t r = rows, acts = 2 * r * a.d + std::max(r * (a.hq * a.hd + a.F), (size_t)3 * a.hd);
  return std::max(acts, (size_t)(a.head_w ? a.vocab : 0)) * sizeof(float);
}

template <int R, int HD>
void launch_k(const SmallStep& a, hipStream_t st) {
  const int bytes = (int)lds_bytes(a, R);
  static std::atomic<int> allowed[64];
  allow_dynamic_lds_up_to((const void*)k_step_small_f32<R, HD>, bytes, allowed);
  k_step_small_f32<R, HD><<<WGS, NT, bytes, st>>>(a);
}

template <int R>
void launch_r(const SmallStep& a, hipStream_t st) {
  if (a.hd == 64) launch_k<R, 64>(a, st);
  else launch_k<R, 128>(a, st);
}

}  // namespace

// Rows of one piece of 256 columns.  Two layers and a head of 512 entries, separate launches / this one, 1 row and 4, 40 and
// 600 keys: 128 columns 37.7 / 24.5, 50.5 / 39.4, 43.2 / 28.2, 54.5 / 42.9 us; 256 columns 39.2 / 28.4, 51.1 / 46.2, 56.1 / 33.0,
// 68.4 / 51.1; 384 columns 47.7 / 44.7, 58.3 / 83.6: sixteen CUs then take longer over the weights than the launches cost.  The O
// and down projections' rows likewise, one row: 16 heads of 128 37 / 46, 16 of 64 39 / 33; ffn of 2904 42 / 48, 2376 43 / 49, 1884
// 54 / 51.  Of 76 shapes drawn at random that are taken the slowest takes 0.98 of the separate launches' time, all in the mean 0.75.
bool small_step_shape(int d, int hq, int hkv, int hd, int F, int vocab) {
  if (!attn_decode_supported(hq, hkv, hd) || d % 4 || F % 4 || d < WGS || F < WGS || (vocab && vocab < WGS)) return false;
  if (d > COLUMNS || (long)hq * hd > QUERY || F > FFN || vocab > VOCAB) return false;
  return (size_t)d * (2 * (size_t)(hq + hkv) * hd + 3 * (size_t)F) <= (1u << 20);  // weights of a layer
}

// A workgroup takes its heads of a row one after the other, each behind an exchange: no more of them than workgroups.  Every
// workgroup gathers all of the SwiGLU's output, 1024 values to an exchange: three of them.  Separate launches / this one, two
// layers: 44 columns, 32 heads, 4 rows, 200 keys (8 units to a workgroup) 58 / 143 us, 32 heads and one row (2) 44 / 55, 8 and
// two rows (1) 42 / 36; ffn of 1608 and two rows 48 / 51, 804 and two 40 / 33.
bool small_step_rows(int rows, int hq, int F) { return rows >= 1 && rows <= ROWS && (long)rows * hq <= UNITS && (long)rows * F <= FFN_ROWS; }

SmallStepPlaces take_small_step_places(int device, int d, int hq, int hkv, int hd, int F, int vocab) {
  static_assert(PARTS == 64, "");
  if (device < 0 || device >= MAX_DEVICES || !small_step_shape(d, hq, hkv, hd, F, vocab) || !small_step_rows(1, hq, F)) return {};
  std::lock_guard<std::mutex> lock(pool_mutex);
  Pool& p = pools[device];
  if (!p.base) {
    void* base = nullptr;
    if (hipGetSymbolAddress(&base, HIP_SYMBOL(places)) != hipSuccess || hipMemset(base, 0, sizeof places) != hipSuccess ||
        hipStreamSynchronize(nullptr) != hipSuccess) {
      (void)hipGetLastError();
      return {};
    }
    p.base = (u64*)base;
  }
  if (!~p.taken) return {};
  const int i = __builtin_ctzll(~p.taken);
  p.taken |= (u64)1 << i;
  u64* part = p.base + (size_t)i * PART_WORDS;
  return {part + HEAD, (unsigned*)part};  // a stage before this one may have left tags: the next steps go on behind them
}

void give_small_step_places(int device, SmallStepPlaces places) {
  if (!places.xch) return;
  std::lock_guard<std::mutex> lock(pool_mutex);
  pools[device].taken &= ~((u64)1 << (places.xch - pools[device].base) / PART_WORDS);
}

bool small_step_supported(const SmallStep& a, int rows, int max_keys) {
  return a.xch && small_step_shape(a.d, a.hq, a.hkv, a.hd, a.F, a.head_w ? a.vocab : 0) && small_step_rows(rows, a.hq, a.F) &&
         attn_decode_chunks(rows, a.hkv, max_keys) == 1 && (!a.head_w || gemm_rows_f32_norm_supported(rows, a.vocab, a.d));
}

// Room for one launch on each of the device's hardware queues, on every XCD (two workgroups of each launch go to each, whatever is
// free elsewhere), on the CUs that the stream's mask leaves it; the mask's bits may be dealt to the XCDs in turn or one after the
// other.  Asked for anew each time: 0.2 us.
bool small_step_room(hipStream_t st) {
  constexpr int QUEUES = 24, XCDS = 8, CUS = QUEUES * (WGS / XCDS) / 2, MASK_WORDS = 32;
  if (st == hipStreamLegacy || st == hipStreamPerThread) st = nullptr;  // the query knows no handle of these
  uint32_t mask[MASK_WORDS] = {};
  if (hipExtStreamGetCUMask(st, MASK_WORDS, mask) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  for (int x = 0; x < XCDS; ++x) {
    int in_turn = 0;
    for (int i = 0; i < XCDS; ++i) in_turn += __builtin_popcount(mask[i] & 0x01010101u << x);
    if (in_turn < CUS || __builtin_popcount(mask[x]) < CUS) return false;
  }
  return true;
}

void launch_small_step(const SmallStep& a, int rows, hipStream_t st) {
  ++launches;
  switch (rows) {
    case 1: launch_r<1>(a, st); break;
    case 2: launch_r<2>(a, st); break;
    case 3: launch_r<3>(a, st); break;
    case 4: launch_r<4>(a, st); break;
  }
}

}  // namespace ls

// For the tests; not declared in ls_stage.h: steps that took the one launch so far.
extern "C" long ls_test_small_steps(void) { return ls::launches; }
