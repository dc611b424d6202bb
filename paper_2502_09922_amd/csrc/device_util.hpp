// Small device helpers shared by the HIP kernels (gfx950, 64-lane wavefronts).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <atomic>
#include <cstdint>
#include <mutex>

#include "kernels.hpp"

namespace ls {

// kernel<<<grid, block, smem, st>>>(args...), or the same launch with the runtime's per-kernel
// start/stop events when the stage runtime has armed launch_timing().
template <typename... KArgs, typename... Args>
inline void launch_kernel(void (*kernel)(KArgs...), dim3 grid, dim3 block, unsigned smem, hipStream_t st, Args... args) {
  LaunchTiming& t = launch_timing();
  if (t.start) {
    hipExtLaunchKernelGGL(kernel, grid, block, smem, st, t.start, t.stop, 0, static_cast<KArgs>(args)...);
    t.start = t.stop = nullptr;
    t.used = true;
  } else {
    hipLaunchKernelGGL(kernel, grid, block, smem, st, static_cast<KArgs>(args)...);
  }
}

// Raise a kernel's dynamic-LDS limit, once per device (`done` holds one bit per device ordinal;
// the attribute belongs to each device's copy of the kernel).  Safe from several threads: a
// race only sets the same attribute twice.
inline void allow_dynamic_lds(const void* kernel, int bytes, std::atomic<uint64_t>& done) {
  int dev = 0;
  (void)hipGetDevice(&dev);
  const uint64_t bit = 1ull << (dev & 63);
  if (done.load(std::memory_order_acquire) & bit) return;
  (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  done.fetch_or(bit, std::memory_order_release);
}

// The same for a kernel whose LDS need varies with the shape: `allowed[device]` is the limit set
// so far, raised (under a lock, so that a smaller request cannot overwrite a larger one) when a
// launch needs more.
inline void allow_dynamic_lds_up_to(const void* kernel, int bytes, std::atomic<int> (&allowed)[64]) {
  static std::mutex m;
  int dev = 0;
  (void)hipGetDevice(&dev);
  std::atomic<int>& a = allowed[dev & 63];
  if (bytes <= a.load(std::memory_order_acquire)) return;
  std::lock_guard<std::mutex> lock(m);
  if (bytes <= a.load(std::memory_order_relaxed)) return;
  (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  a.store(bytes, std::memory_order_release);
}

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));  // a raw 16-byte load
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float to_f(float v) { return v; }
__device__ __forceinline__ float to_f(bf16 v) { return (float)v; }
// float -> storage type; the bf16 conversion rounds to nearest, ties to even.
template <class T> __device__ __forceinline__ T from_f(float f);
template <> __device__ __forceinline__ float from_f<float>(float f) { return f; }
template <> __device__ __forceinline__ bf16 from_f<bf16>(float f) { return (bf16)f; }

// f(v, v of lane ^ OFF): register-to-register exchanges (DPP inside a row of 16 lanes, permlane swaps across rows) instead of
// a trip through the LDS crossbar, which a chain of exchanges waits for at every step.  f has to be commutative.
template <int CTRL, int BANKS = 0xF>
__device__ __forceinline__ float dpp(float old, float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old), __builtin_bit_cast(int, v), CTRL, 0xF, BANKS, BANKS == 0xF));
}
template <int OFF, class F>
__device__ __forceinline__ float with_lane_xor(float v, F f) {
  static_assert(OFF == 1 || OFF == 2 || OFF == 4 || OFF == 8 || OFF == 16 || OFF == 32, "");
  if constexpr (OFF >= 16) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const unsigned u = __builtin_bit_cast(unsigned, v);
    u32x2 r;
    if constexpr (OFF == 32) r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    else r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return f(__uint_as_float(r[0]), __uint_as_float(r[1]));
  } else if constexpr (OFF == 8) {
    return f(v, dpp<0x128>(v, v));  // row_ror:8
  } else if constexpr (OFF == 4) {  // banks of four lanes: 0 and 2 take four lanes up, 1 and 3 four lanes down
    return f(v, dpp<0x114, 0xA>(dpp<0x104, 0x5>(v, v), v));
  } else {
    return f(v, dpp<OFF == 2 ? 0x4E : 0xB1>(v, v));  // quad_perm
  }
}
// v of lane ^ OFF.
template <int OFF>
__device__ __forceinline__ float lane_xor(float v) {
  if constexpr (OFF < 16) return with_lane_xor<OFF>(v, [](float, float other) { return other; });
  else return with_lane_xor<OFF>(v, [](float low, float high) { return threadIdx.x & OFF ? low : high; });
}
// f over the aligned groups of `2 FROM / TO` lanes TO apart, the exchanges from lane ^ FROM down to lane ^ TO or, FROM < TO, up
// to it: every lane of the group gets the result, summed in the order of the exchanges.
template <int FROM, int TO, class F>
__device__ __forceinline__ float exchange(float v, F f) {
  v = with_lane_xor<FROM>(v, f);
  if constexpr (FROM == TO) return v;
  else return exchange<(FROM > TO ? FROM / 2 : FROM * 2), TO>(v, f);
}
struct Add { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };
struct Max { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };

// Sum over the 64 lanes of a wavefront; every lane gets the total (fixed butterfly order).
__device__ __forceinline__ float wave_sum(float v) { return exchange<32, 1>(v, Add{}); }

// Sum over each aligned group of 16 lanes, every lane of the group gets the total.  Four
// register-to-register DPP exchanges (lane^1, lane^2, mirrored half row, mirrored row) in a
// fixed order -- no trip through the LDS crossbar as with a general shuffle.
__device__ __forceinline__ float row16_sum(float v) {
#define LS_DPP_ADD(ctrl) \
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, 0xF, 0xF, true))
  LS_DPP_ADD(0xB1);   // quad_perm [1,0,3,2]
  LS_DPP_ADD(0x4E);   // quad_perm [2,3,0,1]
  LS_DPP_ADD(0x141);  // row_half_mirror: the other quad of the half row
  LS_DPP_ADD(0x140);  // row_mirror: the other half row
#undef LS_DPP_ADD
  return v;
}

// Sequences of a decode attention launch by length: which row has rank `rank`, the longest first (of equals the lower
// index), among `rows` <= 64 C rows with positions below `limit`, and its position.  Every wavefront finds it on its
// own, a bit of the position at a time by counting the rows that reach it: no LDS, no barrier.  (Comparing every row
// with every other through LDS took 5 us of every workgroup at 256 rows.)
template <int C>
__device__ __forceinline__ int row_by_length(const int32_t* __restrict__ row_pos, int rows, int rank, int limit, int& pos) {
  const int lane = threadIdx.x & 63;
  int len[C];  // position + 1: a sequence without room has 0, a row that is not there -1
#pragma unroll
  for (int c = 0; c < C; ++c) len[c] = c * 64 + lane < rows ? row_pos[c * 64 + lane] + 1 : -1;
  auto reach = [&](int v) {
    int n = 0;
#pragma unroll
    for (int c = 0; c < C; ++c) n += __builtin_popcountll(__builtin_amdgcn_ballot_w64(len[c] >= v));
    return n;
  };
  int v = 0;  // the largest length that more than `rank` rows reach
  for (int bit = 1 << (31 - __builtin_clz(limit | 1)); bit; bit >>= 1)
    if (reach(v | bit) > rank) v |= bit;
  int nth = rank - reach(v + 1), row = 0;  // among the rows of that length
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const uint64_t like = __builtin_amdgcn_ballot_w64(len[c] == v);
    const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(like >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)like, 0));
    const uint64_t is = __builtin_amdgcn_ballot_w64(len[c] == v && before == nth);
    if (is) row = c * 64 + __builtin_ctzll(is);
    nth -= __builtin_popcountll(like);
  }
  pos = v - 1;
  return row;
}

constexpr int waitcnt_vm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }  // vector memory only

// Wait until at most n of this wavefront's vector memory instructions are on their way, n known at run time (the
// instruction holds a constant).  More than 48: all are waited for.
__device__ __forceinline__ void wait_vm(int n) {
  switch (n) {
#define LS_WAIT(i) case i: __builtin_amdgcn_s_waitcnt(waitcnt_vm(i)); break;
#define LS_WAIT8(i) LS_WAIT(i) LS_WAIT(i + 1) LS_WAIT(i + 2) LS_WAIT(i + 3) LS_WAIT(i + 4) LS_WAIT(i + 5) LS_WAIT(i + 6) LS_WAIT(i + 7)
    LS_WAIT8(1) LS_WAIT8(9) LS_WAIT8(17) LS_WAIT8(25) LS_WAIT8(33) LS_WAIT8(41)
#undef LS_WAIT8
#undef LS_WAIT
    default: __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
  }
}

// The workgroup's barrier for wavefronts that hand LDS slots over: no read or write of memory moves across it, and with
// `done` every LDS read of this wavefront has its value before it.
template <bool done>
__device__ __forceinline__ void slot_barrier() {
  if constexpr (done) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  else asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// A pair turned by (cos, sin), with the product that is rounded chosen here and not by the compiler.
__device__ __forceinline__ float turn0(float u0, float u1, float2 cs) { return fmaf(u0, cs.x, -(u1 * cs.y)); }
__device__ __forceinline__ float turn1(float u0, float u1, float2 cs) { return fmaf(u0, cs.y, u1 * cs.x); }

// silu(z) = z / (1 + exp(-z)), the quotient as a product with the hardware reciprocal (1 ulp):
// a correctly rounded fp32 division is ten instructions, and every result is rounded to bf16
__device__ __forceinline__ float silu_f(float z) { return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

}  // namespace ls
