// Shared device/host helpers for the gfx950 kernels of libsama.  Not part of the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string>

namespace sama {

typedef uint16_t bf16_t;  // raw bfloat16 bits

constexpr int WAVE = 64;

__device__ __forceinline__ float bf16_to_f32(bf16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// two floats -> packed bf16 pair (a in the low half), round-to-nearest-even in hardware (v_cvt_pk_bf16_f32)
typedef __bf16 bf16x2_hw __attribute__((ext_vector_type(2)));
typedef float f32x2_hw __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  const f32x2_hw v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_hw));
}

// round-to-nearest-even; NaN stays NaN
__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return (bf16_t)pack_bf16x2(f, 0.f); }

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}
__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
  return x;
}

// Sum over a block of up to 1024 threads in a fixed order: wave shuffles, then the wave leaders' values
// added serially from LDS.  Every thread gets the result.  `red` holds >= 16 floats.
__device__ __forceinline__ float block_sum(float x, float* red) {
  x = wave_sum(x);
  const int w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = x;
  __syncthreads();
  float s = 0.f;
  for (int i = 0; i < nw; ++i) s += red[i];
  return s;
}

// Results that workgroups of one launch hand to the last of them.  publish() / collect() are agent-scope accesses, coherent
// between the XCDs' caches one by one, so that no workgroup has to write back or invalidate its L2 (a device-wide fence in every
// workgroup cost ~3 us of a 5 us kernel).
// They are relaxed: what orders them is gfx950 itself.  An agent-scope store is written through its XCD's L2 and counted by vmcnt
// until it has arrived where every XCD sees it, so after the wait and the barrier of last_block() all of the workgroup's
// published values are visible before its ticket is; the loads of collect() are issued after the last ticket came back and bypass
// what the caches hold.  That is the instruction sequence of a release on the ticket and an acquire behind it, less the write-back
// and the invalidation of the L2, which concern ordinary accesses: nothing but published values may be handed over this way.
// With the pair written out a logistic-regression iteration takes 63.4 us instead of 62.1 and an adaptation of 512 workgroups
// 17 us instead of 12.
#if defined(__HIP_DEVICE_COMPILE__) && !defined(__gfx950__)
#error "publish() / last_block() / collect() rest on gfx950's agent-scope accesses; another chip needs a release and an acquire"
#endif
__device__ __forceinline__ void publish(double* p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ double collect(const double* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// Whether this workgroup is the last of `total` to get here, for every thread of it; the last one may collect() what the
// others published before they came.  `ticket` starts at zero and is left at zero.
__device__ __forceinline__ bool last_block(uint32_t* ticket, int total, int* s_last) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's published values have reached memory
  __syncthreads();
  if (threadIdx.x == 0) {
    const bool last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)total - 1u;
    if (last) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *s_last = last ? 1 : 0;
  }
  __syncthreads();
  return *s_last != 0;
}

// b^t for an integer t >= 0 by squaring: forty dependent multiplications at most, where pow() costs a microsecond or two.  Its
// relative error is about t 2^-53 (a millionth step: 1e-10), far below the fp32 scalars it is for.
__device__ __forceinline__ double ipow(double b, int64_t t) {
  double r = 1.0;
  for (; t > 0; t >>= 1, b *= b)
    if (t & 1) r *= b;
  return r;
}

// A non-GEMM parameter as the current pass sees it: theta[k] + s * v[k], with s = +-eps read from the device
// (s_ptr == nullptr: the unperturbed parameter).
struct ParamView {
  const float* theta;
  const float* vdir;
  const float* eps_ptr;
  float sign;
  int flip_row;  // > 0: a kernel's rows >= flip_row see the opposite sign (the + and the - pass stacked in one launch)
  __device__ __forceinline__ float scale() const { return (eps_ptr != nullptr && sign != 0.f) ? sign * (*eps_ptr) : 0.f; }
  __device__ __forceinline__ float scale_row(int row) const {
    const float s = scale();
    return (flip_row > 0 && row >= flip_row) ? -s : s;
  }
  __device__ __forceinline__ float at(int64_t k, float s) const { return s != 0.f ? fmaf(s, vdir[k], theta[k]) : theta[k]; }
};

}  // namespace sama
