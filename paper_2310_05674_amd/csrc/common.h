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

// Butterflies over a wave, or over each group of sixteen of its lanes, without LDS: lanes 32 and 16 apart by the permlane swaps,
// lanes of a group by rotations.  A level joins the lanes 32, 16, 8, 4, 2, 1 apart; once the lanes 8 (4, 2) apart agree, a
// rotation by 4 (2, 1) reaches the same value as the exchange with the lane that far apart would.  A shuffle goes through the LDS
// unit, ~60 cycles a level; these are one or two vector instructions.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
template <int N>
__device__ __forceinline__ uint32_t rot16(uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x120 + N, 0xf, 0xf, false); }
template <int N>
__device__ __forceinline__ float rot16(float x) { return __uint_as_float(rot16<N>(__float_as_uint(x))); }
template <int N>
__device__ __forceinline__ double rot16(double x) {
  const u32x2 v = __builtin_bit_cast(u32x2, x);
  return __builtin_bit_cast(double, (u32x2){rot16<N>(v[0]), rot16<N>(v[1])});
}
// the two halves of every pair of lanes 32 (16) apart, for both of them
__device__ __forceinline__ void halves32(uint32_t x, uint32_t& a, uint32_t& b) { const u32x2 r = __builtin_amdgcn_permlane32_swap(x, x, false, false); a = r[0]; b = r[1]; }
__device__ __forceinline__ void halves16(uint32_t x, uint32_t& a, uint32_t& b) { const u32x2 r = __builtin_amdgcn_permlane16_swap(x, x, false, false); a = r[0]; b = r[1]; }
template <typename F>
__device__ __forceinline__ float join32(float x, F op) { uint32_t a, b; halves32(__float_as_uint(x), a, b); return op(__uint_as_float(a), __uint_as_float(b)); }
template <typename F>
__device__ __forceinline__ float join16(float x, F op) { uint32_t a, b; halves16(__float_as_uint(x), a, b); return op(__uint_as_float(a), __uint_as_float(b)); }
template <typename F>
__device__ __forceinline__ double join32(double x, F op) {
  const u32x2 v = __builtin_bit_cast(u32x2, x);
  u32x2 a, b; uint32_t p, q;
  halves32(v[0], p, q); a[0] = p; b[0] = q;
  halves32(v[1], p, q); a[1] = p; b[1] = q;
  return op(__builtin_bit_cast(double, a), __builtin_bit_cast(double, b));
}
template <typename F>
__device__ __forceinline__ double join16(double x, F op) {
  const u32x2 v = __builtin_bit_cast(u32x2, x);
  u32x2 a, b; uint32_t p, q;
  halves16(v[0], p, q); a[0] = p; b[0] = q;
  halves16(v[1], p, q); a[1] = p; b[1] = q;
  return op(__builtin_bit_cast(double, a), __builtin_bit_cast(double, b));
}
// over the sixteen lanes of a group; every one of them gets the result
template <typename T, typename F>
__device__ __forceinline__ T join_group(T x, F op) {
  x = op(x, rot16<8>(x)); x = op(x, rot16<4>(x)); x = op(x, rot16<2>(x));
  return op(x, rot16<1>(x));
}
// The same from the other end, over runs of n lanes (a power of two, the same for the wave): neighbours, pairs, then mirror images,
// which are as good as the exchange across the run once the halves agree within themselves.
template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
  const u32x2 v = __builtin_bit_cast(u32x2, x);
  return __builtin_bit_cast(double, (u32x2){(uint32_t)__builtin_amdgcn_update_dpp(0, (int)v[0], CTRL, 0xf, 0xf, false), (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v[1], CTRL, 0xf, 0xf, false)});
}
__device__ __forceinline__ double run_sum(double x, int n) {
  const auto add = [](double a, double b) { return a + b; };
  if (n > 1) x += dpp<0xb1>(x);     // quad_perm 1 0 3 2
  if (n > 2) x += dpp<0x4e>(x);     // quad_perm 2 3 0 1
  if (n > 4) x += dpp<0x141>(x);    // row_half_mirror
  if (n > 8) x += dpp<0x140>(x);    // row_mirror
  if (n > 16) x = join16(x, add);
  if (n > 32) x = join32(x, add);
  return x;
}
// over the wave
template <typename T, typename F>
__device__ __forceinline__ T join_wave(T x, F op) { return join_group(join16(join32(x, op), op), op); }
__device__ __forceinline__ float wave_sum(float x) { return join_wave(x, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ double wave_sum(double x) { return join_wave(x, [](double a, double b) { return a + b; }); }

// Sum over a block of up to 1024 threads in a fixed order: joined over the lanes of a wave, then the wave leaders' values
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
