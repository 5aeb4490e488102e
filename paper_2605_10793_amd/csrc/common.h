// Shared device/host helpers for the gfx950 kernels of libconqur.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace conqur {

// A kernel's dynamic-LDS limit (hipFuncSetAttribute) belongs to the device that is current when it is set: launchers
// raise it once per device and kernel.  One bit per device ordinal; ordinals beyond 63 set it on every launch.
class PerDeviceOnce {
 public:
  template <typename F>
  hipError_t run(F&& set) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = (dev >= 0 && dev < 64) ? (1ull << dev) : 0ull;
    if (bit && (done_.load(std::memory_order_acquire) & bit)) return hipSuccess;
    e = set();
    if (e == hipSuccess && bit) done_.fetch_or(bit, std::memory_order_release);
    return e;
  }

 private:
  std::atomic<uint64_t> done_{0};
};


typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short bf16_bits;  // raw bf16 storage

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// fp32 -> bf16, round to nearest even (NaN stays NaN, Inf stays Inf): the hardware conversion
// (v_cvt_pk_bf16_f32, one instruction for two values).
__device__ __forceinline__ bf16_bits f32_to_bf16(float f) {
  const __bf16 b = (__bf16)f;
  return __builtin_bit_cast(unsigned short, b);
}
// Two values at once, packed lo | hi << 16.
__device__ __forceinline__ uint32_t f32x2_to_bf16x2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
// Two values as fp16 (round to nearest even), packed lo | hi << 16.
__device__ __forceinline__ uint32_t f32x2_to_f16x2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
}
__device__ __forceinline__ bf16_bits f32_to_f16(float f) {
  const _Float16 h = (_Float16)f;  // round to nearest even
  return __builtin_bit_cast(unsigned short, h);
}
__device__ __forceinline__ float bf16_to_f32(bf16_bits b) { return __uint_as_float(((uint32_t)b) << 16); }

// Sums and maxima over lanes, known to every lane afterwards: the butterfly with offsets 32, 16, 8, 4, 2, 1 (or 8, 4, 2, 1 within
// rows of 16 lanes), one VALU operation per offset.  Swapping the halves (odd and even rows) of a register with itself leaves either
// half in both; behind offset 8 the values of a row repeat every 8 lanes, so that a rotation by 4 meets the same partner as the
// XOR, and so on.  A lane exchange through LDS (ds_bpermute) instead takes some 60 cycles per offset and another half dozen instructions
// for a workgroup that reads one row: see k_quant_error.
template <int N>
__device__ __forceinline__ uint32_t row_rotated(uint32_t v) {   // by N lanes within rows of 16
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x120 + N, 0xf, 0xf, true);
}
template <int N>
__device__ __forceinline__ float row_rotated(float v) { return __uint_as_float(row_rotated<N>(__float_as_uint(v))); }
template <int N>
__device__ __forceinline__ double row_rotated(double v) {
  const uint2 u = __builtin_bit_cast(uint2, v);
  return __builtin_bit_cast(double, make_uint2(row_rotated<N>(u.x), row_rotated<N>(u.y)));
}
template <typename T, typename Op>
__device__ __forceinline__ T row16_reduce(T v, Op op) {
  v = op(v, row_rotated<8>(v));
  v = op(v, row_rotated<4>(v));
  v = op(v, row_rotated<2>(v));
  return op(v, row_rotated<1>(v));
}
template <typename Op>
__device__ __forceinline__ float wave_reduce(float v, Op op) {
  const uint32_t u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const uint32_t w = __float_as_uint(op(__uint_as_float(a[0]), __uint_as_float(a[1])));
  const auto b = __builtin_amdgcn_permlane16_swap(w, w, false, false);
  return row16_reduce(op(__uint_as_float(b[0]), __uint_as_float(b[1])), op);
}
template <typename Op>
__device__ __forceinline__ double wave_reduce(double v, Op op) {
  auto both = [&](auto swap) {
    const uint2 u = __builtin_bit_cast(uint2, v);
    const auto x = swap(u.x), y = swap(u.y);
    v = op(__builtin_bit_cast(double, make_uint2(x[0], y[0])), __builtin_bit_cast(double, make_uint2(x[1], y[1])));
  };
  both([](uint32_t u) { return __builtin_amdgcn_permlane32_swap(u, u, false, false); });
  both([](uint32_t u) { return __builtin_amdgcn_permlane16_swap(u, u, false, false); });
  return row16_reduce(v, op);
}
__device__ __forceinline__ float wave_sum(float v) { return wave_reduce(v, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ double wave_sum_d(double v) { return wave_reduce(v, [](double a, double b) { return a + b; }); }
__device__ __forceinline__ float wave_max(float v) { return wave_reduce(v, [](float a, float b) { return fmaxf(a, b); }); }
__device__ __forceinline__ float row16_sum(float v) { return row16_reduce(v, [](float a, float b) { return a + b; }); }

// A value for the host, in pinned memory: stored through every cache, so that it is there once the kernel (and an event behind it)
// has completed, whatever that event releases.
template <typename T>
__device__ __forceinline__ void store_for_host(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }

static inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// The accumulate operand holds the unit rows x^ = x / ||x|| times this power of two, in fp16.  |x^| <= 1, and on
// outlier-dominated rows most entries are 1e-3 .. 1e-5: times 1/sqrt(dh) (the corner's magnitude) they would sit in
// fp16's subnormal range (below 6.1e-5) and lose bits; scaled up they keep all 11.  The factor and 1/sqrt(dh) are
// applied to the fp32 result instead (exact power of two; the sum cannot overflow: 64 * tokens * 1).
constexpr float kXhatScale = 64.0f;

}  // namespace conqur
