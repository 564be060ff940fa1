// Device helpers shared by the kernel sources (internal).
#pragma once
#include <hip/hip_runtime.h>

#include "gw_kernels.h"

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ long long map3(const Map3& m, unsigned i) {
  const unsigned r = udiv(i, m.qin);
  const unsigned a = i - r * m.din;
  const unsigned c = udiv(r, m.qmid);
  const unsigned b = r - c * m.dmid;
  return (long long)c * m.sout + (long long)b * m.smid + (long long)a * m.sin;
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return double2{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}

// the larger of x and that of the lane which the DPP control CTRL names
template <int CTRL> __device__ __forceinline__ unsigned dpp_max(unsigned x) {
  return max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, false));
}

// accumulators of a three-product (Gauss) complex product
struct Acc3 {
  d4 p1, p2, p3;
};

__device__ __forceinline__ double2 to_d2(double2 v) { return v; }
__device__ __forceinline__ double2 to_d2(float2 v) { return double2{(double)v.x, (double)v.y}; }
__device__ __forceinline__ float2 to_f2(double2 v) { return float2{(float)v.x, (float)v.y}; }
__device__ __forceinline__ float2 to_f2(float2 v) { return v; }
template <class T> __device__ __forceinline__ T from_d2(double2 v);
template <> __device__ __forceinline__ double2 from_d2<double2>(double2 v) { return v; }
template <> __device__ __forceinline__ float2 from_d2<float2>(double2 v) {
  return float2{(float)v.x, (float)v.y};
}

// bf16 pairs (round to nearest even) for the split-bf16 contractions:
// element 0 in the low half, as in memory.
typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  const bf2v v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(unsigned, v);
}
__device__ __forceinline__ float bf16_low(unsigned p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float bf16_high(unsigned p) { return __builtin_bit_cast(float, p & 0xffff0000u); }

template <bool F32> struct Mfma;
template <> struct Mfma<false> {
  typedef double S;
  typedef double2 S2;
  typedef d4 Acc;
  static __device__ __forceinline__ Acc run(S a, S b, Acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // c - a b: the f64 MFMA reads its last control field as negate flags
  static __device__ __forceinline__ Acc run_neg(S a, S b, Acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 1);
  }
  template <class T> static __device__ __forceinline__ S2 cvt(T v) { return to_d2(v); }
  // output row of accumulator element r held by lane group g = lane / 16
  static __device__ __forceinline__ int row(int g, int r) { return g + 4 * r; }
};
template <> struct Mfma<true> {
  typedef float S;
  typedef float2 S2;
  typedef f4 Acc;
  static __device__ __forceinline__ Acc run(S a, S b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ Acc run_neg(S a, S b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(-a, b, c, 0, 0, 0);
  }
  template <class T> static __device__ __forceinline__ S2 cvt(T v) { return to_f2(v); }
  static __device__ __forceinline__ int row(int g, int r) { return 4 * g + r; }
};

// Raw buffer loads (gfx9 descriptor format).  A lane whose byte offset is not
// below the record count reads zeros.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, 0x7fffffff, 0x00020000);
}
// (The loaded vector is reinterpreted as a whole: element-wise access of the
// builtins' vector results is not reliable with this compiler.)
struct Dd { double x, y; };
struct Ff { float x, y; };
template <class T> __device__ __forceinline__ T buf_load(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so);
template <> __device__ __forceinline__ double2 buf_load<double2>(__amdgpu_buffer_rsrc_t r, unsigned vo,
                                                                 unsigned so) {
  const Dd v = __builtin_bit_cast(Dd, __builtin_amdgcn_raw_buffer_load_b128(r, (int)vo, (int)so, 0));
  double2 x;
  x.x = v.x;
  x.y = v.y;
  return x;
}
template <> __device__ __forceinline__ float2 buf_load<float2>(__amdgpu_buffer_rsrc_t r, unsigned vo,
                                                               unsigned so) {
  const Ff v = __builtin_bit_cast(Ff, __builtin_amdgcn_raw_buffer_load_b64(r, (int)vo, (int)so, 0));
  float2 x;
  x.x = v.x;
  x.y = v.y;
  return x;
}
// x or -x by a uniform sign mask (0 or the sign bit of the high word)
__device__ __forceinline__ double flip(double x, unsigned m) {
  return __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, x) ^ ((unsigned long long)m << 32));
}
__device__ __forceinline__ float flip(float x, unsigned m) {
  return __builtin_bit_cast(float, __builtin_bit_cast(unsigned, x) ^ m);
}
