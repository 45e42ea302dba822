// Device-side global-memory accessors.
//
// Buffer pointers reach the kernels inside descriptor tables, so the compiler
// cannot tell that they point to global memory and would emit flat
// instructions.  Flat loads count against the LDS wait counter as well as the
// vector-memory one, so a wait for an LDS read would also wait for every
// outstanding prefetch.  These helpers cast to the global address space (and
// use native vector types, which the cast needs to stay a single 16-byte
// access), so every access below is a global_load / global_store.
#pragma once

#include <hip/hip_runtime.h>

namespace mkor {

#define MKOR_GLOBAL __attribute__((address_space(1)))

typedef float        mk_f4 __attribute__((ext_vector_type(4)));
typedef unsigned int mk_u4 __attribute__((ext_vector_type(4)));
typedef unsigned int mk_u2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float gld(const float* p) { return *(const MKOR_GLOBAL float*)p; }

__device__ __forceinline__ int gld_i32(const int32_t* p) { return *(const MKOR_GLOBAL int32_t*)p; }

__device__ __forceinline__ unsigned short gld_u16(const unsigned short* p) {
    return *(const MKOR_GLOBAL unsigned short*)p;
}

__device__ __forceinline__ float4 gld4(const float* p) {
    const mk_f4 v = *(const MKOR_GLOBAL mk_f4*)p;
    return make_float4(v.x, v.y, v.z, v.w);
}

// four floats at any multiple of 4 bytes: one 16-byte load all the same
typedef float mk_f4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 gld4u(const float* p) {
    const mk_f4u v = *(const MKOR_GLOBAL mk_f4u*)p;
    return make_float4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ uint4 gld_u4(const void* p) {
    const mk_u4 v = *(const MKOR_GLOBAL mk_u4*)p;
    return make_uint4(v.x, v.y, v.z, v.w);
}

// eight 16-bit values at any multiple of 2 bytes, four words at any of 4
typedef unsigned int mk_u4w __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int mk_u4h __attribute__((ext_vector_type(4), aligned(2)));
__device__ __forceinline__ uint4 gld_u4w(const void* p) {
    const mk_u4w v = *(const MKOR_GLOBAL mk_u4w*)p;
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint4 gld_u4h(const void* p) {
    const mk_u4h v = *(const MKOR_GLOBAL mk_u4h*)p;
    return make_uint4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ uint2 gld_u2(const void* p) {
    const mk_u2 v = *(const MKOR_GLOBAL mk_u2*)p;
    return make_uint2(v.x, v.y);
}

// Streaming variants (non-temporal hint: the data is not re-read soon), at any
// multiple of 4 bytes (the rows of a matrix with any row length): still one
// 16-byte access.
__device__ __forceinline__ float4 gld4_nt(const float* p) {
    const mk_f4u v = __builtin_nontemporal_load((const MKOR_GLOBAL mk_f4u*)p);
    return make_float4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ void gst4_nt(float* p, const float4& v) {
    mk_f4u w;
    w.x = v.x; w.y = v.y; w.z = v.z; w.w = v.w;
    __builtin_nontemporal_store(w, (MKOR_GLOBAL mk_f4u*)p);
}

__device__ __forceinline__ uint4 gld_u4_nt(const void* p) {
    const mk_u4 v = __builtin_nontemporal_load((const MKOR_GLOBAL mk_u4*)p);
    return make_uint4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ void gst_u4_nt(void* p, const uint4& v) {
    mk_u4 w;
    w.x = v.x; w.y = v.y; w.z = v.z; w.w = v.w;
    __builtin_nontemporal_store(w, (MKOR_GLOBAL mk_u4*)p);
}

// base (wave-uniform) + 32-bit byte offset: the form of the scalar-base
// addressing mode, so per-thread addresses need one 32-bit register.
__device__ __forceinline__ float4 gld4_off(const void* base, unsigned byte_off) {
    const mk_f4 v = *(const MKOR_GLOBAL mk_f4*)((const MKOR_GLOBAL char*)base + byte_off);
    return make_float4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ uint2 gld_u2_off(const void* base, unsigned byte_off) {
    const mk_u2 v = *(const MKOR_GLOBAL mk_u2*)((const MKOR_GLOBAL char*)base + byte_off);
    return make_uint2(v.x, v.y);
}

__device__ __forceinline__ float gld_off(const void* base, unsigned byte_off) {
    return *(const MKOR_GLOBAL float*)((const MKOR_GLOBAL char*)base + byte_off);
}

__device__ __forceinline__ void gst(float* p, float v) { *(MKOR_GLOBAL float*)p = v; }

__device__ __forceinline__ void gst_u16(unsigned short* p, unsigned short v) {
    *(MKOR_GLOBAL unsigned short*)p = v;
}

__device__ __forceinline__ void gst_u4(void* p, uint4 v) {
    mk_u4 w;
    w.x = v.x; w.y = v.y; w.z = v.z; w.w = v.w;
    *(MKOR_GLOBAL mk_u4*)p = w;
}

__device__ __forceinline__ void gst_u2(void* p, uint2 v) {
    mk_u2 w;
    w.x = v.x; w.y = v.y;
    *(MKOR_GLOBAL mk_u2*)p = w;
}

// bf16 <-> fp32.  The conversion to bf16 is the hardware's (v_cvt_pk_bf16_f32):
// round to nearest, ties to even; NaN stays NaN.
typedef __bf16 mk_bf2 __attribute__((ext_vector_type(2)));
typedef float  mk_f2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float(((unsigned)h) << 16); }

// two floats -> packed bf16 pair (a in the low half)
__device__ __forceinline__ unsigned f2bf2(float a, float b) {
    const mk_f2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, mk_bf2));
}

// two floats -> fp16 pair, round to nearest, ties to even
typedef _Float16 mk_h2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ mk_h2 f2h2(float a, float b) {
    const mk_f2 v = {a, b};
    return __builtin_convertvector(v, mk_h2);
}

__device__ __forceinline__ unsigned short f2bf(float f) {
    return __builtin_bit_cast(unsigned short, (__bf16)f);
}

__device__ __forceinline__ void gst4(float* p, const float4& v) {
    mk_f4 w;
    w.x = v.x; w.y = v.y; w.z = v.z; w.w = v.w;
    *(MKOR_GLOBAL mk_f4*)p = w;
}

__device__ __forceinline__ void gst4u(float* p, const float4& v) {   // at any multiple of 4 bytes
    mk_f4u w;
    w.x = v.x; w.y = v.y; w.z = v.z; w.w = v.w;
    *(MKOR_GLOBAL mk_f4u*)p = w;
}

// The sums over 32 lanes (each half of the wave its own) of sixteen per-lane
// values: a butterfly that halves the values a lane keeps; lanes 2 n, 2 n + 1
// end with the total of value n, in a fixed order.
__device__ __forceinline__ float row_sums16(const float (&v)[16], int lane) {
    const bool h4 = (lane & 16) != 0, h3 = (lane & 8) != 0, h2 = (lane & 4) != 0, h1 = (lane & 2) != 0;
    float a[8], b[4], c[2];
#pragma unroll
    for (int k = 0; k < 8; ++k) a[k] = (h4 ? v[k + 8] : v[k]) + __shfl_xor(h4 ? v[k] : v[k + 8], 16, 64);
#pragma unroll
    for (int k = 0; k < 4; ++k) b[k] = (h3 ? a[k + 4] : a[k]) + __shfl_xor(h3 ? a[k] : a[k + 4], 8, 64);
#pragma unroll
    for (int k = 0; k < 2; ++k) c[k] = (h2 ? b[k + 2] : b[k]) + __shfl_xor(h2 ? b[k] : b[k + 2], 4, 64);
    float d = (h1 ? c[1] : c[0]) + __shfl_xor(h1 ? c[0] : c[1], 2, 64);
    return d + __shfl_xor(d, 1, 64);
}

// The same with the maximum in place of the sum.
__device__ __forceinline__ float row_max16(const float (&v)[16], int lane) {
    const bool h4 = (lane & 16) != 0, h3 = (lane & 8) != 0, h2 = (lane & 4) != 0, h1 = (lane & 2) != 0;
    float a[8], b[4], c[2];
#pragma unroll
    for (int k = 0; k < 8; ++k) a[k] = fmaxf(h4 ? v[k + 8] : v[k], __shfl_xor(h4 ? v[k] : v[k + 8], 16, 64));
#pragma unroll
    for (int k = 0; k < 4; ++k) b[k] = fmaxf(h3 ? a[k + 4] : a[k], __shfl_xor(h3 ? a[k] : a[k + 4], 8, 64));
#pragma unroll
    for (int k = 0; k < 2; ++k) c[k] = fmaxf(h2 ? b[k + 2] : b[k], __shfl_xor(h2 ? b[k] : b[k + 2], 4, 64));
    const float d = fmaxf(h1 ? c[1] : c[0], __shfl_xor(h1 ? c[0] : c[1], 2, 64));
    return fmaxf(d, __shfl_xor(d, 1, 64));
}

// The maxima over the wave of eight per-lane values: lanes 8 r .. 8 r + 7 end
// with that of value r.
__device__ __forceinline__ float row_max8(const float (&v)[8], int lane) {
    const bool h5 = (lane & 32) != 0, h4 = (lane & 16) != 0, h3 = (lane & 8) != 0;
    float a[4], b[2];
#pragma unroll
    for (int k = 0; k < 4; ++k) a[k] = fmaxf(h5 ? v[k + 4] : v[k], __shfl_xor(h5 ? v[k] : v[k + 4], 32, 64));
#pragma unroll
    for (int k = 0; k < 2; ++k) b[k] = fmaxf(h4 ? a[k + 2] : a[k], __shfl_xor(h4 ? a[k] : a[k + 2], 16, 64));
    float c = fmaxf(h3 ? b[1] : b[0], __shfl_xor(h3 ? b[0] : b[1], 8, 64));
    c = fmaxf(c, __shfl_xor(c, 4, 64));
    c = fmaxf(c, __shfl_xor(c, 2, 64));
    return fmaxf(c, __shfl_xor(c, 1, 64));
}

}  // namespace mkor
