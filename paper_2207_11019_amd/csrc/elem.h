// Element load/store helpers: float or bfloat16 storage, float arithmetic.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace lpm {

struct bf16_t { uint16_t bits; };   // storage only

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// round to nearest, ties to even; NaN stays NaN: v_cvt_pk_bf16_f32, one instruction for two values (the same in integer
// arithmetic took seven per value, a third of the epilogue instructions of a contraction)
typedef __bf16 lpm_bf2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const lpm_bf2 v = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// Streaming accesses: data touched once per kernel (parameters in the update, the fp32 gradient of a large FC
// layer) is read and written with the non-temporal hint so it does not displace reusable lines from the caches.
typedef float lpm_f4 __attribute__((ext_vector_type(4)));
typedef unsigned int lpm_u2 __attribute__((ext_vector_type(2)));
typedef unsigned int lpm_u4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 ld_stream(const float4* a) {
    const lpm_f4 t = __builtin_nontemporal_load(reinterpret_cast<const lpm_f4*>(a));
    return make_float4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ uint4 ld_stream(const uint4* a) {
    const lpm_u4 t = __builtin_nontemporal_load(reinterpret_cast<const lpm_u4*>(a));
    return make_uint4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ void st_stream(float4* a, float4 x) {
    const lpm_f4 t = {x.x, x.y, x.z, x.w};
    __builtin_nontemporal_store(t, reinterpret_cast<lpm_f4*>(a));
}
__device__ __forceinline__ void st_stream(uint2* a, uint2 x) {
    const lpm_u2 t = {x.x, x.y};
    __builtin_nontemporal_store(t, reinterpret_cast<lpm_u2*>(a));
}

// XCD-aware tile order: consecutive workgroup ids land on different XCDs (each with its own L2), so give
// every XCD one contiguous range of tiles.
__device__ __forceinline__ int xcd_remap(int bid, int nblocks) {
    const int per = nblocks >> 3, rem = nblocks & 7;
    const int xcd = bid & 7, idx = bid >> 3;
    return xcd * per + min(xcd, rem) + idx;
}

// n / d for 0 <= n < 2^31 by multiplication: 2n * mul / 2^(32 + sh), mul = ceil(2^(31 + sh) / d), sh = ceil(log2 d)
struct FastDiv { unsigned mul, sh; };
static inline FastDiv fast_div(int d) {
    FastDiv f{0, 0};
    if (d < 1) d = 1;
    f.sh = d > 1 ? 32u - (unsigned)__builtin_clz((unsigned)d - 1u) : 0u;      // (a launch makes a dozen of these)
    f.mul = (unsigned)((((uint64_t)1 << (31 + f.sh)) + d - 1) / d);
    return f;
}
__device__ __forceinline__ int div_by(int n, const FastDiv& f) { return (int)(__umulhi((unsigned)n << 1, f.mul) >> f.sh); }

__device__ __forceinline__ float ld(const float* p, int64_t i) { return p[i]; }
__device__ __forceinline__ float ld(const bf16_t* p, int64_t i) { return bf2f(p[i].bits); }
// the value as it is stored
template <typename T> __device__ __forceinline__ T to_store(float v);
template <> __device__ __forceinline__ float to_store<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t to_store<bf16_t>(float v) { return {f2bf(v)}; }
__device__ __forceinline__ void st(float* p, int64_t i, float v) { p[i] = v; }
__device__ __forceinline__ void st(bf16_t* p, int64_t i, float v) { p[i].bits = f2bf(v); }

}  // namespace lpm
