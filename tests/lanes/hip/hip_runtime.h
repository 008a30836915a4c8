// The part of HIP that the library's sources use, for the CPU: every lane of a kernel is a fiber, a block runs on one host
// thread, streams and events are handles whose work is done by the time a call returns.  See ../lanes.cpp.
#pragma once
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __launch_bounds__(...)
#define __forceinline__ inline __attribute__((always_inline))
#define __shared__ static thread_local
#define __align__(n) __attribute__((aligned(n)))

struct dim3 { unsigned x, y, z; dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {} };
struct __attribute__((aligned(16))) float4 { float x, y, z, w; };
struct __attribute__((aligned(16))) uint4 { unsigned x, y, z, w; };
struct __attribute__((aligned(8))) uint2 { unsigned x, y; };
struct __attribute__((aligned(16))) int4 { int x, y, z, w; };
struct __attribute__((aligned(8))) int2 { int x, y; };
static inline float4 make_float4(float a, float b, float c, float d) { return {a, b, c, d}; }
static inline uint4 make_uint4(unsigned a, unsigned b, unsigned c, unsigned d) { return {a, b, c, d}; }
static inline uint2 make_uint2(unsigned a, unsigned b) { return {a, b}; }
static inline int4 make_int4(int a, int b, int c, int d) { return {a, b, c, d}; }
static inline int2 make_int2(int a, int b) { return {a, b}; }

// ---- the engine (lanes.cpp) ----------------------------------------------------------------------
namespace lanes {
struct Idx { unsigned x, y, z; };
extern thread_local Idx tid, bid, bdim, gdim;
extern thread_local int lane;                        // of the wavefront
void* dynamic_lds();
void barrier(int place);
// hands n bytes to the other lanes of the wavefront; returns the 64 lanes' slots of n bytes
const unsigned char* exchange(const void* mine, size_t n, int place);
void run(dim3 grid, dim3 block, size_t lds, const void* kernel, const std::function<void()>& body);
// 16 bytes per lane from a buffer to LDS address dst + 16 * lane, and the wait for all but the n youngest of them
void load_to_lds(const unsigned* rsrc, unsigned char* dst, unsigned off, unsigned soff);
void wait_loads(int n);
bool in_buffer(const unsigned char* base, unsigned records, unsigned off, unsigned soff, unsigned bytes, bool store);
int device();
int set_device(int d);
int allow_lds(const void* kernel, int bytes);
long launched();                                     // launches so far
extern thread_local long element_loads;              // ld() of a host thread's lanes
}  // namespace lanes
#define threadIdx lanes::tid
#define blockIdx lanes::bid
#define blockDim lanes::bdim
#define gridDim lanes::gdim
#define __syncthreads() lanes::barrier(__LINE__)

static inline int min(int a, int b) { return a < b ? a : b; }
static inline int max(int a, int b) { return a > b ? a : b; }
static inline unsigned min(unsigned a, unsigned b) { return a < b ? a : b; }
static inline unsigned max(unsigned a, unsigned b) { return a > b ? a : b; }
static inline int64_t min(int64_t a, int64_t b) { return a < b ? a : b; }
static inline int64_t max(int64_t a, int64_t b) { return a > b ? a : b; }
static inline float rsqrtf(float x) { return 1.0f / sqrtf(x); }
static inline float __uint_as_float(unsigned u) { float f; memcpy(&f, &u, 4); return f; }
static inline unsigned __float_as_uint(float f) { unsigned u; memcpy(&u, &f, 4); return u; }
static inline unsigned __umulhi(unsigned a, unsigned b) { return (unsigned)(((unsigned long long)a * b) >> 32); }
static inline long long wall_clock64() { static thread_local long long t = 0; return t += 100000; }

// ---- lane exchanges and ordering -----------------------------------------------------------------
template <typename T> static inline T lane_value(T v, int src, int place) {
    const unsigned char* p = lanes::exchange(&v, sizeof v, place);
    T r;
    memcpy(&r, p + (size_t)(src & 63) * sizeof v, sizeof v);
    return r;
}
#define __shfl_xor(v, o, ...) lane_value(v, lanes::lane ^ (o), __LINE__)
#define __shfl(v, s, ...) lane_value(v, s, __LINE__)
#define __builtin_amdgcn_readfirstlane(v) lane_value((int)(v), 0, __LINE__)
#define __builtin_amdgcn_wave_barrier() ((void)lane_value(0, 0, __LINE__))
#define __builtin_amdgcn_fence(...) ((void)lane_value(0, 0, __LINE__))
#define __builtin_amdgcn_s_barrier() lanes::barrier(__LINE__)
#define __builtin_amdgcn_s_waitcnt(imm) lanes::wait_loads(((imm) & 15) | ((((imm) >> 14) & 3) << 4))
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_s_sleep(x) ((void)0)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_fetch_add(p, v, order, scope) __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, __ATOMIC_SEQ_CST)
#define __builtin_nontemporal_load(p) (*(p))
#define __builtin_nontemporal_store(v, p) (*(p) = (v))
static inline unsigned lane_alignbit(unsigned hi, unsigned lo, unsigned s) { return (unsigned)((((unsigned long long)hi << 32) | lo) >> s); }
static inline unsigned lane_perm(unsigned a, unsigned b, unsigned sel) {
    const unsigned long long v = ((unsigned long long)a << 32) | b;
    unsigned r = 0;
    for (int i = 0; i < 4; ++i) r |= (unsigned)((v >> (((sel >> (8 * i)) & 7) * 8)) & 255) << (8 * i);
    return r;
}
#define __builtin_amdgcn_alignbit lane_alignbit
#define __builtin_amdgcn_perm lane_perm

// ---- buffer accesses -----------------------------------------------------------------------------
struct LaneBuffer { const unsigned char* p; unsigned n; };
typedef unsigned int lane_u4 __attribute__((ext_vector_type(4)));
#define __amdgpu_buffer_rsrc_t LaneBuffer
#define __builtin_amdgcn_make_buffer_rsrc(p, stride, n, flags) LaneBuffer{(const unsigned char*)(p), n}
template <typename T> static inline T lane_buffer_load(LaneBuffer r, unsigned off, unsigned soff) {
    T v;
    memset(&v, 0, sizeof v);
    if (lanes::in_buffer(r.p, r.n, off, soff, sizeof v, false)) memcpy(&v, r.p + off + soff, sizeof v);
    return v;
}
template <typename T> static inline void lane_buffer_store(T v, LaneBuffer r, unsigned off, unsigned soff) {
    if (lanes::in_buffer(r.p, r.n, off, soff, sizeof v, true)) memcpy(const_cast<unsigned char*>(r.p) + off + soff, &v, sizeof v);
}
#define __builtin_amdgcn_raw_buffer_load_b16(r, o, s, aux) lane_buffer_load<unsigned short>(r, o, s)
#define __builtin_amdgcn_raw_buffer_load_b32(r, o, s, aux) lane_buffer_load<unsigned>(r, o, s)
#define __builtin_amdgcn_raw_buffer_load_b128(r, o, s, aux) lane_buffer_load<lane_u4>(r, o, s)
#define __builtin_amdgcn_raw_buffer_store_b32(v, r, o, s, aux) lane_buffer_store<unsigned>(v, r, o, s)
#define __builtin_amdgcn_raw_buffer_store_b128(v, r, o, s, aux) lane_buffer_store<lane_u4>(v, r, o, s)

// ---- matrix instructions -------------------------------------------------------------------------
static inline float lane_bf16(const unsigned char* p) { unsigned short u; memcpy(&u, p, 2); return __uint_as_float((unsigned)u << 16); }
static inline float lane_f32(const unsigned char* p) { float f; memcpy(&f, p, 4); return f; }
// D = A (ROWS x K) * B (K x ROWS) + C of bf16: a lane holds 8 consecutive k of row / column lane % ROWS, and four (of every eight)
// consecutive rows of column lane % ROWS of the result
template <int ROWS, typename V, typename A> static inline A lane_mfma_bf16(V a, V b, A c, int place) {
    struct { V a, b; } m = {a, b};
    const unsigned char* p = lanes::exchange(&m, sizeof m, place);
    const int col = lanes::lane % ROWS, part = lanes::lane / ROWS, groups = 64 / ROWS;
    float bv[64 / ROWS * 8];
    for (int k = 0; k < groups * 8; ++k) bv[k] = lane_bf16(p + (size_t)(col + ROWS * (k >> 3)) * 32 + 16 + 2 * (k & 7));
    for (int i = 0; i < ROWS * ROWS / 64; ++i) {
        const int row = (i >> 2) * 4 * groups + part * 4 + (i & 3);
        float s = c[i];
        for (int k = 0; k < groups * 8; ++k) s += lane_bf16(p + (size_t)(row + ROWS * (k >> 3)) * 32 + 2 * (k & 7)) * bv[k];
        c[i] = s;
    }
    return c;
}
template <typename A> static inline A lane_mfma_f32(float a, float b, A c, int place) {
    struct { float a, b; } m = {a, b};
    const unsigned char* p = lanes::exchange(&m, sizeof m, place);
    const int col = lanes::lane & 31, part = lanes::lane >> 5;
    for (int i = 0; i < 16; ++i) {
        const int row = (i >> 2) * 8 + part * 4 + (i & 3);
        for (int k = 0; k < 2; ++k) c[i] += lane_f32(p + (size_t)(row + 32 * k) * 8) * lane_f32(p + (size_t)(col + 32 * k) * 8 + 4);
    }
    return c;
}
#define __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, x, y, z) lane_mfma_bf16<32>(a, b, c, __LINE__)
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, x, y, z) lane_mfma_bf16<16>(a, b, c, __LINE__)
#define __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, x, y, z) lane_mfma_f32(a, b, c, __LINE__)

// ---- runtime -------------------------------------------------------------------------------------
// Recording an event writes to it and waiting for it reads it, so a thread sanitizer sees whether the wait is ordered behind the
// record; it keeps how many launches it stands behind, and whether it came with the last of them.  Nothing can be captured.
typedef int hipError_t;
enum { hipSuccess = 0, hipErrorInvalidValue = 1, hipFuncAttributeMaxDynamicSharedMemorySize = 8, hipEventDisableTiming = 2, hipStreamNonBlocking = 1, hipMemcpyDeviceToDevice = 3 };
typedef struct LaneStream* hipStream_t;
typedef struct LaneEvent { int records; long behind; bool with_kernel; }* hipEvent_t;
typedef struct LaneGraph* hipGraph_t;
typedef struct LaneGraphExec* hipGraphExec_t;
typedef struct LaneGraphNode* hipGraphNode_t;
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone = 0 };
enum { hipStreamCaptureModeRelaxed = 2, hipStreamAddCaptureDependencies = 0, hipStreamSetCaptureDependencies = 1 };
static inline hipError_t hipGetLastError() { return hipSuccess; }
static inline const char* hipGetErrorString(hipError_t) { return "error"; }
static inline hipError_t hipGetDevice(int* d) { *d = lanes::device(); return hipSuccess; }
static inline hipError_t hipSetDevice(int d) { return lanes::set_device(d); }
static inline hipError_t hipFuncSetAttribute(const void* k, int, int bytes) { return lanes::allow_lds(k, bytes); }
static inline hipError_t hipEventCreate(hipEvent_t* e) { *e = new LaneEvent{0, 0, false}; return hipSuccess; }
static inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
static inline hipError_t hipEventDestroy(hipEvent_t e) { delete e; return hipSuccess; }
static inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { ++e->records; e->behind = lanes::launched(); e->with_kernel = false; return hipSuccess; }
static inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
static inline hipError_t hipEventElapsedTime(float* f, hipEvent_t, hipEvent_t) { *f = 0.01f; return hipSuccess; }
static inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)malloc(16); return hipSuccess; }
static inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
static inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t e, unsigned) { return *(volatile int*)&e->records < 0 ? hipErrorInvalidValue : hipSuccess; }
static inline hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
static inline hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, int, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
static inline hipError_t hipGetSymbolAddress(void** p, const void* s) { *p = const_cast<void*>(s); return hipSuccess; }
#define HIP_SYMBOL(x) ((const void*)(x))
static inline hipError_t hipStreamGetCaptureInfo_v2(hipStream_t, hipStreamCaptureStatus*, void*, void*, const hipGraphNode_t**, size_t*) { return hipErrorInvalidValue; }
static inline hipError_t hipStreamUpdateCaptureDependencies(hipStream_t, hipGraphNode_t*, size_t, unsigned) { return hipErrorInvalidValue; }
static inline hipError_t hipStreamBeginCapture(hipStream_t, int) { return hipErrorInvalidValue; }
static inline hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorInvalidValue; }
static inline hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, void*, void*, int) { return hipErrorInvalidValue; }
static inline hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorInvalidValue; }
static inline hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
static inline hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

template <typename K, typename... A> static inline void lane_launch(K kernel, dim3 grid, dim3 block, size_t lds, A... args) {
    lanes::run(grid, block, lds, (const void*)kernel, [=]() { kernel(args...); });
}
#define hipLaunchKernelGGL(k, g, b, lds, st, ...) lane_launch(k, g, b, lds, ##__VA_ARGS__)
#define hipExtLaunchKernelGGL(k, g, b, lds, st, e0, e1, fl, ...) (lane_launch(k, g, b, lds, ##__VA_ARGS__), (void)hipEventRecord(e1, st), (void)((e1)->with_kernel = true))
