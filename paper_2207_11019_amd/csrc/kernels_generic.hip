// Shape-generic kernels: every layer kind, any extent, float or bf16 elements.
//
// These are the contraction kernels for what the matrix-core kernels leave (a group of lanes per output element, fp32
// accumulation: float contractions of a few hundred thousand products, heads of a few classes, long filters), plus the
// memory-bound kernels of the step: epilogue backward + bias gradient, pooling, loss, update.
// Layouts: activations [m][H][W][C], weights [Cout][Kh][Kw][Cin].
#include "lpm_internal.h"
#include "elem.h"
#include <algorithm>
#include <type_traits>

namespace lpm {

#define LPM_DISPATCH(dtype, ...)                       \
    do {                                               \
        if ((dtype) == LPM_BF16) { typedef bf16_t T; __VA_ARGS__; } \
        else { typedef float T; __VA_ARGS__; }         \
    } while (0)

static inline unsigned nblk(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

// --------------------------------------------------------------------------------------------------
// convolution forward, eq. 1 for a conv/FC layer:  y = relu?(scale*z + bias + add)
// (two- and three-dimensional: a 2-D layer has D = Do = Kd = 1)
// R lanes share an output element: lane p of the group takes the channels p, p + R, ... of every filter tap, and the R
// partial sums are added by a butterfly of lane exchanges, the same order on every run.  (One thread per element walked
// taps x channels dependent loads alone: 34 us for the 960 outputs of a 256 -> 120 fully connected layer.)
template <int R>
__device__ __forceinline__ float group_sum(float v) {
#pragma unroll
    for (int off = R / 2; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}
// lanes per element for a reduction whose innermost extent is n
static inline int group_lanes(int n) { return n >= 48 ? 64 : n >= 12 ? 16 : n >= 4 ? 4 : 1; }
#define LPM_DISPATCH_R(R_, ...)                                    \
    do {                                                           \
        if ((R_) == 64) { constexpr int R = 64; __VA_ARGS__; }     \
        else if ((R_) == 16) { constexpr int R = 16; __VA_ARGS__; } \
        else if ((R_) == 4) { constexpr int R = 4; __VA_ARGS__; }  \
        else { constexpr int R = 1; __VA_ARGS__; }                 \
    } while (0)

// How an element's index splits into channel, column, row, slice and sample: by multiplication while indices have 31 bits (a 64-bit division
// is some hundred instructions, and there are four in a launch of 3 us).
struct Split { FastDiv c, w, h, d; int small; };
static Split split_of(int c, int w, int h, int d, int64_t total) { return {fast_div(c), fast_div(w), fast_div(h), fast_div(d), total < ((int64_t)1 << 31)}; }
struct Place { int c, w, h, d, n; };
__device__ __forceinline__ Place place_of(int64_t idx, const Split& s, int C, int W, int H, int D) {
    if (s.small) {
        const int i = (int)idx, t = div_by(i, s.c), q = div_by(t, s.w), u = div_by(q, s.h), n = div_by(u, s.d);
        return {i - t * C, t - q * W, q - u * H, u - n * D, n};
    }
    Place r;
    int64_t t = idx / C;
    r.c = (int)(idx - t * C);
    r.w = (int)(t % W); t /= W;
    r.h = (int)(t % H); t /= H;
    r.d = (int)(t % D); r.n = (int)(t / D);
    return r;
}
// acc += a[k] * b[k] over the lane's k = p, p + R, ... below n, in that order.  DEEP: the loads of up to eight terms in flight, what is left of fewer
// turns in fours, twos and one.  (Eight at a time whatever the number loaded turns that do not exist, and where launches fill the card they are
// bound by their loads: 18 x 27^2, 106 -> 8 channels, 14x14, bf16, forward 790 us one by one, 2704 so, data gradient 1076 / 2834.)
template <int U, int R, bool WHOLE, typename T>
__device__ __forceinline__ float dot_turns(float acc, const T* a, const T* b, int k0, int n) {
    float va[U], vb[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int k = WHOLE ? k0 + u * R : min(k0 + u * R, n - 1);
        va[u] = ld(a, k); vb[u] = ld(b, k);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float next = fmaf(va[u], vb[u], acc);
        acc = WHOLE || k0 + u * R < n ? next : acc;
    }
    return acc;
}
template <int R, bool DEEP, typename T>
__device__ __forceinline__ float dot(float acc, const T* a, const T* b, int p, int n) {
    if (!DEEP) {
        for (int k = p; k < n; k += R) acc = fmaf(ld(a, k), ld(b, k), acc);
        return acc;
    }
    constexpr bool WHOLE = R == 1;
    int k = p, left = (n + R - 1) / R;             // turns
    for (; left > 8; left -= 8, k += 8 * R) acc = dot_turns<8, R, true>(acc, a, b, k, n);
    if (left == 8) return dot_turns<8, R, WHOLE>(acc, a, b, k, n);
    if (left & 4) { acc = dot_turns<4, R, WHOLE>(acc, a, b, k, n); k += 4 * R; }
    if (left & 2) { acc = dot_turns<2, R, WHOLE>(acc, a, b, k, n); k += 2 * R; }
    if (left & 1) acc = dot_turns<1, R, WHOLE>(acc, a, b, k, n);
    return acc;
}

template <typename T, int R, bool DEEP>
__global__ void __launch_bounds__(256) conv_fwd_generic(ConvGeom g, Split sp, const T* __restrict__ x, const T* __restrict__ w,
                                                        const float* __restrict__ scale, const float* __restrict__ bias,
                                                        const T* __restrict__ add, int relu, T* __restrict__ y) {
    const int64_t total = g.rows_out() * g.Cout;
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int p = (int)(gid % R);
    const bool live = gid / R < total;          // (a group is live or idle as a whole; idle groups still take part in the exchange)
    const int64_t idx = live ? gid / R : 0;
    const Place at = place_of(idx, sp, g.Cout, g.Wo, g.Ho, g.Do);
    const int co = at.c, wo = at.w, ho = at.h, dq = at.d, n = at.n;
    float acc = 0.f;
    for (int kd = 0; kd < g.Kd; ++kd) {
        const int d = dq * g.stride + kd - g.pad_d;
        if (d < 0 || d >= g.D) continue;
        for (int kh = 0; kh < g.Kh; ++kh) {
            const int h = ho * g.stride + kh - g.pad;
            if (h < 0 || h >= g.H) continue;
            for (int kw = 0; kw < g.Kw; ++kw) {
                const int ww = wo * g.stride + kw - g.pad;
                if (ww < 0 || ww >= g.W) continue;
                const T* xp = x + ((((int64_t)n * g.D + d) * g.H + h) * g.W + ww) * g.Cin;
                const T* wp = w + ((((int64_t)co * g.Kd + kd) * g.Kh + kh) * g.Kw + kw) * g.Cin;
                acc = dot<R, DEEP>(acc, xp, wp, p, g.Cin);
            }
        }
    }
    acc = group_sum<R>(acc);
    if (!live || p) return;
    if (scale) acc *= scale[co];
    if (bias) acc += bias[co];
    if (add) acc += ld(add, idx);
    if (relu) acc = fmaxf(acc, 0.f);
    st(y, idx, acc);
}

hipError_t conv_fwd_generic_launch(int dtype, const ConvGeom& g_, const void* x, const void* w, const float* scale,
                                   const float* bias, const void* add, int relu, void* y, hipStream_t s) {
    const int64_t total = g_.rows_out() * g_.Cout;
    const int lanes = group_lanes(g_.Cin);
    // A filter that covers its input, whose taps are whole turns of the lanes, is one tap of all its channels: the same terms in the
    // same order, eight of them in flight instead of one (a 4x4x16 -> 120 fully connected layer at 8 samples).
    ConvGeom g = g_;
    if (g.covers_input() && g.Cin % lanes == 0)
        g = ConvGeom{g.m, 1, 1, g.K(), 1, 1, g.Cout, 1, 1, 1, 0};
    // DEEP where there is one tap to wait for; tap after tap the choice of a block costs more than it hides.  One by one / so, us: 1 x 4095 -> 33
    // 9.5 / 4.5, 16 x 2047 -> 10 6.0 / 4.4, 100 x 20^2 x 301 -> 7 26.6 / 26.4; of 14x14 taps, 18 x 27^2, 106 -> 8, 790 / 1197.
    const bool deep = g.taps() == 1 && g.Cin > lanes;
    LPM_DISPATCH_R(lanes, LPM_DISPATCH(dtype, launch_last(deep ? conv_fwd_generic<T, R, true> : conv_fwd_generic<T, R, false>, dim3(nblk(total * R, 256)), dim3(256), 0, s, g, split_of(g.Cout, g.Wo, g.Ho, g.Do, total),
                                                                 (const T*)x, (const T*)w, scale, bias, (const T*)add, relu, (T*)y)));
    return hipGetLastError();
}

// --------------------------------------------------------------------------------------------------
// data gradient, eq. 9: dx[n,h,w,ci] (+)= sum_{kh,kw,co} dz[n,(h+p-kh)/s,(w+p-kw)/s,co] * w[co,kh,kw,ci]
// (R lanes per element, each taking the output channels p, p + R, ... of every tap.  The quotient by the stride is a multiplication, also where the
// stride is 1: a test for that ahead of each division, us: 27 x 3^2, 8 -> 1 channels, 13x13, stride 3 10.3, division alone 8.5, so 7.3.)
template <typename T, int R>
__global__ void __launch_bounds__(256) conv_dgrad_generic(ConvGeom g, Split sp, FastDiv by_stride, const T* __restrict__ dz, const float* __restrict__ dzscale,
                                                          const T* __restrict__ w, T* __restrict__ dx, int accumulate,
                                                          const T* __restrict__ mask, const float* __restrict__ mscale) {
    const int64_t total = g.rows_in() * g.Cin;
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int p = (int)(gid % R);
    const bool live = gid / R < total;
    const int64_t idx = live ? gid / R : 0;
    const Place at = place_of(idx, sp, g.Cin, g.W, g.H, g.D);
    const int ci = at.c, ww = at.w, h = at.h, d = at.d, n = at.n;
    const int64_t wstride = (int64_t)g.taps() * g.Cin;
    float acc = 0.f;
    for (int kd = 0; kd < g.Kd; ++kd) {
        const int dd = d + g.pad_d - kd;
        const int dq = div_by(dd, by_stride);
        if (dd < 0 || dq * g.stride != dd || dq >= g.Do) continue;
        for (int kh = 0; kh < g.Kh; ++kh) {
            const int hh = h + g.pad - kh;
            const int ho = div_by(hh, by_stride);
            if (hh < 0 || ho * g.stride != hh || ho >= g.Ho) continue;
            for (int kw = 0; kw < g.Kw; ++kw) {
                const int wq = ww + g.pad - kw;
                const int wo = div_by(wq, by_stride);
                if (wq < 0 || wo * g.stride != wq || wo >= g.Wo) continue;
                const T* dp = dz + ((((int64_t)n * g.Do + dq) * g.Ho + ho) * g.Wo + wo) * g.Cout;
                const T* wp = w + (((int64_t)kd * g.Kh + kh) * g.Kw + kw) * g.Cin + ci;
                if (dzscale) { for (int co = p; co < g.Cout; co += R) acc = fmaf(ld(dp, co) * dzscale[co], ld(wp, co * wstride), acc); }
                else { for (int co = p; co < g.Cout; co += R) acc = fmaf(ld(dp, co), ld(wp, co * wstride), acc); }
            }
        }
    }
    acc = group_sum<R>(acc);
    if (!live || p) return;
    if (accumulate) acc += ld(dx, idx);
    if (mask && !(ld(mask, idx) > 0.f)) acc = 0.f;
    if (mscale) acc *= mscale[ci];
    st(dx, idx, acc);
}

hipError_t conv_dgrad_generic_launch(int dtype, const ConvGeom& g, const void* dz, const float* dzscale, const void* w, void* dx,
                                     int accumulate, const void* mask, const float* mscale, hipStream_t s) {
    const int64_t total = g.rows_in() * g.Cin;
    const int lanes = group_lanes(g.Cout);
    LPM_DISPATCH_R(lanes, LPM_DISPATCH(dtype, launch_last(conv_dgrad_generic<T, R>, dim3(nblk(total * R, 256)), dim3(256), 0, s, g, split_of(g.Cin, g.W, g.H, g.D, total), fast_div(g.stride),
                                                                 (const T*)dz, dzscale, (const T*)w, (T*)dx, accumulate, (const T*)mask, mscale)));
    return hipGetLastError();
}

// --------------------------------------------------------------------------------------------------
// weight gradient, eq. 8: dw[co,kh,kw,ci] (+)= sum_{n,ho,wo} dz[n,ho,wo,co] * x[n,ho*s+kh-p,wo*s+kw-p,ci]
// The (n,ho) range is split into `chunks` slices (blockIdx.y); with more than one slice each writes a
// partial to ws[chunk][Cout*K] and a second kernel adds the partials in slice order (no float atomics,
// so the result does not depend on scheduling).  Within a slice R lanes share an element: lane p takes the
// lines p, p + R, ... and the group adds its partial sums by lane exchanges in a fixed order.
template <typename T, int R>
__global__ void __launch_bounds__(256) conv_wgrad_generic(ConvGeom g, const T* __restrict__ x, const T* __restrict__ dz,
                                                          float* __restrict__ out, int chunks, int accumulate) {
    const int K = g.K();
    const int64_t total = (int64_t)g.Cout * K;
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int p = (int)(gid % R);
    const bool live = gid / R < total;
    const int64_t idx = live ? gid / R : 0;
    const int ci = (int)(idx % g.Cin);
    int64_t t = idx / g.Cin;
    const int kw = (int)(t % g.Kw); t /= g.Kw;
    const int kh = (int)(t % g.Kh); t /= g.Kh;
    const int kd = (int)(t % g.Kd);
    const int co = (int)(t / g.Kd);
    const int nho = g.m * g.Do * g.Ho;                 // lines of Wo output pixels: (n, do, ho)
    const int per = (nho + chunks - 1) / chunks;
    const int r0 = blockIdx.y * per, r1 = min(nho, r0 + per);
    float acc = 0.f;
    for (int r = r0 + p; r < r1; r += R) {
        const int ho = r % g.Ho, nd = r / g.Ho, dq = nd % g.Do, n = nd / g.Do;
        const int h = ho * g.stride + kh - g.pad, d = dq * g.stride + kd - g.pad_d;
        if (h < 0 || h >= g.H || d < 0 || d >= g.D) continue;
        const T* dp = dz + ((int64_t)r * g.Wo) * g.Cout + co;
        const T* xp = x + ((((int64_t)n * g.D + d) * g.H + h) * g.W) * g.Cin + ci;
        for (int wo = 0; wo < g.Wo; ++wo) {
            const int ww = wo * g.stride + kw - g.pad;
            if (ww < 0 || ww >= g.W) continue;
            acc = fmaf(ld(dp, (int64_t)wo * g.Cout), ld(xp, (int64_t)ww * g.Cin), acc);
        }
    }
    acc = group_sum<R>(acc);
    if (!live || p) return;
    if (chunks > 1) out[(int64_t)blockIdx.y * total + idx] = acc;
    else out[idx] = accumulate ? out[idx] + acc : acc;
}

// dst[i] (+)= sum_{c<chunks} part[c][i], added in slice order
__global__ void __launch_bounds__(256) reduce_partials(const float* __restrict__ part, float* __restrict__ dst,
                                                       int64_t n, int chunks, int accumulate) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float acc = part[i];
    for (int c = 1; c < chunks; ++c) acc += part[(int64_t)c * n + i];
    dst[i] = accumulate ? dst[i] + acc : acc;
}

hipError_t reduce_partials_launch(const float* part, float* dst, int64_t n, int chunks, int accumulate, hipStream_t s) {
    hipLaunchKernelGGL(reduce_partials, dim3(nblk(n, 256)), dim3(256), 0, s, part, dst, n, chunks, accumulate);
    return hipGetLastError();
}

static int wgrad_generic_lanes(const ConvGeom& g) { return group_lanes(g.m * g.Do * g.Ho); }

static int wgrad_generic_chunks(const ConvGeom& g) {
    const int64_t total = (int64_t)g.Cout * g.K();
    const int nho = g.m * g.Do * g.Ho;
    int64_t c = ((int64_t)1 << 22) / total;     // keep the partials within a few MB
    const int64_t want = (nho + 4 * wgrad_generic_lanes(g) - 1) / (4 * wgrad_generic_lanes(g));      // a lane walks at most 4 (n,ho) lines
    if (c > want) c = want;
    if (c > 256) c = 256;
    if (c > nho) c = nho;
    if (c < 1) c = 1;
    return (int)c;
}

size_t wgrad_generic_ws_bytes(const ConvGeom& g) {
    const int c = wgrad_generic_chunks(g);
    return c > 1 ? (size_t)c * g.Cout * g.K() * sizeof(float) : 0;
}

hipError_t conv_wgrad_generic_launch(int dtype, const ConvGeom& g, const void* x, const void* dz, float* dw,
                                     int accumulate, void* ws, hipStream_t s) {
    const int64_t total = (int64_t)g.Cout * g.K();
    const int chunks = wgrad_generic_chunks(g);
    float* out = chunks > 1 ? (float*)ws : dw;
    const int lanes = wgrad_generic_lanes(g);
    LPM_DISPATCH_R(lanes, LPM_DISPATCH(dtype, hipLaunchKernelGGL((conv_wgrad_generic<T, R>), dim3(nblk(total * R, 256), chunks), dim3(256), 0, s, g,
                                                                 (const T*)x, (const T*)dz, out, chunks, accumulate)));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || chunks == 1) return e;
    return reduce_partials_launch((const float*)ws, dw, total, chunks, accumulate, s);
}

// --------------------------------------------------------------------------------------------------
// epilogue backward (eqs. 8-9 through y = relu(scale*z + bias + add)):
//   gm = dy * [y > 0];  dz = gm * scale_c;  gadd (+)= gm;  dbias_c (+)= sum_rows gm
// A thread owns V consecutive channels (16 bytes; V = 1 where the channel count is no multiple of that) of four rows at a
// time, all of whose loads are requested before the first is used.  The block's 256 threads are split into channel chunks and
// row lanes by the channel count (cl_log: log2 of the chunks), so six channels keep as many threads busy as 64.  A block
// covers epi_rows() rows and leaves one partial per channel, which bias_reduce adds in block order.
// (Float, 8192 x 64: 18 -> 4 us; a thread used to walk 32 rows, one 4-byte load at a time.)
template <typename T, int V> struct EpiVec;
template <typename T> struct EpiVec<T, 1> {
    static __device__ __forceinline__ void get(const T* p, int64_t i, float (&f)[1]) { f[0] = ld(p, i); }
    static __device__ __forceinline__ void put(T* p, int64_t i, const float (&f)[1]) { st(p, i, f[0]); }
};
template <> struct EpiVec<float, 4> {
    static __device__ __forceinline__ void get(const float* p, int64_t i, float (&f)[4]) {
        const float4 v = *reinterpret_cast<const float4*>(p + i);
        f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    }
    static __device__ __forceinline__ void put(float* p, int64_t i, const float (&f)[4]) { *reinterpret_cast<float4*>(p + i) = make_float4(f[0], f[1], f[2], f[3]); }
};
template <> struct EpiVec<bf16_t, 8> {
    static __device__ __forceinline__ void get(const bf16_t* p, int64_t i, float (&f)[8]) {
        const uint4 v = *reinterpret_cast<const uint4*>(p + i);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) { f[2 * k] = bf2f((uint16_t)(w[k] & 0xffffu)); f[2 * k + 1] = bf2f((uint16_t)(w[k] >> 16)); }
    }
    static __device__ __forceinline__ void put(bf16_t* p, int64_t i, const float (&f)[8]) {
        *reinterpret_cast<uint4*>(p + i) = make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
    }
};

static inline int epi_chunks_log(int C, int V) {           // channel chunks side by side in a block
    int l = 0;
    while (l < (V == 8 ? 3 : V == 4 ? 4 : 6) && (V << l) < C) ++l;
    return l;
}
static inline int epi_rows(int cl_log) { return std::max(64, 4 * (256 >> cl_log)); }

template <typename T, int V>
__global__ void __launch_bounds__(256) epilogue_bwd_kernel(int64_t rows, int C, int cl_log, int block_rows, const T* __restrict__ dy,
                                                           const T* __restrict__ y, const float* __restrict__ scale,
                                                           T* __restrict__ dz, T* __restrict__ gadd, int gadd_acc,
                                                           float* __restrict__ part) {
    __shared__ float red[256 * V + 256];
    typedef EpiVec<T, V> Vec;
    const int CL = 1 << cl_log, RL = 256 >> cl_log, cx = threadIdx.x & (CL - 1), ty = threadIdx.x >> cl_log;
    const int cb = blockIdx.x * CL * V, c0 = cb + cx * V;
    const int64_t r0 = (int64_t)blockIdx.y * block_rows, r1 = min(rows, r0 + block_rows);
    float sum[V];
#pragma unroll
    for (int k = 0; k < V; ++k) sum[k] = 0.f;
    if (c0 < C) {
        float sc[V];
#pragma unroll
        for (int k = 0; k < V; ++k) sc[k] = scale ? scale[c0 + k] : 1.f;
        for (int64_t rr = r0 + ty; rr < r1; rr += 4 * RL) {
            float g[4][V], yv[4][V], av[4][V];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t r = rr + u * RL, i = (r < r1 ? r : rr) * C + c0;
                Vec::get(dy, i, g[u]);
                if (y) Vec::get(y, i, yv[u]);
                if (gadd && gadd_acc) Vec::get(gadd, i, av[u]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t r = rr + u * RL, i = r * C + c0;
                if (r >= r1) continue;
                float z[V];
#pragma unroll
                for (int k = 0; k < V; ++k) {
                    if (y && !(yv[u][k] > 0.f)) g[u][k] = 0.f;
                    sum[k] += g[u][k];
                    z[k] = g[u][k] * sc[k];
                }
                if (dz) Vec::put(dz, i, z);
                if (gadd) {
                    if (gadd_acc) {
#pragma unroll
                        for (int k = 0; k < V; ++k) g[u][k] += av[u][k];
                    }
                    Vec::put(gadd, i, g[u]);
                }
            }
        }
    }
    if (!part) return;
    const int pitch = CL * V + 1;
#pragma unroll
    for (int k = 0; k < V; ++k) red[ty * pitch + cx * V + k] = sum[k];
    __syncthreads();
    if ((int)threadIdx.x < CL * V && cb + (int)threadIdx.x < C) {
        float acc = 0.f;
#pragma unroll 8
        for (int r = 0; r < RL; ++r) acc += red[r * pitch + threadIdx.x];
        part[(int64_t)blockIdx.y * C + cb + threadIdx.x] = acc;
    }
}

// The same without a bias gradient: nothing ties a thread to a channel column, so thread i simply takes the i-th
// 16-byte chunk of the tensor -- a wavefront covers 1 KiB of consecutive memory, and small tensors still spread over
// many blocks (ResNet-18/CIFAR: 6.8 -> about 3.5 us per launch, twelve launches per micro-batch on the data-phase chain).
__global__ void __launch_bounds__(256) epilogue_bwd_flat_bf16x8(unsigned chunks, unsigned C8, const uint4* __restrict__ dy,
                                                                const uint4* __restrict__ y, const float* __restrict__ scale,
                                                                uint4* __restrict__ dz, uint4* __restrict__ gadd, int gadd_acc) {
    const unsigned i = blockIdx.x * 256u + threadIdx.x;
    if (i >= chunks) return;
    const uint4 g4 = dy[i];
    const uint4 y4 = y ? y[i] : make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
    const uint4 a4 = (gadd && gadd_acc) ? gadd[i] : make_uint4(0, 0, 0, 0);
    float sc[8] = {1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f};
    if (scale) {                                   // two 16-byte loads: the chunk's first channel is a multiple of 8
        const float* sp = scale + (i % C8) * 8u;
        const float4 lo = *reinterpret_cast<const float4*>(sp), hi = *reinterpret_cast<const float4*>(sp + 4);
        sc[0] = lo.x; sc[1] = lo.y; sc[2] = lo.z; sc[3] = lo.w; sc[4] = hi.x; sc[5] = hi.y; sc[6] = hi.z; sc[7] = hi.w;
    }
    const uint32_t gw[4] = {g4.x, g4.y, g4.z, g4.w}, yw[4] = {y4.x, y4.y, y4.z, y4.w}, aw[4] = {a4.x, a4.y, a4.z, a4.w};
    uint32_t zo[4], go[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float g0 = bf2f((uint16_t)(gw[k] & 0xffffu)), g1 = bf2f((uint16_t)(gw[k] >> 16));
        if (!(bf2f((uint16_t)(yw[k] & 0xffffu)) > 0.f)) g0 = 0.f;
        if (!(bf2f((uint16_t)(yw[k] >> 16)) > 0.f)) g1 = 0.f;
        zo[k] = pack_bf16x2(g0 * sc[2 * k], g1 * sc[2 * k + 1]);
        go[k] = pack_bf16x2(g0 + bf2f((uint16_t)(aw[k] & 0xffffu)), g1 + bf2f((uint16_t)(aw[k] >> 16)));
    }
    if (dz) dz[i] = make_uint4(zo[0], zo[1], zo[2], zo[3]);
    if (gadd) gadd[i] = make_uint4(go[0], go[1], go[2], go[3]);
}

// db[c] (+)= sum over the row blocks' partials; 16 lanes per channel, each a contiguous part of the blocks in order, the
// lanes' sums added in lane order
__global__ void __launch_bounds__(256) bias_reduce(const float* __restrict__ part, float* __restrict__ db, int C,
                                                   int nblocks, int accumulate) {
    __shared__ float red[16][17];
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int c = blockIdx.x * 16 + tx;
    float acc = 0.f;
    if (c < C) {
        const int per = (nblocks + 15) / 16;
        const int b1 = min(nblocks, (ty + 1) * per);
#pragma unroll 8
        for (int b = ty * per; b < b1; ++b) acc += part[(int64_t)b * C + c];
    }
    red[ty][tx] = acc;
    __syncthreads();
    if (ty == 0 && c < C) {
        float v = red[0][tx];
#pragma unroll
        for (int k = 1; k < 16; ++k) v += red[k][tx];
        db[c] = accumulate ? db[c] + v : v;
    }
}

size_t epi_bwd_ws_bytes(int64_t rows, int32_t C) { return (size_t)nblk(rows, 64) * C * sizeof(float); }

template <typename T, int V>
static unsigned epi_launch(int64_t rows, int32_t C, const void* dy, const void* y, const float* scale, void* dz, void* gadd, int gadd_acc, float* part, hipStream_t s) {
    const int cl = epi_chunks_log(C, V);
    int br = epi_rows(cl);
    while (nblk(rows, br) > 32768) br *= 2;            // (the grid's second extent is limited)
    const unsigned rb = nblk(rows, br);
    hipLaunchKernelGGL((epilogue_bwd_kernel<T, V>), dim3(nblk(C, V << cl), rb), dim3(256), 0, s, rows, C, cl, br, (const T*)dy, (const T*)y, scale,
                       (T*)dz, (T*)gadd, gadd_acc, part);
    return rb;
}

hipError_t launch_epilogue_bwd(int dtype, int64_t rows, int32_t C, const void* dy, const void* y, const float* scale,
                               void* dz, void* gadd, int gadd_acc, float* dbias, int db_acc, void* ws, hipStream_t s) {
    float* part = dbias ? (float*)ws : nullptr;
    if (dtype == LPM_BF16 && (C & 7) == 0 && !dbias && rows * (C >> 3) < ((int64_t)1 << 31)) {
        const unsigned chunks = (unsigned)(rows * (C >> 3));
        hipLaunchKernelGGL(epilogue_bwd_flat_bf16x8, dim3((chunks + 255u) / 256u), dim3(256), 0, s, chunks, (unsigned)(C >> 3),
                           (const uint4*)dy, (const uint4*)y, scale, (uint4*)dz, (uint4*)gadd, gadd_acc);
        return hipGetLastError();
    }
    unsigned rb;
    if (dtype == LPM_BF16) rb = (C & 7) == 0 ? epi_launch<bf16_t, 8>(rows, C, dy, y, scale, dz, gadd, gadd_acc, part, s) : epi_launch<bf16_t, 1>(rows, C, dy, y, scale, dz, gadd, gadd_acc, part, s);
    else rb = (C & 3) == 0 ? epi_launch<float, 4>(rows, C, dy, y, scale, dz, gadd, gadd_acc, part, s) : epi_launch<float, 1>(rows, C, dy, y, scale, dz, gadd, gadd_acc, part, s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !dbias) return e;
    hipLaunchKernelGGL(bias_reduce, dim3(nblk(C, 16)), dim3(256), 0, s, (const float*)part, dbias, C, (int)rb, db_acc);
    return hipGetLastError();
}

// --------------------------------------------------------------------------------------------------
// 2x2/2 max pooling
template <typename T>
__global__ void __launch_bounds__(256) maxpool_fwd_kernel(int m, int H, int W, int C, Split sp, const T* __restrict__ x,
                                                          T* __restrict__ y) {
    const int Ho = H / 2, Wo = W / 2;
    const int64_t total = (int64_t)m * Ho * Wo * C;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const Place at = place_of(idx, sp, C, Wo, Ho, 1);
    const int c = at.c, wo = at.w, ho = at.h, n = at.n;
    const T* p = x + (((int64_t)n * H + 2 * ho) * W + 2 * wo) * C + c;
    const float a = ld(p, 0), b = ld(p, C), d = ld(p, (int64_t)W * C), e = ld(p, (int64_t)W * C + C);
    st(y, idx, fmaxf(fmaxf(a, b), fmaxf(d, e)));
}

// gradient to the first element (row-major in the window) equal to the window maximum
template <typename T>
__global__ void __launch_bounds__(256) maxpool_bwd_kernel(int m, int H, int W, int C, Split sp, const T* __restrict__ x,
                                                          const T* __restrict__ y, const T* __restrict__ dy,
                                                          T* __restrict__ dx, int accumulate, int mask,
                                                          const float* __restrict__ mscale) {
    const int Ho = H / 2, Wo = W / 2;
    const int64_t total = (int64_t)m * Ho * Wo * C;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const Place at = place_of(idx, sp, C, Wo, Ho, 1);
    const int c = at.c, wo = at.w, ho = at.h, n = at.n;
    const int64_t base = (((int64_t)n * H + 2 * ho) * W + 2 * wo) * C + c;
    const int64_t off[4] = {0, C, (int64_t)W * C, (int64_t)W * C + C};
    const float mx = ld(y, idx);
    float g = ld(dy, idx), xin[4], old[4];               // (all loads before the first use: eight latencies one after the other otherwise)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        xin[k] = ld(x, base + off[k]);
        old[k] = accumulate ? ld(dx, base + off[k]) : 0.f;
    }
    if (mask && !(mx > 0.f)) g = 0.f;        // the pooled tensor is a ReLU output: its mask at the maximum
    if (mscale) g *= mscale[c];
    bool found = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool hit = !found && xin[k] == mx;
        found = found || hit;
        const float v = hit ? g : 0.f;
        st(dx, base + off[k], accumulate ? v + old[k] : v);
    }
}

// bf16 with C a multiple of 8: a thread takes 8 channels of one pooled pixel with 16-byte accesses (the element-wise
// kernels above issue a 2-byte access per tensor and thread).  Same arithmetic and the same first-maximum rule.
__device__ __forceinline__ void unpack8x(const uint4 v, float (&f)[8]) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) { f[2 * k] = bf2f((uint16_t)(w[k] & 0xffffu)); f[2 * k + 1] = bf2f((uint16_t)(w[k] >> 16)); }
}
__device__ __forceinline__ uint4 pack8x(const float (&f)[8]) {
    return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
}

__global__ void __launch_bounds__(256) maxpool_fwd_bf16x8(unsigned total8, int H, int W, int C8, const uint4* __restrict__ x,
                                                          uint4* __restrict__ y) {
    const unsigned idx = blockIdx.x * 256u + threadIdx.x;
    if (idx >= total8) return;
    const unsigned Ho = H / 2, Wo = W / 2;
    const unsigned c = idx % (unsigned)C8, r = idx / (unsigned)C8;
    const unsigned wo = r % Wo, ho = (r / Wo) % Ho, n = r / (Wo * Ho);
    const size_t base = ((size_t)(n * H + 2 * ho) * W + 2 * wo) * C8 + c;
    float a[8], b[8], d[8], e[8], o[8];
    unpack8x(x[base], a); unpack8x(x[base + C8], b);
    unpack8x(x[base + (size_t)W * C8], d); unpack8x(x[base + (size_t)W * C8 + C8], e);
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = fmaxf(fmaxf(a[k], b[k]), fmaxf(d[k], e[k]));
    y[idx] = pack8x(o);
}

__global__ void __launch_bounds__(256) maxpool_bwd_bf16x8(unsigned total8, int H, int W, int C8, const uint4* __restrict__ x,
                                                          const uint4* __restrict__ y, const uint4* __restrict__ dy,
                                                          uint4* __restrict__ dx, int accumulate, int mask,
                                                          const float* __restrict__ mscale) {
    const unsigned idx = blockIdx.x * 256u + threadIdx.x;
    if (idx >= total8) return;
    const unsigned Ho = H / 2, Wo = W / 2;
    const unsigned c = idx % (unsigned)C8, r = idx / (unsigned)C8;
    const unsigned wo = r % Wo, ho = (r / Wo) % Ho, n = r / (Wo * Ho);
    const size_t base = ((size_t)(n * H + 2 * ho) * W + 2 * wo) * C8 + c;
    const size_t off[4] = {0, (size_t)C8, (size_t)W * C8, (size_t)W * C8 + C8};
    float mx[8], g[8], xin[4][8], old[4][8];
    unpack8x(y[idx], mx);
    unpack8x(dy[idx], g);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        unpack8x(x[base + off[k]], xin[k]);
        if (accumulate) unpack8x(dx[base + off[k]], old[k]);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (mask && !(mx[j] > 0.f)) g[j] = 0.f;        // the pooled tensor is a ReLU output: its mask at the maximum
        if (mscale) g[j] *= mscale[c * 8 + j];
    }
    float out[4][8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        bool found = false;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool hit = !found && (xin[k][j] == mx[j]);
            found = found || hit;
            float v = hit ? g[j] : 0.f;
            if (accumulate) v += old[k][j];
            out[k][j] = v;
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) dx[base + off[k]] = pack8x(out[k]);
}

hipError_t launch_maxpool_fwd(int dtype, int32_t m, int32_t H, int32_t W, int32_t C, const void* x, void* y, hipStream_t s) {
    const int64_t total = (int64_t)m * (H / 2) * (W / 2) * C;
    if (dtype == LPM_BF16 && (C & 7) == 0 && (int64_t)m * H * W * C < ((int64_t)1 << 31)) {
        const unsigned total8 = (unsigned)(total / 8);
        hipLaunchKernelGGL(maxpool_fwd_bf16x8, dim3((total8 + 255u) / 256u), dim3(256), 0, s, total8, H, W, C / 8, (const uint4*)x, (uint4*)y);
        return hipGetLastError();
    }
    LPM_DISPATCH(dtype, hipLaunchKernelGGL(maxpool_fwd_kernel<T>, dim3(nblk(total, 256)), dim3(256), 0, s, m, H, W, C, split_of(C, W / 2, H / 2, 1, total),
                                           (const T*)x, (T*)y));
    return hipGetLastError();
}

hipError_t launch_maxpool_bwd(int dtype, int32_t m, int32_t H, int32_t W, int32_t C, const void* x, const void* y,
                              const void* dy, void* dx, int accumulate, int mask, const float* mscale, hipStream_t s) {
    const int64_t total = (int64_t)m * (H / 2) * (W / 2) * C;
    if (dtype == LPM_BF16 && (C & 7) == 0 && (int64_t)m * H * W * C < ((int64_t)1 << 31)) {
        const unsigned total8 = (unsigned)(total / 8);
        launch_last(maxpool_bwd_bf16x8, dim3((total8 + 255u) / 256u), dim3(256), 0, s, total8, H, W, C / 8, (const uint4*)x,
                           (const uint4*)y, (const uint4*)dy, (uint4*)dx, accumulate, mask, mscale);
        return hipGetLastError();
    }
    LPM_DISPATCH(dtype, launch_last(maxpool_bwd_kernel<T>, dim3(nblk(total, 256)), dim3(256), 0, s, m, H, W, C, split_of(C, W / 2, H / 2, 1, total),
                                           (const T*)x, (const T*)y, (const T*)dy, (T*)dx, accumulate, mask, mscale));
    return hipGetLastError();
}

// --------------------------------------------------------------------------------------------------
// global average pooling
// A block takes one sample and a chunk of channels, 16 bytes of them per thread where the count allows; its row lanes share the
// positions and meet in LDS.  (A thread per channel walked all positions: 17 us for 512 of them, 4 now.)
template <typename T, int V>
__global__ void __launch_bounds__(256) gap_fwd_kernel(int HW, int C, int cl_log, const T* __restrict__ x, T* __restrict__ y) {
    __shared__ float red[256 * V + 256];
    const int CL = 1 << cl_log, RL = 256 >> cl_log, cx = threadIdx.x & (CL - 1), ty = threadIdx.x >> cl_log;
    const int cb = blockIdx.x * CL * V, c0 = cb + cx * V, pitch = CL * V + 1;
    const T* xs = x + (int64_t)blockIdx.y * HW * C;
    float sum[V];
#pragma unroll
    for (int k = 0; k < V; ++k) sum[k] = 0.f;
    if (c0 < C) {
        for (int r = ty; r < HW; r += 4 * RL) {
            float v[4][V];
#pragma unroll
            for (int u = 0; u < 4; ++u) EpiVec<T, V>::get(xs, (int64_t)min(r + u * RL, HW - 1) * C + c0, v[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (r + u * RL < HW) {
#pragma unroll
                    for (int k = 0; k < V; ++k) sum[k] += v[u][k];
                }
        }
    }
#pragma unroll
    for (int k = 0; k < V; ++k) red[ty * pitch + cx * V + k] = sum[k];
    __syncthreads();
    if ((int)threadIdx.x < CL * V && cb + (int)threadIdx.x < C) {
        float acc = 0.f;
#pragma unroll 8
        for (int r = 0; r < RL; ++r) acc += red[r * pitch + threadIdx.x];
        st(y, (int64_t)blockIdx.y * C + cb + threadIdx.x, acc / (float)HW);
    }
}

template <typename T>
__global__ void __launch_bounds__(256) gap_bwd_kernel(int m, int HW, int C, const T* __restrict__ dy, T* __restrict__ dx,
                                                      int accumulate, const T* __restrict__ mask,
                                                      const float* __restrict__ mscale) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)m * HW * C) return;
    const int c = (int)(idx % C), n = (int)(idx / ((int64_t)HW * C));
    float v = ld(dy, (int64_t)n * C + c) / (float)HW;
    if (accumulate) v += ld(dx, idx);
    if (mask && !(ld(mask, idx) > 0.f)) v = 0.f;
    if (mscale) v *= mscale[c];
    st(dx, idx, v);
}

template <typename T, int V>
static void gap_launch(int32_t m, int32_t HW, int32_t C, const void* x, void* y, hipStream_t s) {
    const int cl = epi_chunks_log(C, V);
    for (int n0 = 0; n0 < m; n0 += 32768)          // (the grid's second extent is limited)
        hipLaunchKernelGGL((gap_fwd_kernel<T, V>), dim3(nblk(C, V << cl), (unsigned)std::min(m - n0, 32768)), dim3(256), 0, s, HW, C, cl,
                           (const T*)x + (int64_t)n0 * HW * C, (T*)y + (int64_t)n0 * C);
}

hipError_t launch_gap_fwd(int dtype, int32_t m, int32_t HW, int32_t C, const void* x, void* y, hipStream_t s) {
    if (dtype == LPM_BF16) { if (C % 8 == 0) gap_launch<bf16_t, 8>(m, HW, C, x, y, s); else gap_launch<bf16_t, 1>(m, HW, C, x, y, s); }
    else { if (C % 4 == 0) gap_launch<float, 4>(m, HW, C, x, y, s); else gap_launch<float, 1>(m, HW, C, x, y, s); }
    return hipGetLastError();
}

hipError_t launch_gap_bwd(int dtype, int32_t m, int32_t HW, int32_t C, const void* dy, void* dx, int accumulate,
                          const void* mask, const float* mscale, hipStream_t s) {
    LPM_DISPATCH(dtype, launch_last(gap_bwd_kernel<T>, dim3(nblk((int64_t)m * HW * C, 256)), dim3(256), 0, s, m, HW,
                                           C, (const T*)dy, (T*)dx, accumulate, (const T*)mask, mscale));
    return hipGetLastError();
}

// --------------------------------------------------------------------------------------------------
// Global average pooling and the fully connected layer that alone reads it, the head of a residual network: one kernel forward and one for the
// data gradient, where each had two of a few microseconds and next to no work on the chain that every micro-batch waits for (ResNet-18/CIFAR at 32 samples
// a micro-batch, in a trace of the step: forward 4.3 + 6.2 us -> 5.1, data gradient 4.8 + 3.5 -> 3.9; per step 2634 -> 2584, float 2373 -> 2334, width 48 with 100 classes 2143 ->
// 2123, volumetric 1598 -> 1588, 16 images forward 133.4 -> 130.2).  What bounds them is the launch and two round trips to memory.

// A block takes a sample: its threads hold V channels of every RL-th position, then eight lanes share NB outputs of the layer at a time (whose
// loads are under way together).  A float lane keeps 2 V sums of an output, each of every 16 V-th channel, and folds them: one sum over all the
// lane's channels was 1.5 to 1.75 times as far from 64 bits as the kernels of the pooling and the layer (512 channels at 16 positions 1.67e-7, 1.10e-7).
constexpr int HEAD_C = 2048;
template <typename T, int V, int NB>
__global__ void __launch_bounds__(256) head_fwd_kernel(int HW, int C, int cl_log, int N, const T* __restrict__ x, T* __restrict__ y,
                                                       const T* __restrict__ w, const float* __restrict__ bias, T* __restrict__ z) {
    __shared__ __attribute__((aligned(16))) float red[256 * V];
    __shared__ __attribute__((aligned(16))) float pooled[HEAD_C];
    const int CL = 1 << cl_log, RL = 256 >> cl_log, cx = threadIdx.x & (CL - 1), ty = threadIdx.x >> cl_log;
    const T* xs = x + (int64_t)blockIdx.x * HW * C;
    for (int cb = 0; cb < C; cb += CL * V) {
        const int c0 = cb + cx * V;
        float sum[V];
#pragma unroll
        for (int k = 0; k < V; ++k) sum[k] = 0.f;
        if (c0 < C) {
            for (int r = ty; r < HW; r += 4 * RL) {
                float v[4][V];
#pragma unroll
                for (int u = 0; u < 4; ++u) EpiVec<T, V>::get(xs, (int64_t)min(r + u * RL, HW - 1) * C + c0, v[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (r + u * RL < HW) {
#pragma unroll
                        for (int k = 0; k < V; ++k) sum[k] += v[u][k];
                    }
            }
        }
#pragma unroll
        for (int k = 0; k < V; ++k) red[(ty * CL + cx) * V + k] = sum[k];
        __syncthreads();
        for (int c = threadIdx.x; c < CL * V && cb + c < C; c += 256) {
            float acc = 0.f;
            for (int r = 0; r < RL; ++r) acc += red[r * CL * V + c];
            const T one = to_store<T>(acc / (float)HW);
            y[(int64_t)blockIdx.x * C + cb + c] = one;
            pooled[cb + c] = ld(&one, 0);
        }
        __syncthreads();
    }
    const int j = threadIdx.x & 7;
    for (int n = threadIdx.x >> 3; n < N; n += 32 * NB) {
        constexpr int U = sizeof(T) == 4 ? 2 : 1, S = sizeof(T) == 4 ? U * V : 1;
        float s[NB][S];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int i = 0; i < S; ++i) s[b][i] = 0.f;
        auto step = [&](int c, int u) __attribute__((always_inline)) {
            float v[NB][V];
#pragma unroll
            for (int b = 0; b < NB; ++b) EpiVec<T, V>::get(w, (int64_t)min(n + 32 * b, N - 1) * C + c, v[b]);
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int k = 0; k < V; ++k) {
                    float& a = s[b][S == 1 ? 0 : u * V + k];
                    a = fmaf(v[b][k], pooled[c + k], a);
                }
        };
        int c = j * V;
#pragma unroll (NB == 1 ? 8 / U : 2 / U)
        for (; c + (U - 1) * 8 * V < C; c += U * 8 * V) {
#pragma unroll
            for (int u = 0; u < U; ++u) step(c + u * 8 * V, u);
        }
        if (U > 1 && c < C) step(c, 0);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
#pragma unroll
            for (int o = S / 2; o > 0; o >>= 1)
#pragma unroll
                for (int i = 0; i < o; ++i) s[b][i] += s[b][i + o];
            float z1 = s[b][0];
#pragma unroll
            for (int o = 4; o > 0; o >>= 1) z1 += __shfl_xor(z1, o, 64);
            const int nb = n + 32 * b;
            if (j == 0 && nb < N) st(z, (int64_t)blockIdx.x * N + nb, bias ? z1 + bias[nb] : z1);
        }
    }
}

// A block takes 16 channel chunks of a sample; 16 groups of threads share the outputs of the layer, then the positions.  Their sums are added up
// once a channel: every thread for itself, eight of them on a bank, cost more than all else (the backward pass of 2048 samples, 2048 channels of one
// position, 10 outputs 239 -> 38 us, in kernels of their own 28; float 132 -> 45 and 34).
template <typename T, int V>
__global__ void __launch_bounds__(256) head_bwd_kernel(int HW, int C, int N, const T* __restrict__ dz, const T* __restrict__ w, T* __restrict__ dp,
                                                       T* __restrict__ dx, int accumulate, const T* __restrict__ mask, const float* __restrict__ mscale) {
    __shared__ __attribute__((aligned(16))) float red[16][16 * V];
    const int cx = threadIdx.x & 15, ty = threadIdx.x >> 4, c0 = (blockIdx.y * 16 + cx) * V, n0 = blockIdx.x;
    const bool ok = c0 < C;
    float g[V];
#pragma unroll
    for (int k = 0; k < V; ++k) g[k] = 0.f;
    if (ok) {
#pragma unroll 4
        for (int n = ty; n < N; n += 16) {
            const float d = ld(dz, (int64_t)n0 * N + n);
            float v[V];
            EpiVec<T, V>::get(w, (int64_t)n * C + c0, v);
#pragma unroll
            for (int k = 0; k < V; ++k) g[k] = fmaf(d, v[k], g[k]);
        }
    }
#pragma unroll
    for (int k = 0; k < V; ++k) red[ty][cx * V + k] = g[k];
    __syncthreads();
    if (threadIdx.x < 16 * V) {             // (a thread a channel, neighbours on neighbouring banks)
        // (float's in 64 bits: the layer's own kernel adds fewer terms one after the other, and these were 1.23 to 1.29 times as far from the exact sum)
        typename std::conditional<sizeof(T) == 4, double, float>::type sum = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) sum += red[r][threadIdx.x];
        const T one = to_store<T>((float)sum);
        red[0][threadIdx.x] = ld(&one, 0);
    }
    __syncthreads();
    if (!ok) return;
    float ms[V];
#pragma unroll
    for (int k = 0; k < V; ++k) {
        g[k] = red[0][cx * V + k];
        ms[k] = mscale ? mscale[c0 + k] : 1.f;
    }
    if (!ty) EpiVec<T, V>::put(dp, (int64_t)n0 * C + c0, g);
    if (!dx) return;
#pragma unroll
    for (int k = 0; k < V; ++k) g[k] = g[k] / (float)HW;
    for (int r = ty; r < HW; r += 16) {
        const int64_t at = ((int64_t)n0 * HW + r) * C + c0;
        float v[V], t[V];
#pragma unroll
        for (int k = 0; k < V; ++k) v[k] = g[k];
        if (accumulate) {
            EpiVec<T, V>::get(dx, at, t);
#pragma unroll
            for (int k = 0; k < V; ++k) v[k] += t[k];
        }
        if (mask) {
            EpiVec<T, V>::get(mask, at, t);
#pragma unroll
            for (int k = 0; k < V; ++k) v[k] = t[k] > 0.f ? v[k] : 0.f;
        }
#pragma unroll
        for (int k = 0; k < V; ++k) v[k] *= ms[k];
        EpiVec<T, V>::put(dx, at, v);
    }
}

// Channels in whole 16-byte chunks.  A sample of up to 64 KB and 128 outputs: one block walks either in a few round trips to memory.
// Each block reads all of the layer's weights that it needs, the contraction reads them once a tile: with many samples or large weights one kernel takes
// longer than two.  Kernel times in two / in one, us, over 1 to 128 outputs and 1 to 49 positions.  Forward, over 32 outputs, the worst: 512 channels x 512
// samples bf16 9.3 / 7.0, x 1024 14.9 / 15.3, x 2048 20.6 / 27.8; 64 channels x 2048 bf16 1.15 of the time, float .80, x 4096 1.16; 768 channels x 256
// (in a graph) bf16 9.0 / 8.7, float 14.4 / 9.4; 1024 channels x 128 bf16 9.0 / 8.2, float 13 / 11, x 256
// float 15.2 / 18.8; 2048 channels x 8 bf16 11.1 / 15.0, float 12.3 / 15.2.  (768 to 1024 channels of a few samples take up to 1 us longer back to back in a graph, where
// the gap between two kernels is hidden, and save a launch elsewhere.)  Up to 32 outputs, 64 channels, bf16 x 1024 6.7 / 4.4, x 2048 6.5 / 6.7,
// x 4096 8.2 / 11.2 (float .71 of the time); 128 channels x 2048 .73 of the time, x 4096 1.08; 512 .86 and .97.  Data gradient, which reads a sixteenth of a row of weights
// at a time and is soon bound by its stores: 16 positions and more .17 to .80 of the time at every size; one position, 128 outputs, 2^18 values bf16 .86 to .92,
// float .85 to .99, 2^19 1.28 and 1.54.
bool head_ok(int dtype, int32_t m, int32_t HW, int32_t C, int32_t N, bool fwd) {
    if (C % (dtype == LPM_BF16 ? 8 : 4) != 0 || C > HEAD_C || N > 128 || (int64_t)HW * C * (dtype == LPM_BF16 ? 2 : 4) > 65536) return false;
    const bool few = (int64_t)m * C <= (1 << 18);
    if (!fwd) return few || (HW >= 16 && m < (1 << 23));      // (a block of 256 threads a sample, and a launch holds fewer than 2^32 threads)
    const bool f32 = dtype == LPM_F32;
    return N <= 32 ? m <= (f32 ? 4096 : 1024 + 8 * C) : few && m <= (f32 ? 2048 : 1024) && (C <= 768 || (C <= 1024 && m <= 192));
}
hipError_t launch_head_fwd(int dtype, int32_t m, int32_t HW, int32_t C, int32_t N, const void* x, void* y, const void* w, const float* bias, void* z, hipStream_t s) {
    const int V = dtype == LPM_BF16 ? 8 : 4;
    int cl = 0;
    while (cl < 8 && (V << cl) < C) ++cl;
    auto go = [&](auto kernel, auto t) {
        typedef decltype(t) T;
        launch_last(kernel, dim3(m), dim3(256), 0, s, HW, C, cl, N, (const T*)x, (T*)y, (const T*)w, bias, (T*)z);
    };
    if (dtype == LPM_BF16) N > 32 ? go(head_fwd_kernel<bf16_t, 8, 4>, bf16_t{}) : go(head_fwd_kernel<bf16_t, 8, 1>, bf16_t{});
    else N > 32 ? go(head_fwd_kernel<float, 4, 4>, 0.f) : go(head_fwd_kernel<float, 4, 1>, 0.f);
    return hipGetLastError();
}
hipError_t launch_head_bwd(int dtype, int32_t m, int32_t HW, int32_t C, int32_t N, const void* dz, const void* w, void* dp, void* dx, int accumulate,
                           const void* mask, const float* mscale, hipStream_t s) {
    // (samples on the grid's first extent, which has room for them: one launch, so that a stop event stands behind all of them)
    const dim3 grid((unsigned)m, (unsigned)((C / (dtype == LPM_BF16 ? 8 : 4) + 15) / 16));
    if (dtype == LPM_BF16) launch_last(head_bwd_kernel<bf16_t, 8>, grid, dim3(256), 0, s, HW, C, N, (const bf16_t*)dz, (const bf16_t*)w, (bf16_t*)dp, (bf16_t*)dx, accumulate,
                                       (const bf16_t*)mask, mscale);
    else launch_last(head_bwd_kernel<float, 4>, grid, dim3(256), 0, s, HW, C, N, (const float*)dz, (const float*)w, (float*)dp, (float*)dx, accumulate,
                     (const float*)mask, mscale);
    return hipGetLastError();
}

// --------------------------------------------------------------------------------------------------
// softmax cross-entropy (eq. 3 with the cross-entropy loss), one wavefront per row, one block in all:
//   dlogits = (softmax(z) - onehot(label)) * loss_scale
//   *loss_accum += loss_scale * sum_rows ( log sum exp(z - max) - (z[label] - max) )   (rows added in order)
__device__ inline float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ inline float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// One block of 16 wavefronts, a wavefront per row at a time; a row of up to 64 * KEEP classes is read once and kept in
// registers, labels and the loss so far are requested with the first row (the kernel closes every forward chain, so its
// latency counts: every dependent pass over global memory is a microsecond).  The loss is summed in row order by one thread.
template <typename T, int KEEP>
__global__ void __launch_bounds__(1024) softmax_ce_kernel(int m, int C, const T* __restrict__ z,
                                                          const int32_t* __restrict__ labels, float loss_scale,
                                                          T* __restrict__ dz, float* __restrict__ loss_accum) {
    __shared__ float rowloss[256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float before = threadIdx.x == 0 ? *loss_accum : 0.f;
    float total = 0.f;
    for (int base = 0; base < m; base += 256) {
        const int nrow = min(256, m - base);
        for (int r = wave; r < nrow; r += 16) {
            const T* zr = z + (int64_t)(base + r) * C;
            T* dr = dz + (int64_t)(base + r) * C;
            // a label outside [0, C) selects no class: no one-hot term, and the row's loss becomes NaN so the host sees it
            const int lab = labels[base + r];
            const bool lab_ok = (unsigned)lab < (unsigned)C;
            float v[KEEP > 0 ? KEEP : 1];
            float mx = -INFINITY, zl = 0.f;
            if (KEEP > 0) {
#pragma unroll
                for (int k = 0; k < KEEP; ++k) {
                    const int c = lane + 64 * k;
                    v[k] = c < C ? ld(zr, c) : -INFINITY;
                }
#pragma unroll
                for (int k = 0; k < KEEP; ++k) {
                    mx = fmaxf(mx, v[k]);
                    if (lane + 64 * k == lab) zl = v[k];
                }
            } else {
                for (int c = lane; c < C; c += 64) {
                    const float x = ld(zr, c);
                    mx = fmaxf(mx, x);
                    if (c == lab) zl = x;
                }
            }
            mx = wave_max(mx);
            float se = 0.f;
            if (KEEP > 0) {
#pragma unroll
                for (int k = 0; k < KEEP; ++k) { v[k] = expf(v[k] - mx); se += v[k]; }      // exp(-inf) = 0 past the end
            } else {
                for (int c = lane; c < C; c += 64) se += expf(ld(zr, c) - mx);
            }
            se = wave_sum(se);
            zl = __shfl(zl, lab & 63, 64);           // (the lane that met the label)
            const float inv = 1.f / se;
            if (KEEP > 0) {
#pragma unroll
                for (int k = 0; k < KEEP; ++k) {
                    const int c = lane + 64 * k;
                    if (c < C) st(dr, c, (v[k] * inv - (c == lab ? 1.f : 0.f)) * loss_scale);
                }
            } else {
                for (int c = lane; c < C; c += 64) {
                    const float p = expf(ld(zr, c) - mx) * inv;
                    st(dr, c, (p - (c == lab ? 1.f : 0.f)) * loss_scale);
                }
            }
            if (lane == 0) rowloss[r] = lab_ok ? logf(se) - (zl - mx) : __builtin_nanf("");
        }
        __syncthreads();
        if (threadIdx.x == 0)
            for (int r = 0; r < nrow; ++r) total += rowloss[r];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss_accum = before + loss_scale * total;
}

hipError_t launch_softmax_ce(int dtype, int32_t m, int32_t C, const void* logits, const int32_t* labels, float loss_scale,
                             void* dlogits, float* loss_accum, hipStream_t s) {
    if (C <= 64) LPM_DISPATCH(dtype, launch_last(softmax_ce_kernel<T, 1>, dim3(1), dim3(1024), 0, s, m, C, (const T*)logits, labels, loss_scale, (T*)dlogits, loss_accum));
    else if (C <= 1024) LPM_DISPATCH(dtype, launch_last(softmax_ce_kernel<T, 16>, dim3(1), dim3(1024), 0, s, m, C, (const T*)logits, labels, loss_scale, (T*)dlogits, loss_accum));
    else LPM_DISPATCH(dtype, launch_last(softmax_ce_kernel<T, 0>, dim3(1), dim3(1024), 0, s, m, C, (const T*)logits, labels, loss_scale, (T*)dlogits, loss_accum));
    return hipGetLastError();
}

// --------------------------------------------------------------------------------------------------
// update, eq. 6 with momentum: v = mu*v + g; p = p - lr*v; bf16 copy; optional g = 0.  Pure streaming: one
// float4 per thread, consecutive threads on consecutive addresses, non-temporal accesses (measured at 103 M
// parameters: 5.9 TB/s against 4.3 TB/s for a grid-stride loop over 4096 blocks).
// (p_in and p_out may be the same buffer: every element is read and written by one thread)
struct SgdRule {
    static constexpr int NM = 1;
    float lr, mu;
    __device__ __forceinline__ void step(float g, float* m, float& p) const {
        m[0] = fmaf(mu, m[0], g);
        p = fmaf(-lr, m[0], p);
    }
};

// Adam update (Kingma & Ba), the alternative to eq. 6 that the paper's problem statement names: the same streaming
// shape with two moment buffers.  inv_c1 = 1 / (1 - beta1^t), inv_c2 = 1 / (1 - beta2^t).
struct AdamRule {
    static constexpr int NM = 2;
    float lr, beta1, beta2, eps, inv_c1, inv_c2;
    __device__ __forceinline__ void step(float g, float* m, float& p) const {
        m[0] = beta1 * m[0] + (1.f - beta1) * g;
        m[1] = beta2 * m[1] + (1.f - beta2) * g * g;
        p -= lr * (m[0] * inv_c1) / (sqrtf(m[1] * inv_c2) + eps);
    }
};

constexpr int UPD_T = 256, UPD_CO = 64;      // threads; output channels of a tile (512 or 1024 threads, 32 channels: the same within 1 %)
struct UpdateArgs {
    UpdateSeg d[LPM_UPDATE_BATCH];
    int first[LPM_UPDATE_BATCH + 1];         // first block of every segment
    int count;
    const float4* p_in;
    float4 *p, *g, *m[2];
    uint16_t* lowp;
    int zero_g;
};

// V float4s per thread: all their loads are issued before the first is used
template <typename R, int V>
__device__ __forceinline__ void update_elements(const UpdateArgs& a, const R& r, const size_t (&at)[V], const bool (&ok)[V], float4 (&pp)[V]) {
    float4 gg[V], mm[R::NM][V];
#pragma unroll
    for (int k = 0; k < V; ++k) {
        if (!ok[k]) continue;
        gg[k] = ld_stream(&a.g[at[k]]);
        pp[k] = ld_stream(&a.p_in[at[k]]);
#pragma unroll
        for (int n = 0; n < R::NM; ++n) mm[n][k] = ld_stream(&a.m[n][at[k]]);
    }
#pragma unroll
    for (int k = 0; k < V; ++k) {
        if (!ok[k]) continue;
        const float gv[4] = {gg[k].x, gg[k].y, gg[k].z, gg[k].w};
        float pv[4] = {pp[k].x, pp[k].y, pp[k].z, pp[k].w}, mv[4][R::NM];
#pragma unroll
        for (int n = 0; n < R::NM; ++n) { mv[0][n] = mm[n][k].x; mv[1][n] = mm[n][k].y; mv[2][n] = mm[n][k].z; mv[3][n] = mm[n][k].w; }
#pragma unroll
        for (int e = 0; e < 4; ++e) r.step(gv[e], mv[e], pv[e]);
#pragma unroll
        for (int n = 0; n < R::NM; ++n) st_stream(&a.m[n][at[k]], make_float4(mv[0][n], mv[1][n], mv[2][n], mv[3][n]));
        pp[k] = make_float4(pv[0], pv[1], pv[2], pv[3]);
        st_stream(&a.p[at[k]], pp[k]);
        if (a.lowp) st_stream((uint2*)a.lowp + at[k], make_uint2(pack_bf16x2(pv[0], pv[1]), pack_bf16x2(pv[2], pv[3])));
        if (a.zero_g) st_stream(&a.g[at[k]], make_float4(0.f, 0.f, 0.f, 0.f));
    }
}

// Every segment of a stage's parameters in one launch.  A segment with a [Cin][Kh][Kw][Cout] copy goes by tiles of 64 (co) x 64 (ci)
// of one filter tap, whose new values also leave through LDS for that copy.  Bound by memory: 30 bytes a parameter for Adam with the copy,
// 22 for SGD.  As a kernel of its own the transposition waited for the update and read the new weights again: Adam over 3.5 M parameters
// 18.6 + 11.4 us, now 25.8; SGD over 7 M 25.8 + 20.2, now 30.9.
template <typename R>
__global__ void __launch_bounds__(UPD_T) update_kernel(UpdateArgs a, R r) {
    __shared__ float tile[UPD_CO][65];
    int k = 0;
    while (k + 1 < a.count && (int)blockIdx.x >= a.first[k + 1]) ++k;
    const UpdateSeg& d = a.d[k];
    int t = (int)blockIdx.x - a.first[k];
    if (!d.wt) {
        const size_t i = (size_t)t * UPD_T + threadIdx.x;
        const size_t at[1] = {d.off / 4 + i};
        const bool ok[1] = {i < d.n / 4};
        float4 pp[1];
        update_elements<R, 1>(a, r, at, ok, pp);
        return;
    }
    const int cit = (d.Cin + 63) / 64, cot = (d.Cout + UPD_CO - 1) / UPD_CO;
    const int ci0 = (t % cit) * 64; t /= cit;
    const int co0 = (t % cot) * UPD_CO;
    const int kk = t / cot;
    constexpr int V = UPD_CO * 16 / UPD_T, RS = UPD_T / 16, OL = UPD_CO / 4, OS = UPD_T / OL;
    const int lx = threadIdx.x & 15, ly = threadIdx.x >> 4;
    size_t at[V];
    bool ok[V];
    float4 pp[V];
#pragma unroll
    for (int q = 0; q < V; ++q) {
        const int co = co0 + ly + q * RS, ci = ci0 + lx * 4;
        ok[q] = co < d.Cout && ci < d.Cin;
        at[q] = (d.off + ((size_t)co * d.KK + kk) * d.Cin + ci) / 4;
    }
    update_elements<R, V>(a, r, at, ok, pp);
#pragma unroll
    for (int q = 0; q < V; ++q) {
        if (!ok[q]) continue;
        const float sc = d.scale ? d.scale[co0 + ly + q * RS] : 1.f;
        float* row = &tile[ly + q * RS][lx * 4];
        row[0] = pp[q].x * sc; row[1] = pp[q].y * sc; row[2] = pp[q].z * sc; row[3] = pp[q].w * sc;
    }
    __syncthreads();
    const int o = (threadIdx.x % OL) * 4, iy = threadIdx.x / OL;
#pragma unroll
    for (int q = 0; q < 64 / OS; ++q) {
        const int i = iy + q * OS, ci = ci0 + i, co = co0 + o;
        if (ci >= d.Cin || co >= d.Cout) continue;
        *(uint2*)(d.wt + ((size_t)ci * d.KK + kk) * d.Cout + co) =
            make_uint2(pack_bf16x2(tile[o][i], tile[o + 1][i]), pack_bf16x2(tile[o + 2][i], tile[o + 3][i]));
    }
}

template <typename R>
static hipError_t launch_update(const UpdateSeg* d, int count, UpdateArgs a, const R& r, hipStream_t s) {
    for (int done = 0; done < count;) {
        int64_t tot = 0;
        int k = 0;
        for (; k < LPM_UPDATE_BATCH && done + k < count; ++k) {
            const UpdateSeg& u = d[done + k];
            if (u.off % 4 || u.n % 4 || (u.wt && (u.Cin % 4 || u.Cout % 4))) return hipErrorInvalidValue;
            const int64_t blocks = u.wt ? (int64_t)((u.Cin + 63) / 64) * ((u.Cout + UPD_CO - 1) / UPD_CO) * u.KK : (int64_t)((u.n / 4 + UPD_T - 1) / UPD_T);
            if (tot + blocks > INT32_MAX) break;
            a.d[k] = u;
            a.first[k] = (int)tot;
            tot += blocks;
        }
        if (k == 0) return hipErrorInvalidValue;
        a.first[k] = (int)tot;
        a.count = k;
        done += k;
        if (tot == 0) continue;
        hipLaunchKernelGGL(update_kernel<R>, dim3((unsigned)tot), dim3(UPD_T), 0, s, a, r);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_sgd(const UpdateSeg* d, int count, const float* p_in, float* p, uint16_t* lowp, float* g, float* v, float lr, float mu,
                      int zero_g, hipStream_t s) {
    UpdateArgs a{};
    a.p_in = (const float4*)p_in; a.p = (float4*)p; a.g = (float4*)g; a.m[0] = (float4*)v; a.lowp = lowp; a.zero_g = zero_g;
    return launch_update(d, count, a, SgdRule{lr, mu}, s);
}

hipError_t launch_adam(const UpdateSeg* d, int count, float* p, uint16_t* lowp, float* g, float* m1, float* m2, float lr, float beta1,
                       float beta2, float eps, float inv_c1, float inv_c2, int zero_g, hipStream_t s) {
    UpdateArgs a{};
    a.p_in = (const float4*)p; a.p = (float4*)p; a.g = (float4*)g; a.m[0] = (float4*)m1; a.m[1] = (float4*)m2; a.lowp = lowp; a.zero_g = zero_g;
    return launch_update(d, count, a, AdamRule{lr, beta1, beta2, eps, inv_c1, inv_c2}, s);
}

__global__ void __launch_bounds__(256) f32_to_bf16_kernel(const float4* __restrict__ src, uint2* __restrict__ dst, size_t n4) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n4) return;
    const float4 a = ld_stream(&src[i]);
    st_stream(&dst[i], make_uint2(pack_bf16x2(a.x, a.y), pack_bf16x2(a.z, a.w)));
}

hipError_t launch_f32_to_bf16(const float* src, uint16_t* dst, size_t n, hipStream_t s) {
    const size_t n4 = n / 4;
    if (n4 == 0) return hipSuccess;
    hipLaunchKernelGGL(f32_to_bf16_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, (const float4*)src, (uint2*)dst, n4);
    return hipGetLastError();
}

// dst[ci][k][co] = bf16(src[co][k][ci] * scale[co])   (k = kh*Kw+kw; scale may be NULL), for up to LPM_TRANSPOSE_BATCH weight
// tensors in one launch.
// A block moves a 32 (co) x 32 (ci) tile of one filter tap through LDS: reads run along ci, writes along co.
struct TransposeBatchArgs {
    TransposeDesc d[LPM_TRANSPOSE_BATCH];
    int first[LPM_TRANSPOSE_BATCH + 1];      // first block of every tensor
    int count;
};

__global__ void __launch_bounds__(256) weight_transpose_batch(TransposeBatchArgs a) {
    __shared__ float tile[32][33];
    int k = 0;
    while (k + 1 < a.count && (int)blockIdx.x >= a.first[k + 1]) ++k;
    const TransposeDesc& d = a.d[k];
    int t = (int)blockIdx.x - a.first[k];
    const int cit = (d.Cin + 31) / 32, cot = (d.Cout + 31) / 32;
    const int ci0 = (t % cit) * 32; t /= cit;
    const int co0 = (t % cot) * 32;
    const int kk = t / cot;
    const int lx = threadIdx.x & 31, ly = threadIdx.x >> 5;      // 32 x 8
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int co = co0 + ly + r * 8, ci = ci0 + lx;
        tile[ly + r * 8][lx] = (co < d.Cout && ci < d.Cin) ? d.src[((size_t)co * d.KK + kk) * d.Cin + ci] * (d.scale ? d.scale[co] : 1.f) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int ci = ci0 + ly + r * 8, co = co0 + lx;
        if (ci < d.Cin && co < d.Cout) d.dst[((size_t)ci * d.KK + kk) * d.Cout + co] = f2bf(tile[lx][ly + r * 8]);
    }
}

hipError_t launch_weight_transpose_batch(const TransposeDesc* d, int count, hipStream_t s) {
    for (int done = 0; done < count;) {
        TransposeBatchArgs a{};
        int tot = 0, k = 0;
        for (; k < LPM_TRANSPOSE_BATCH && done + k < count; ++k) {
            a.d[k] = d[done + k];
            a.first[k] = tot;
            tot += ((a.d[k].Cin + 31) / 32) * ((a.d[k].Cout + 31) / 32) * a.d[k].KK;
        }
        a.first[k] = tot;
        a.count = k;
        done += k;
        if (tot == 0) continue;
        hipLaunchKernelGGL(weight_transpose_batch, dim3((unsigned)tot), dim3(256), 0, s, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

__global__ void __launch_bounds__(256) fill_kernel(float* p, size_t n, float v) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = v;
}

hipError_t launch_fill_f32(float* p, size_t n, float v, hipStream_t s) {
    if (n == 0) return hipSuccess;
    unsigned blocks = (unsigned)((n + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_kernel, dim3(blocks), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

// One wavefront that does nothing for `ticks` periods of the constant 100 MHz device clock (it leaves the loop as soon
// as the clock has advanced that far): the probe kernel of streams_share_queue.
__global__ void spin_kernel(long long ticks) {
    const long long t0 = wall_clock64();
    while (wall_clock64() - t0 < ticks) __builtin_amdgcn_s_sleep(16);
}

hipError_t launch_spin(long long ticks, hipStream_t s) {
    hipLaunchKernelGGL(spin_kernel, dim3(1), dim3(64), 0, s, ticks);
    return hipGetLastError();
}

}  // namespace lpm
