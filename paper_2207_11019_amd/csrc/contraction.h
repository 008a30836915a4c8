// What the contraction kernels share: their arguments and the epilogue that a wavefront runs on its piece of the output.
#pragma once
#include "lpm_internal.h"
#include "elem.h"

namespace lpm {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr unsigned OOB = 0xffffffffu;

enum { MODE_FWD = 0, MODE_DGRAD = 1 /* stride 1 */, MODE_DGRAD_S = 2 /* stride 2..4, by residue class */, MODE_UNPOOL = 3 /* stride 1, routed through a max-pooling */,
       MODE_FWD_POOL = 4 /* forward, the rows by pooling window */ };

constexpr int MAX_TAB = 128;              // taps a layer without whole K tiles per tap may have
constexpr int MAX_KSCALE = 2048;          // channels of a float layer whose data gradient applies its scale (LDS)

struct IgemmArgs {
    const void* A;
    const void* B;
    void* C;                // output [M][N]
    float* part;            // split K: fp32 partial tiles
    unsigned* count;        // split K: blocks that have stored theirs, per output tile
    const float* scale;
    const float* bias;
    const float* kscale;    // float data gradient: per-channel factor of the gathered tensor (the reduction index), or NULL
    const void* add;        // added to the result (data gradient: what the output, or another tensor, holds)
    const void* mask;       // data gradient: zero the result where this tensor (the producer's output) is <= 0
    const float* mscale;    // data gradient: then multiply by the producer's per-channel scale
    void* C2;               // data gradient: the masked, not yet scaled result also goes here (the producer's shortcut), or NULL
    const float* c2scale;   // ... times this per-channel factor (NULL: 1)
    int acc2;               // ... added to what C2 holds
    int relu;
    int M, N;
    int Hi, Wi, Di, Ci;     // extent of the gathered tensor
    int Hr, Wr, Dr;         // extent of the row space
    int Kh, Kw, Kd, stride, pad, pad_d;
    FastDiv dWr, dHr, dDr, dCc;       // row decoding; chunks per tap
    FastDiv dNt, dKt, dKhw, dKw;      // tiles along N, K tiles per tap (whole ones), taps per filter slice and per filter row
    unsigned a_bytes, b_bytes, b_pitch;
    int kt_total, kt_per_split, splits;
    int free_taps;          // no tap can leave the image: no mask bits needed
    // strided data gradient: first row tile of residue class c = (pd * s + ph) * s + pw, images, the stride, and the two extents that a class
    // can have along an axis: whole strides, and one more
    int cls_tile0[17], images;
    FastDiv dS, dWc[2], dHc[2], dDc[2];
    const uint16_t* pool_x; // stride-1 data gradient routed through a 2x2 max-pooling (see UnpoolDesc): its input [m][2*Hr][2*Wr][N]
    uint16_t* pool_dst;
    int pool_acc, pool_mask;
    uint16_t* fwd_pool;     // forward: also store the 2x2 max-pooling of C, [m][Hr/2][Wr/2][N] (bf16, Wr = 2, 4, 8, 16 or 32; MODE_FWD_POOL: any)
};

// ---- eight consecutive channels of a row -----------------------------------------------------------
template <typename E> struct Raw8;
template <> struct Raw8<bf16_t> { uint4 v; };
template <> struct Raw8<float> { float4 lo, hi; };
__device__ __forceinline__ Raw8<bf16_t> ld_raw8(const bf16_t* p) { return {*reinterpret_cast<const uint4*>(p)}; }
__device__ __forceinline__ Raw8<float> ld_raw8(const float* p) {
    return {*reinterpret_cast<const float4*>(p), *reinterpret_cast<const float4*>(p + 4)};
}
__device__ __forceinline__ void un8(const Raw8<bf16_t>& r, float (&f)[8]) {
    const uint32_t w[4] = {r.v.x, r.v.y, r.v.z, r.v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) { f[2 * k] = bf2f((uint16_t)(w[k] & 0xffffu)); f[2 * k + 1] = bf2f((uint16_t)(w[k] >> 16)); }
}
__device__ __forceinline__ void un8(const Raw8<float>& r, float (&f)[8]) {
    f[0] = r.lo.x; f[1] = r.lo.y; f[2] = r.lo.z; f[3] = r.lo.w; f[4] = r.hi.x; f[5] = r.hi.y; f[6] = r.hi.z; f[7] = r.hi.w;
}
__device__ __forceinline__ void st8(bf16_t* p, const float (&f)[8]) {
    *reinterpret_cast<uint4*>(p) = make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
}
__device__ __forceinline__ void st8(float* p, const float (&f)[8]) {
    *reinterpret_cast<float4*>(p) = make_float4(f[0], f[1], f[2], f[3]);
    *reinterpret_cast<float4*>(p + 4) = make_float4(f[4], f[5], f[6], f[7]);
}

// Strided data gradient: pixel index (in the full tensor) of row `row` of the residue class (pd, ph, pw).
__device__ __forceinline__ int class_pixel(const IgemmArgs& p, int row, int Hc, int Wc, int ph, int pw, int Dc, int pd) {
    const int t = div_by(row, p.dWc[Wc - div_by(p.Wr, p.dS)]), wq = row - t * Wc;
    int n = div_by(t, p.dHc[Hc - div_by(p.Hr, p.dS)]), img = n;
    const int hq = t - n * Hc;
    if (p.Dr > 1) { const int ns = div_by(n, p.dDc[Dc - div_by(p.Dr, p.dS)]), dq = n - ns * Dc; n = ns; img = n * p.Dr + dq * p.stride + pd; }
    return (img * p.Hr + hq * p.stride + ph) * p.Wr + wq * p.stride + pw;
}

// MODE_FWD_POOL: row 4w + 2y + x is position (y, x) of pooling window w (dWr, dHr: of the pooled image).
struct WinPixel { int n, h, w; };
__device__ __forceinline__ WinPixel win_pixel(const IgemmArgs& p, int row) {
    const int q = row >> 2, t = div_by(q, p.dWr), n = div_by(t, p.dHr);
    return {n, 2 * (t - n * (p.Hr >> 1)) + ((row >> 1) & 1), 2 * (q - t * (p.Wr >> 1)) + (row & 1)};
}
__device__ __forceinline__ int win_row(const IgemmArgs& p, int row) {
    const WinPixel x = win_pixel(p, row);
    return (x.n * p.Hr + x.h) * p.Wr + x.w;
}

// A wavefront's part of the output, MI pieces of 32 rows x 32*NIW channels, held in its private LDS area (rows of 32*NIW + 4
// floats).  A lane takes 8 channels of a row at a time, so every tensor access is 16 (float: 32) bytes.  load() requests the
// operands of all the lane's chunks; the kernels call it before their main loop where the registers allow, so that a
// launch of a few K tiles does not end with a memory latency of its own.
template <typename E, int MI, int NIW, int MODE>
struct Epilogue {
    static constexpr bool WIN = MODE == MODE_FWD_POOL, FWD = MODE == MODE_FWD || WIN;      // (forward: scale, bias, add, relu; data gradient: add, mask, C2, mscale)
    static constexpr int PITCH = NIW * 32 + 4, PIECE = 32 * PITCH, CPR = NIW * 4, RPP = 64 / CPR, NP = 32 / RPP, R = MI * NP;
    Raw8<E> ra[R], rm[FWD ? 1 : R], r2[FWD ? 1 : R];
    float f0[8], f1[8];                       // forward: scale, bias; data gradient: mscale, c2scale
    int o[R];                                 // element offset of the chunk, -1: none

    // row0: the part's first row, in the residue class (pd, ph, pw) of extent (Dc, Hc, Wc) for a strided data gradient
    __device__ __forceinline__ void load(const IgemmArgs& p, int row0, int col0, int rows, int lane, int Hc, int Wc, int ph, int pw, int Dc, int pd) {
        if ((p.N & 7) || MODE == MODE_UNPOOL) return;
        const int col = col0 + (lane % CPR) * 8;
        const bool cok = col < p.N;
        auto vec = [&](const float* q, float (&d)[8], float fill) __attribute__((always_inline)) {
            if (q && cok) un8(ld_raw8(q + col), d);
            else {
#pragma unroll
                for (int k = 0; k < 8; ++k) d[k] = fill;
            }
        };
        vec(FWD ? p.scale : p.mscale, f0, 1.f);
        vec(FWD ? p.bias : p.c2scale, f1, FWD ? 0.f : 1.f);
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int row = row0 + q * RPP + lane / CPR;
            const bool live = row < rows && cok;
            const int prow = MODE == MODE_DGRAD_S && live ? class_pixel(p, row, Hc, Wc, ph, pw, Dc, pd) : WIN ? win_row(p, row) : row;
            o[q] = live ? prow * p.N + col : -1;
        }
        if (p.add) {
#pragma unroll
            for (int q = 0; q < R; ++q) ra[q] = ld_raw8((const E*)p.add + max(o[q], 0));
        }
        if (!FWD && p.mask) {
#pragma unroll
            for (int q = 0; q < R; ++q) rm[q] = ld_raw8((const E*)p.mask + max(o[q], 0));
        }
        if (!FWD && p.C2 && p.acc2) {
#pragma unroll
            for (int q = 0; q < R; ++q) r2[q] = ld_raw8((const E*)p.C2 + max(o[q], 0));
        }
    }

    __device__ __forceinline__ void store(const IgemmArgs& p, float* area, int row0, int col0, int rows, int lane, int Hc, int Wc, int ph, int pw, int Dc, int pd) {
        const int ch = (lane % CPR) * 8, col = col0 + ch;
        const E* add = (const E*)p.add;
        const E* msk = (const E*)p.mask;
        E* out = (E*)p.C;
        E* out2 = (E*)p.C2;
        if constexpr (MODE == MODE_UNPOOL) {
            unpool(p, area, row0, col0, rows, lane);
            return;
        }
        if (p.N & 7) {                           // ragged rows: the lanes take consecutive elements
            const int nc = min(p.N - col0, NIW * 32), total = nc > 0 ? min(32 * MI, rows - row0) * nc : 0;
#pragma unroll 1
            for (int i = lane; i < total; i += 64) {
                const int r = i / nc, c = i - r * nc, row = row0 + r, cc = col0 + c;
                const size_t prow = MODE == MODE_DGRAD_S ? (size_t)class_pixel(p, row, Hc, Wc, ph, pw, Dc, pd) : WIN ? (size_t)win_row(p, row) : (size_t)row;
                const size_t e = prow * p.N + cc;
                float v = area[r * PITCH + c];
                if (FWD && p.scale) v *= p.scale[cc];
                if (FWD && p.bias) v += p.bias[cc];
                if (add) v += ld(add, e);
                if (FWD && p.relu) v = fmaxf(v, 0.f);
                if (!FWD && msk && !(ld(msk, e) > 0.f)) v = 0.f;
                if (!FWD && out2) {
                    const float u = p.c2scale ? v * p.c2scale[cc] : v;
                    st(out2, e, p.acc2 ? u + ld(out2, e) : u);
                }
                if (!FWD && p.mscale) v *= p.mscale[cc];
                st(out, e, v);
                if (WIN) area[r * PITCH + c] = sizeof(E) == 2 ? bf2f(f2bf(v)) : v;
            }
            if (WIN) pool_windows(p, area, row0, col0, rows, lane);
            return;
        }
#pragma unroll
        for (int q = 0; q < R; ++q) {
            float* t8 = area + (q * RPP + lane / CPR) * PITCH + ch;
            float v[8], t[8];
            un8(ld_raw8(t8), v);
            if (FWD) {
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = v[k] * f0[k] + f1[k];
            }
            if (add) { un8(ra[q], t);
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] += t[k]; }
            if (FWD && p.relu) {
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = fmaxf(v[k], 0.f); }
            if (!FWD && msk) { un8(rm[FWD ? 0 : q], t);
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = t[k] > 0.f ? v[k] : 0.f; }
            if (!FWD && out2) {
                float u[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) u[k] = v[k] * f1[k];
                if (p.acc2) { un8(r2[FWD ? 0 : q], t);
#pragma unroll
                    for (int k = 0; k < 8; ++k) u[k] += t[k]; }
                if (o[q] >= 0) st8(out2 + o[q], u);
            }
            if (!FWD) {
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] *= f0[k];
            }
            if (o[q] >= 0) st8(out + o[q], v);
            if (FWD && p.fwd_pool) {
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = sizeof(E) == 2 ? bf2f(f2bf(v[k])) : v[k];
                st8(t8, v);
            }
        }
        if (WIN) pool_windows(p, area, row0, col0, rows, lane);
        else if (FWD && p.fwd_pool && p.Wr < 32) pool(p, area, row0, col0, rows, lane);
    }

    // forward, 2x2 max-pooling of the stored values: a piece's 32 rows are whole pairs of image rows, eight windows of rows
    // (r, r+1, r+Wr, r+Wr+1)
    __device__ __forceinline__ void pool(const IgemmArgs& p, float* area, int row0, int col0, int rows, int lane) {
        const int ch = (lane % CPR) * 8, col = col0 + ch, w = lane / CPR;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (w >= 8 || col >= p.N) return;
        const int hw = p.Wr >> 1, py = w / hw, px = w - py * hw, r = 2 * py * p.Wr + 2 * px;
#pragma unroll 1
        for (int mi = 0; mi < MI; ++mi) {
            const int r0 = row0 + mi * 32;
            if (r0 + r >= rows) return;
            const float* t = area + mi * PIECE + ch;
            float a[8], b[8], c[8], d[8];
            un8(ld_raw8(t + r * PITCH), a);
            un8(ld_raw8(t + (r + 1) * PITCH), b);
            un8(ld_raw8(t + (r + p.Wr) * PITCH), c);
            un8(ld_raw8(t + (r + p.Wr + 1) * PITCH), d);
#pragma unroll
            for (int k = 0; k < 8; ++k) a[k] = fmaxf(fmaxf(a[k], b[k]), fmaxf(c[k], d[k]));
            st8((bf16_t*)p.fwd_pool + (size_t)((r0 >> 2) + w) * p.N + col, a);
        }
    }

    // MODE_FWD_POOL, any image width and channel count
    __device__ __forceinline__ void pool_windows(const IgemmArgs& p, const float* area, int row0, int col0, int rows, int lane) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int nc = min(p.N - col0, NIW * 32), nw = min(8 * MI, (rows - row0) >> 2);
#pragma unroll 1
        for (int i = lane; i < nw * nc; i += 64) {
            const int w = i / nc, c = i - w * nc;
            const float* t = area + 4 * w * PITCH + c;
            st((E*)p.fwd_pool, (size_t)((row0 >> 2) + w) * p.N + col0 + c, fmaxf(fmaxf(t[0], t[PITCH]), fmaxf(t[2 * PITCH], t[3 * PITCH])));
        }
    }

    // pool() for images 32 wide: an image row is a piece, its windows reach into the next one (the wavefront's own, or another's
    // that has stored it)
    __device__ __forceinline__ void pool32(const IgemmArgs& p, const float* upper, const float* lower, int row0, int col0, int rows, int lane) {
        const int ch = (lane % CPR) * 8, col = col0 + ch;
        if (row0 >= rows || col >= p.N) return;
#pragma unroll
        for (int w = lane / CPR; w < 16; w += RPP) {
            float a[8], b[8], c[8], d[8];
            un8(ld_raw8(upper + 2 * w * PITCH + ch), a);
            un8(ld_raw8(upper + (2 * w + 1) * PITCH + ch), b);
            un8(ld_raw8(lower + 2 * w * PITCH + ch), c);
            un8(ld_raw8(lower + (2 * w + 1) * PITCH + ch), d);
#pragma unroll
            for (int k = 0; k < 8; ++k) a[k] = fmaxf(fmaxf(a[k], b[k]), fmaxf(c[k], d[k]));
            st8((bf16_t*)p.fwd_pool + (size_t)((row0 >> 2) + w) * p.N + col, a);
        }
    }

    // gradient of a 2x2 max-pooling output: to the first maximum of the window (row-major), through the producer's ReLU
    // and scale where asked; all four window positions are written
    __device__ __forceinline__ void unpool(const IgemmArgs& p, float* area, int row0, int col0, int rows, int lane) {
        const int ch = (lane % CPR) * 8, col = col0 + ch;
        if (col >= p.N) return;
        float ms[8];
        if (p.mscale) un8(ld_raw8(p.mscale + col), ms);
        else {
#pragma unroll
            for (int k = 0; k < 8; ++k) ms[k] = 1.f;
        }
#pragma unroll 1
        for (int q = 0; q < R; ++q) {
            const int r = q * RPP + lane / CPR, row = row0 + r;
            if (row >= rows) continue;
            const int t = div_by(row, p.dWr), wq = row - t * p.Wr, n = div_by(t, p.dHr), hq = t - n * p.Hr;
            const size_t base = ((size_t)(n * 2 * p.Hr + 2 * hq) * (2 * p.Wr) + 2 * wq) * p.N + col;
            const size_t off[4] = {0, (size_t)p.N, (size_t)2 * p.Wr * p.N, (size_t)2 * p.Wr * p.N + p.N};
            Raw8<bf16_t> xr[4], dr[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                xr[k] = ld_raw8((const bf16_t*)p.pool_x + base + off[k]);
                if (p.pool_acc) dr[k] = ld_raw8((const bf16_t*)p.pool_dst + base + off[k]);
            }
            float x[4][8], d[4][8], v[8];
            un8(ld_raw8(area + r * PITCH + ch), v);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                un8(xr[k], x[k]);
                if (p.pool_acc) un8(dr[k], d[k]);
                else {
#pragma unroll
                    for (int j = 0; j < 8; ++j) d[k][j] = 0.f;
                }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float mx = fmaxf(fmaxf(x[0][j], x[1][j]), fmaxf(x[2][j], x[3][j]));
                float g = bf2f(f2bf(v[j]));          // the value a stored gradient of the pooling output would have had
                if (p.pool_mask && !(mx > 0.f)) g = 0.f;
                g *= ms[j];
                bool found = false;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const bool hit = !found && x[k][j] == mx;
                    found = found || hit;
                    d[k][j] += hit ? g : 0.f;
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) st8((bf16_t*)p.pool_dst + base + off[k], d[k]);
        }
    }
};

__device__ __forceinline__ unsigned tap_bits(int lo, int hi) { return hi > lo ? (1u << hi) - (1u << lo) : 0u; }

}  // namespace lpm
