// What the contraction kernels share: their arguments and the epilogue that a wavefront runs on its piece of the output.
#pragma once
#include "lpm_internal.h"
#include "elem.h"

namespace lpm {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr unsigned OOB = 0xffffffffu;

enum { MODE_FWD = 0, MODE_DGRAD = 1 /* stride 1 */, MODE_DGRAD_S = 2 /* stride 2..4, by residue class */, MODE_UNPOOL = 3 /* stride 1, routed through a max-pooling */ };

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
    const void* add;
    const void* mask;       // data gradient: zero the result where this tensor (the producer's output) is <= 0
    const float* mscale;    // data gradient: then multiply by the producer's per-channel scale
    void* C2;               // data gradient: the masked, not yet scaled result also goes here (the producer's shortcut), or NULL
    const float* c2scale;   // ... times this per-channel factor (NULL: 1)
    int acc2;               // ... added to what C2 holds
    int relu, accumulate;
    int M, N;
    int Hi, Wi, Di, Ci;     // extent of the gathered tensor
    int Hr, Wr, Dr;         // extent of the row space
    int Kh, Kw, Kd, stride, pad, pad_d;
    FastDiv dWr, dHr, dDr, dCc;       // row decoding; chunks per tap
    unsigned a_bytes, b_bytes, b_pitch;
    int kt_total, kt_per_split, splits;
    int free_taps;          // no tap can leave the image: no mask bits needed
    int tiles_m;            // (strided) row tiles over all classes
    int cls_tile0[17];      // strided data gradient: first row tile of class c = (pd * s + ph) * s + pw
    const uint16_t* pool_x; // stride-1 data gradient routed through a 2x2 max-pooling (see UnpoolDesc): its input [m][2*Hr][2*Wr][N]
    uint16_t* pool_dst;
    int pool_acc, pool_mask;
    uint16_t* fwd_pool;     // forward: also store the 2x2 max-pooling of C, [m][Hr/2][Wr/2][N] (Wr = 2, 4, 8 or 16)
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
    const int wq = row % Wc, t = row / Wc, hq = t % Hc;
    int n = t / Hc, img = n;
    if (p.Dr > 1) { const int dq = n % Dc; n /= Dc; img = n * p.Dr + dq * p.stride + pd; }
    return (img * p.Hr + hq * p.stride + ph) * p.Wr + wq * p.stride + pw;
}

// One wavefront's 32 x (32*NIW) piece of the output, held in its private LDS area `tile` (rows of 32*NIW + 4 floats): a lane
// takes 8 channels of a row at a time, so every tensor access is 16 (float: 32) bytes.  The operands of all the lane's
// pieces are requested before the first is used.
template <typename E, int NIW, int MODE>
__device__ __forceinline__ void store_piece(const IgemmArgs& p, float* tile, int row0, int col0, int rows, int lane,
                                            int Hc, int Wc, int ph, int pw, int Dc, int pd) {
    constexpr bool FWD = MODE == MODE_FWD;   // (forward: scale, bias, add, relu; data gradient: accumulate, add, mask, C2, mscale)
    constexpr int PITCH = NIW * 32 + 4, CPR = NIW * 4, RPP = 64 / CPR, NP = 32 / RPP;
    const int ch = (lane % CPR) * 8, col = col0 + ch;
    const E* add = (const E*)p.add;
    const E* msk = (const E*)p.mask;
    E* out = (E*)p.C;
    E* out2 = (E*)p.C2;
    if (p.N & 7) {                           // ragged rows: the lanes take consecutive elements
        const int nc = min(p.N - col0, NIW * 32), total = nc > 0 ? min(32, rows - row0) * nc : 0;
#pragma unroll 1
        for (int i = lane; i < total; i += 64) {
            const int r = i / nc, c = i - r * nc, row = row0 + r, cc = col0 + c;
            const size_t prow = MODE == MODE_DGRAD_S ? (size_t)class_pixel(p, row, Hc, Wc, ph, pw, Dc, pd) : (size_t)row;
            const size_t o = prow * p.N + cc;
            float v = tile[r * PITCH + c];
            if (FWD && p.scale) v *= p.scale[cc];
            if (FWD && p.bias) v += p.bias[cc];
            if (add) v += ld(add, o);
            if (!FWD && p.accumulate) v += ld(out, o);
            if (FWD && p.relu) v = fmaxf(v, 0.f);
            if (!FWD && msk && !(ld(msk, o) > 0.f)) v = 0.f;
            if (!FWD && out2) {
                const float u = p.c2scale ? v * p.c2scale[cc] : v;
                st(out2, o, p.acc2 ? u + ld(out2, o) : u);
            }
            if (!FWD && p.mscale) v *= p.mscale[cc];
            st(out, o, v);
        }
        return;
    }
    const bool cok = col < p.N;
    float sc[8], bi[8], ms[8], c2[8];
    auto vec = [&](const float* q, float (&d)[8], float fill) __attribute__((always_inline)) {
        if (q && cok) un8(ld_raw8(q + col), d);
        else {
#pragma unroll
            for (int k = 0; k < 8; ++k) d[k] = fill;
        }
    };
    if (FWD) { vec(p.scale, sc, 1.f); vec(p.bias, bi, 0.f); }
    else { vec(p.mscale, ms, 1.f); vec(p.c2scale, c2, 1.f); }
    if constexpr (MODE == MODE_UNPOOL) {
        // gradient of a 2x2 max-pooling output: to the first maximum of the window (row-major), through the producer's ReLU
        // and scale where asked; all four window positions are written
        static_assert(sizeof(E) == 2, "bf16 only");
#pragma unroll 1
        for (int q = 0; q < NP; ++q) {
            const int r = q * RPP + lane / CPR, row = row0 + r;
            if (row >= rows || !cok) continue;
            const int t = div_by(row, p.dWr), wq = row - t * p.Wr, n = div_by(t, p.dHr), hq = t - n * p.Hr;
            const size_t base = ((size_t)(n * 2 * p.Hr + 2 * hq) * (2 * p.Wr) + 2 * wq) * p.N + col;
            const size_t off[4] = {0, (size_t)p.N, (size_t)2 * p.Wr * p.N, (size_t)2 * p.Wr * p.N + p.N};
            Raw8<bf16_t> xr[4], dr[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                xr[k] = ld_raw8((const bf16_t*)p.pool_x + base + off[k]);
                if (p.pool_acc) dr[k] = ld_raw8((const bf16_t*)p.pool_dst + base + off[k]);
            }
            float x[4][8], o[4][8], v[8];
            un8(ld_raw8(tile + r * PITCH + ch), v);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                un8(xr[k], x[k]);
                if (p.pool_acc) un8(dr[k], o[k]);
                else {
#pragma unroll
                    for (int j = 0; j < 8; ++j) o[k][j] = 0.f;
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
                    o[k][j] += hit ? g : 0.f;
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) st8((bf16_t*)p.pool_dst + base + off[k], o[k]);
        }
        return;
    }
    size_t o[NP];
    bool live[NP];
    Raw8<E> ra[NP], rc[NP], rm[NP], r2[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        const int row = row0 + q * RPP + lane / CPR;
        live[q] = row < rows && cok;
        const int prow = MODE == MODE_DGRAD_S && live[q] ? class_pixel(p, row, Hc, Wc, ph, pw, Dc, pd) : row;
        o[q] = live[q] ? (size_t)prow * p.N + col : 0;
    }
#pragma unroll
    for (int q = 0; q < NP; ++q) if (add) ra[q] = ld_raw8(add + o[q]);
#pragma unroll
    for (int q = 0; q < NP; ++q) if (!FWD && p.accumulate) rc[q] = ld_raw8((const E*)out + o[q]);
#pragma unroll
    for (int q = 0; q < NP; ++q) if (!FWD && msk) rm[q] = ld_raw8(msk + o[q]);
#pragma unroll
    for (int q = 0; q < NP; ++q) if (!FWD && out2 && p.acc2) r2[q] = ld_raw8((const E*)out2 + o[q]);
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        const int r = q * RPP + lane / CPR;
        float v[8], t[8];
        un8(ld_raw8(tile + r * PITCH + ch), v);
        if (FWD) {
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = v[k] * sc[k] + bi[k];
        }
        if (add) { un8(ra[q], t);
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] += t[k]; }
        if (!FWD && p.accumulate) { un8(rc[q], t);
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] += t[k]; }
        if (FWD && p.relu) {
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = fmaxf(v[k], 0.f); }
        if (!FWD && msk) { un8(rm[q], t);
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = t[k] > 0.f ? v[k] : 0.f; }
        if (!FWD && out2) {
            float u[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) u[k] = v[k] * c2[k];
            if (p.acc2) { un8(r2[q], t);
#pragma unroll
                for (int k = 0; k < 8; ++k) u[k] += t[k]; }
            if (live[q]) st8(out2 + o[q], u);
        }
        if (!FWD) {
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] *= ms[k];
        }
        if (live[q]) st8(out + o[q], v);
        if (MODE == MODE_FWD && p.fwd_pool) {
            if constexpr (sizeof(E) == 2) {
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = bf2f(f2bf(v[k]));
                st8(tile + r * PITCH + ch, v);
            }
        }
    }
    if (MODE == MODE_FWD && p.fwd_pool) {
        // the piece's 32 rows are whole pairs of image rows: eight pooling windows of rows (r, r+1, r+Wr, r+Wr+1)
        if constexpr (sizeof(E) == 2) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int w = lane / CPR;
            if (w < 8) {
                const int hw = p.Wr >> 1, py = w / hw, px = w - py * hw, r = 2 * py * p.Wr + 2 * px;
                if (row0 + r < rows && cok) {
                    float a[8], b[8], c[8], d[8];
                    un8(ld_raw8(tile + r * PITCH + ch), a);
                    un8(ld_raw8(tile + (r + 1) * PITCH + ch), b);
                    un8(ld_raw8(tile + (r + p.Wr) * PITCH + ch), c);
                    un8(ld_raw8(tile + (r + p.Wr + 1) * PITCH + ch), d);
#pragma unroll
                    for (int k = 0; k < 8; ++k) a[k] = fmaxf(fmaxf(a[k], b[k]), fmaxf(c[k], d[k]));
                    st8((bf16_t*)p.fwd_pool + (size_t)((row0 >> 2) + w) * p.N + col, a);
                }
            }
        }
    }
}

__device__ __forceinline__ unsigned tap_bits(int lo, int hi) { return hi > lo ? (1u << hi) - (1u << lo) : 0u; }

}  // namespace lpm
