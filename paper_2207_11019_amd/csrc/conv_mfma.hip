// bf16 weight gradient (eq. 8) on the matrix cores over the flattened output pixels, fp32 accumulation, LDS-staged pixel
// tiles, 4 wavefronts per block; the reduction of the weight gradients' split partial sums.
//   dW[co][tap][ci] = sum_rows dz[row][co] * x[pixel(row,tap)][ci]
// Both operands are stored with the reduction index (the pixel) outermost, so the loader transposes 4 pixels x 8 channels
// in registers before writing K-contiguous rows to LDS.
// The matrix instruction is v_mfma_f32_32x32x16_bf16: each lane supplies 8 consecutive K values of row
// (lane % 32); lane holds D[(i/4)*8 + (lane/32)*4 + i%4][lane % 32] in accumulator element i.
#include "lpm_internal.h"
#include "elem.h"
#include "lds_dma.h"
#include <algorithm>

namespace lpm {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Global operands are read through buffer resources: a 16-byte load whose byte offset lies outside the
// buffer returns zeros, so padding taps, ragged tiles and strided gaps need no branch and no select --
// the loader just hands such chunks the offset OOB.  (Buffers are below 4 GiB; the host checks.)
constexpr unsigned OOB = 0xffffffffu;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
__device__ __forceinline__ uint4 buf_load16(__amdgpu_buffer_rsrc_t r, unsigned off) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
    return make_uint4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ unsigned short buf_load2(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
}

template <int BM, int BN, int WGM, int WGN>
struct TileCfg {
    static constexpr int WTM = BM / WGM, WTN = BN / WGN, MI = WTM / 32, NI = WTN / 32;
    static_assert(WGM * WGN == 4 && WTM % 32 == 0 && WTN % 32 == 0, "4 wavefronts, 32x32 MFMA tiles");
};

// acc[mi][ni] += A-tile(wave rows) * B-tile(wave cols) over one BK-deep K tile held in LDS (rows of LDK elements).
// HALF: the rows are only 8-byte aligned, fetch each operand as two 8-byte reads.
template <int MI, int NI, int BK, int LDK, bool HALF>
__device__ __forceinline__ void mma_tile(const uint16_t* As, const uint16_t* Bs, int arow0, int brow0, int lane,
                                         f32x16 (&acc)[MI][NI]) {
    const int r = lane & 31, kq = (lane >> 5) * 8;
    auto fetch = [&](const uint16_t* ptr) __attribute__((always_inline)) -> bf16x8 {
        if (HALF) {
            const uint2 lo = *reinterpret_cast<const uint2*>(ptr), hi = *reinterpret_cast<const uint2*>(ptr + 4);
            return __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
        }
        return *reinterpret_cast<const bf16x8*>(ptr);
    };
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
        bf16x8 a[MI], b[NI];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) a[mi] = fetch(As + (arow0 + mi * 32 + r) * LDK + ks * 16 + kq);
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) b[ni] = fetch(Bs + (brow0 + ni * 32 + r) * LDK + ks * 16 + kq);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mi], b[ni], acc[mi][ni], 0, 0, 0);
    }
}

// Sum of one element's split-K partials in split order.  The loads are issued eight at a time before the first add (a
// plain loop over a run-time split count waits for every load in turn); the additions keep the order.
__device__ __forceinline__ float sum_partials(const float* __restrict__ part, int splits, int64_t stride, int64_t i) {
    float v = 0.f;
    for (int s0 = 0; s0 < splits; s0 += 8) {
        float t[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) t[k] = s0 + k < splits ? part[(int64_t)(s0 + k) * stride + i] : 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) if (s0 + k < splits) v = (s0 + k == 0) ? t[k] : v + t[k];
    }
    return v;
}

// sums split-K partials in split order and applies the epilogue
__global__ void __launch_bounds__(256) splitk_epilogue(const float* __restrict__ part, int splits, int64_t MN, int N,
                                                       const float* __restrict__ scale, const float* __restrict__ bias,
                                                       const uint16_t* __restrict__ add, int relu, int accumulate,
                                                       const uint16_t* __restrict__ mask, const float* __restrict__ mscale,
                                                       uint16_t* __restrict__ C, uint16_t* __restrict__ C2, int acc2,
                                                       const float* __restrict__ c2scale) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= MN) return;
    float v = sum_partials(part, splits, MN, i);
    const int col = (int)((unsigned)i % (unsigned)N);      // (the output has fewer than 2^31 elements)
    if (scale) v *= scale[col];
    if (bias) v += bias[col];
    if (add) v += bf2f(add[i]);
    if (accumulate) v += bf2f(C[i]);
    if (relu) v = fmaxf(v, 0.f);
    if (mask && !(bf2f(mask[i]) > 0.f)) v = 0.f;
    if (C2) {
        const float u = c2scale ? v * c2scale[col] : v;
        C2[i] = f2bf(acc2 ? u + bf2f(C2[i]) : u);
    }
    if (mscale) v *= mscale[col];
    C[i] = f2bf(v);
}

hipError_t launch_splitk_epilogue(const float* part, int splits, int64_t MN, int N, const float* scale, const float* bias,
                                  const void* add, int relu, int accumulate, const void* mask, const float* mscale,
                                  void* C, hipStream_t st) {
    hipLaunchKernelGGL(splitk_epilogue, dim3((unsigned)((MN + 255) / 256)), dim3(256), 0, st, part, splits, MN, N, scale, bias,
                       (const uint16_t*)add, relu, accumulate, (const uint16_t*)mask, mscale, (uint16_t*)C, (uint16_t*)nullptr, 0, (const float*)nullptr);
    return hipGetLastError();
}

// 32-bit byte offsets into every operand, 32-bit element counts of the output
static bool fits32(const ConvGeom& g) {
    const int64_t lim = (int64_t)1 << 31;
    return g.rows_in() * g.Cin < lim && g.rows_out() * g.Cout < lim && (int64_t)g.Cout * g.K() < lim;
}

// --------------------------------------------------------------------------------------------------
// weight gradient
struct WgradArgs {
    const uint16_t* X;
    const uint16_t* DZ;
    float* out;            // dW, or the partials base when splits > 1
    float* db;             // bias gradient (column sums of dz), or NULL
    const float* rscale;   // the layer's per-channel scale, or NULL: dz is the gradient before that scale, so row co of dW is multiplied by it
    size_t part_stride;    // floats between the partials of consecutive splits (>= Cout*K + Cout)
    unsigned dz_bytes, x_bytes;   // extents of DZ and X for the buffer resources
    int Cout, Cin, KhKw, Kw;
    int H, W, Ho, Wo, stride, pad;
    int R;                 // reduction length m*Ho*Wo
    int rt_total, rt_per_split, splits;
    int accumulate;
    int co_tiles, ci_tiles;
    int x_cin, x_taps;     // flattened mode (see wgrad_kernel): channels and filter taps of the real input
    int Kh, D, Do, pad_d;  // volumetric layers: filter height (KhKw then counts Kd*Kh*Kw taps), slices in / out, depth padding
};

template <int LDK>
__device__ __forceinline__ void transpose4x8_store(const uint4 (&q)[4], uint16_t* dst /* row 0 of the 8 channels */) {
    const uint32_t d[4][4] = {{q[0].x, q[0].y, q[0].z, q[0].w}, {q[1].x, q[1].y, q[1].z, q[1].w},
                              {q[2].x, q[2].y, q[2].z, q[2].w}, {q[3].x, q[3].y, q[3].z, q[3].w}};
#pragma unroll
    for (int pr = 0; pr < 4; ++pr) {
        // channel 2*pr: low halves; channel 2*pr+1: high halves; 4 pixels -> 8 bytes, K-contiguous
        const uint32_t lo0 = __builtin_amdgcn_perm(d[1][pr], d[0][pr], 0x05040100u);
        const uint32_t lo1 = __builtin_amdgcn_perm(d[3][pr], d[2][pr], 0x05040100u);
        const uint32_t hi0 = __builtin_amdgcn_perm(d[1][pr], d[0][pr], 0x07060302u);
        const uint32_t hi1 = __builtin_amdgcn_perm(d[3][pr], d[2][pr], 0x07060302u);
        *reinterpret_cast<uint2*>(dst + (2 * pr) * LDK) = make_uint2(lo0, lo1);
        *reinterpret_cast<uint2*>(dst + (2 * pr + 1) * LDK) = make_uint2(hi0, hi1);
    }
}

// FLAT: for an input of very few channels (an image: Cin*Kh*Kw <= BN) the N dimension of the tile is the
// flattened (tap, channel) index instead of the channels of one tap; its operand is gathered 2 bytes at a time.
// There p.Cin holds Cin*Kh*Kw and p.KhKw is 1, so the output index is the same expression in both modes.
template <int BM, int BN, int BK, bool FLAT>
__global__ void __launch_bounds__(256, 2) wgrad_kernel(WgradArgs p) {
    typedef TileCfg<BM, BN, 2, 2> Cfg;
    // LDS rows of BK + 12 elements: 8 rows apart is 192 bytes apart modulo the 256-byte bank period, so the 4
    // channel chunks x 8 pixel groups a half-wavefront writes per step fall on distinct banks (an item mapping
    // with all 16 chunks in one wavefront put 88 % of the LDS cycles into bank conflicts).
    constexpr int LDK = BK + 12;
    constexpr int RGS = BK / 4;       // pixel groups per tile
    constexpr int A_ITEMS = (BM / 8) * (BK / 4), B_ITEMS = (BN / 8) * (BK / 4);   // item = 4 pixels x 8 channels
    constexpr int A_PT = (A_ITEMS + 255) / 256, B_PT = (B_ITEMS + 255) / 256;
    __shared__ __attribute__((aligned(16))) uint16_t As[2][BM * LDK];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][BN * LDK];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    // Workgroups go to the 8 XCDs round-robin in launch order (x fastest, then z).  All tiles of one pixel range
    // read the same dz and x rows (each filter tap a shifted copy), so they are given to one XCD, whose L2 then
    // serves the repeats: virtual index = position in the XCD's contiguous share, pixel range outermost.
    const int v_id = xcd_remap((int)(blockIdx.z * gridDim.x + blockIdx.x), (int)(gridDim.x * gridDim.z));
    const int split = v_id / (int)gridDim.x;
    int tile = v_id - split * (int)gridDim.x;
    const int ci_t = tile % p.ci_tiles; tile /= p.ci_tiles;
    const int tap = tile % p.KhKw;
    const int co_t = tile / p.KhKw;
    const int co0 = co_t * BM, ci0 = ci_t * BN;
    const int kd = tap / (p.Kh * p.Kw), tap2 = tap - kd * (p.Kh * p.Kw);
    const int kh = tap2 / p.Kw, kw = tap2 - kh * p.Kw;
    const int rt0 = split * p.rt_per_split, rt1 = min(p.rt_total, rt0 + p.rt_per_split);

    // Two pixel tiles in flight in registers; out-of-range items (ragged channels, pixels past the end, taps
    // in the padding) load zeros through the buffer resources.
    const __amdgpu_buffer_rsrc_t rsD = make_rsrc(p.DZ, p.dz_bytes), rsX = make_rsrc(p.X, p.x_bytes);
    uint4 qa0[A_PT][4], qb0[B_PT][4], qa1[A_PT][4], qb1[B_PT][4];
    unsigned short qs0[B_PT][4][8], qs1[B_PT][4][8];      // FLAT: the raw 2-byte gathers of the B items

    // Cursors of the next pixel tile to load (tiles are loaded strictly in order).  Per item: the first of its
    // 4 pixels as (row index, wo, ho, image); a tile step adds BK pixels with carries, pixels 1..3 follow by +1.
    const int step_wo = BK % p.Wo, step_q = BK / p.Wo, step_ho = step_q % p.Ho, step_n = step_q / p.Ho;
    int cur_rt = rt0;
    int a_r[A_PT];
    unsigned a_off[A_PT];
    bool a_chok[A_PT];
    int b_r[B_PT], b_wo[B_PT], b_ho[B_PT], b_n[B_PT];
    unsigned b_choff[B_PT];
    bool b_chok[B_PT];
#pragma unroll
    for (int t = 0; t < A_PT; ++t) {
        const int item = tid + t * 256, rg = (item >> 2) % RGS, cc = (item & 3) + 4 * (item / (4 * RGS));
        const int ch = co0 + cc * 8;
        a_chok[t] = (item < A_ITEMS) & (ch < p.Cout);
        a_r[t] = rt0 * BK + rg * 4;
        a_off[t] = (unsigned)(a_r[t] * p.Cout + ch) * 2u;
    }
#pragma unroll
    for (int t = 0; t < B_PT; ++t) {
        const int item = tid + t * 256, rg = (item >> 2) % RGS, cc = (item & 3) + 4 * (item / (4 * RGS));
        const int ch = ci0 + cc * 8;
        b_chok[t] = (item < B_ITEMS) & (ch < p.Cin);
        b_choff[t] = (unsigned)ch * 2u;
        b_r[t] = rt0 * BK + rg * 4;
        const int q = b_r[t] / p.Wo;
        b_wo[t] = b_r[t] - q * p.Wo; b_ho[t] = q % p.Ho; b_n[t] = q / p.Ho;
    }
    // FLAT: the 8 (tap, channel) indices of an item -- element offset from the pixel at tap (0,0), and the tap
    int f_off[B_PT][8], f_hw[B_PT][8];        // f_hw = kd << 24 | kh << 12 | kw, or -1 when the index is past Cin*Kd*Kh*Kw
    if (FLAT) {
#pragma unroll
        for (int t = 0; t < B_PT; ++t) {
            const int item = tid + t * 256, cc = (item & 3) + 4 * (item / (4 * RGS));
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = ci0 + cc * 8 + e;
                const int tp = k / p.x_cin, ci = k - tp * p.x_cin, td = tp / (p.Kh * p.Kw), tr = tp - td * (p.Kh * p.Kw);
                const int th = tr / p.Kw, tw = tr - th * p.Kw;
                const bool ok = (item < B_ITEMS) & (k < p.Cin);
                f_off[t][e] = ((td * p.H + th) * p.W + tw) * p.x_cin + ci;      // (a volume's slices are consecutive images)
                f_hw[t][e] = ok ? ((td << 24) | (th << 12) | tw) : -1;
            }
        }
    }

#define LPM_LOAD_TILE(QA, QB, QS)                                                                            \
    {                                                                                                        \
        const bool live_ = cur_rt < rt1;                                                                     \
        _Pragma("unroll") for (int t = 0; t < A_PT; ++t) {                                                   \
            _Pragma("unroll") for (int j = 0; j < 4; ++j) {                                                  \
                const bool ok_ = a_chok[t] & live_ & (a_r[t] + j < p.R);                                     \
                QA[t][j] = buf_load16(rsD, ok_ ? a_off[t] + (unsigned)(j * p.Cout) * 2u : OOB);              \
            }                                                                                                \
            a_r[t] += BK; a_off[t] += (unsigned)(BK * p.Cout) * 2u;                                          \
        }                                                                                                    \
        _Pragma("unroll") for (int t = 0; t < B_PT; ++t) {                                                   \
            int wo_ = b_wo[t], ho_ = b_ho[t], n_ = b_n[t];                                                   \
            _Pragma("unroll") for (int j = 0; j < 4; ++j) {                                                  \
                if (FLAT) {                                                                                  \
                    const int h0_ = ho_ * p.stride - p.pad, w0_ = wo_ * p.stride - p.pad;                    \
                    int img0_ = n_, d0_ = 0;      /* n_ counts (sample, output slice) pairs */                   \
                    if (p.Do > 1 || p.D > 1) { const int ns_ = n_ / p.Do; d0_ = (n_ - ns_ * p.Do) * p.stride - p.pad_d; img0_ = ns_ * p.D + d0_; } \
                    const int base_ = ((img0_ * p.H + h0_) * p.W + w0_) * p.x_cin;                           \
                    const bool pix_ = live_ & (b_r[t] + j < p.R);                                            \
                    _Pragma("unroll") for (int e = 0; e < 8; ++e) {                                          \
                        const int hw_ = f_hw[t][e];                                                          \
                        const bool ok_ = pix_ & (hw_ >= 0) & ((unsigned)(h0_ + ((hw_ >> 12) & 0xfff)) < (unsigned)p.H) & \
                                         ((unsigned)(w0_ + (hw_ & 0xfff)) < (unsigned)p.W) &                 \
                                         ((unsigned)(d0_ + (hw_ >> 24)) < (unsigned)p.D);                    \
                        QS[t][j][e] = buf_load2(rsX, ok_ ? (unsigned)(base_ + f_off[t][e]) * 2u : OOB);      \
                    }                                                                                        \
                } else {                                                                                     \
                    const int h_ = ho_ * p.stride + kh - p.pad, w_ = wo_ * p.stride + kw - p.pad;            \
                    int img_ = n_, d_ = 0;        /* n_ counts (sample, output slice) pairs */                   \
                    if (p.Do > 1 || p.D > 1) { const int ns_ = n_ / p.Do; d_ = (n_ - ns_ * p.Do) * p.stride + kd - p.pad_d; img_ = ns_ * p.D + d_; } \
                    const bool ok_ = b_chok[t] & live_ & (b_r[t] + j < p.R) & ((unsigned)h_ < (unsigned)p.H) & \
                                     ((unsigned)w_ < (unsigned)p.W) & ((unsigned)d_ < (unsigned)p.D);        \
                    QB[t][j] = buf_load16(rsX, ok_ ? (unsigned)(((img_ * p.H + h_) * p.W + w_) * p.Cin) * 2u + b_choff[t] : OOB); \
                }                                                                                            \
                ++wo_;                                                                                       \
                if (wo_ == p.Wo) { wo_ = 0; ++ho_; if (ho_ == p.Ho) { ho_ = 0; ++n_; } }                     \
            }                                                                                                \
            b_r[t] += BK;                                                                                    \
            b_wo[t] += step_wo; b_ho[t] += step_ho; b_n[t] += step_n;                                        \
            if (b_wo[t] >= p.Wo) { b_wo[t] -= p.Wo; ++b_ho[t]; }                                             \
            if (b_ho[t] >= p.Ho) { b_ho[t] -= p.Ho; ++b_n[t]; }                                              \
        }                                                                                                    \
        ++cur_rt;                                                                                            \
    }
#define LPM_STORE_TILE(BUF, QA, QB, QS)                                                                      \
    {                                                                                                        \
        _Pragma("unroll") for (int t = 0; t < A_PT; ++t) {                                                   \
            const int item_ = tid + t * 256, rg_ = (item_ >> 2) % RGS, cc_ = (item_ & 3) + 4 * (item_ / (4 * RGS)); \
            if (item_ < A_ITEMS) transpose4x8_store<LDK>(QA[t], &As[BUF][(cc_ * 8) * LDK + rg_ * 4]);        \
        }                                                                                                    \
        _Pragma("unroll") for (int t = 0; t < B_PT; ++t) {                                                   \
            const int item_ = tid + t * 256, rg_ = (item_ >> 2) % RGS, cc_ = (item_ & 3) + 4 * (item_ / (4 * RGS)); \
            if (FLAT) {                                                                                      \
                _Pragma("unroll") for (int j = 0; j < 4; ++j)                                                \
                    QB[t][j] = make_uint4(QS[t][j][0] | ((uint32_t)QS[t][j][1] << 16), QS[t][j][2] | ((uint32_t)QS[t][j][3] << 16), \
                                          QS[t][j][4] | ((uint32_t)QS[t][j][5] << 16), QS[t][j][6] | ((uint32_t)QS[t][j][7] << 16)); \
            }                                                                                                \
            if (item_ < B_ITEMS) transpose4x8_store<LDK>(QB[t], &Bs[BUF][(cc_ * 8) * LDK + rg_ * 4]);        \
        }                                                                                                    \
    }

    f32x16 acc[Cfg::MI][Cfg::NI];
#pragma unroll
    for (int mi = 0; mi < Cfg::MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < Cfg::NI; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.f;

    // the blocks of filter tap 0 / Cin tile 0 also sum their dz tile over the pixels: the bias gradient
    const bool do_bias = p.db != nullptr && tap == 0 && ci_t == 0;
    float bsum = 0.f;

    const int wm = wave >> 1, wn = wave & 1;
    auto bias_tile = [&](int buf) __attribute__((always_inline)) {
        if (do_bias && tid < BM) {
            const uint2* rowp = reinterpret_cast<const uint2*>(&As[buf][tid * LDK]);
#pragma unroll
            for (int k = 0; k < BK / 4; ++k) {
                const uint2 v = rowp[k];
                bsum += (bf2f((uint16_t)(v.x & 0xffffu)) + bf2f((uint16_t)(v.x >> 16))) +
                        (bf2f((uint16_t)(v.y & 0xffffu)) + bf2f((uint16_t)(v.y >> 16)));
            }
        }
    };
    const int nk = rt1 - rt0;
    if (nk > 0) {
        LPM_LOAD_TILE(qa0, qb0, qs0);
        LPM_LOAD_TILE(qa1, qb1, qs1);
        LPM_STORE_TILE(0, qa0, qb0, qs0);
        __syncthreads();
        // pixel tiles in pairs with no exit in between; an odd count is padded by one all-zero tile
        const int npair = (nk + 1) >> 1;
        for (int it = 0; it < npair; ++it) {
            LPM_LOAD_TILE(qa0, qb0, qs0);
            bias_tile(0);
            mma_tile<Cfg::MI, Cfg::NI, BK, LDK, true>(As[0], Bs[0], wm * Cfg::WTM, wn * Cfg::WTN, lane, acc);
            LPM_STORE_TILE(1, qa1, qb1, qs1);
            __syncthreads();
            LPM_LOAD_TILE(qa1, qb1, qs1);
            bias_tile(1);
            mma_tile<Cfg::MI, Cfg::NI, BK, LDK, true>(As[1], Bs[1], wm * Cfg::WTM, wn * Cfg::WTN, lane, acc);
            LPM_STORE_TILE(0, qa0, qb0, qs0);
            __syncthreads();
        }
    }
#undef LPM_LOAD_TILE
#undef LPM_STORE_TILE

    const size_t total = (size_t)p.Cout * p.KhKw * p.Cin;
    float* out = p.out + (p.splits > 1 ? (size_t)split * p.part_stride : 0);
    if (do_bias && tid < BM && co0 + tid < p.Cout) {
        const int co = co0 + tid;
        if (p.splits > 1) out[total + co] = bsum;
        else {
            p.db[co] = p.accumulate ? p.db[co] + bsum : bsum;
        }
    }
    const int col_l = lane & 31, rq = (lane >> 5) * 4;
#pragma unroll
    for (int ni = 0; ni < Cfg::NI; ++ni) {
        const int ci = ci0 + wn * Cfg::WTN + ni * 32 + col_l;
        if (ci >= p.Cin) continue;
#pragma unroll
        for (int mi = 0; mi < Cfg::MI; ++mi)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int co = co0 + wm * Cfg::WTM + mi * 32 + (i >> 2) * 8 + rq + (i & 3);
                if (co >= p.Cout) continue;
                const size_t o = ((size_t)co * p.KhKw + tap) * p.Cin + ci;
                float v = acc[mi][ni][i];
                if (p.splits == 1 && p.rscale) v *= p.rscale[co];
                if (p.splits == 1 && p.accumulate) v += out[o];
                out[o] = v;
            }
    }
}

struct WgradPlan { int bk, splits, rt_total, rt_per, co_tiles; };

// threads that share four outputs of a reduction
__host__ __device__ inline int reduce_lanes(int splits) { return splits > 64 ? 16 : splits > 16 ? 4 : 1; }

struct ReduceBatchArgs {
    ReduceDesc d[LPM_REDUCE_BATCH];
    int64_t first[LPM_REDUCE_BATCH + 1];     // first thread of every reduction (a thread sums four outputs)
    int count;
};

// A thread sums four consecutive outputs over the splits with 16-byte loads, eight splits in flight (split s goes to
// chain s % 4, the chains are added pairwise at the end: a fixed order); the bias part and ragged ends go one by one.
// With many splits (a layer of few weights and many pixels) a group of `lanes` = 4 or 16 threads shares four outputs: each
// takes a contiguous part of the splits, and the sums are added by lane exchanges in a fixed order.
template <int LANES>
__device__ __forceinline__ void reduce_one(const ReduceDesc& d, int64_t t) {
    const int part = LANES > 1 ? (int)(t % LANES) : 0;
    const int64_t i = t / LANES * 4;
    const int per = (d.splits + LANES - 1) / LANES, s0 = part * per, s1 = min(d.splits, s0 + per);
    if (i >= d.n + d.nb) return;              // padding up to a whole block (whole groups)
    if (i + 4 <= d.n && (d.stride & 3) == 0 && (d.row_len & 3) == 0) {
        float4 c[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) c[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        const float* p = d.part + i;
        int s = s0;
        for (; s + 8 <= s1; s += 8) {
            float4 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const float4*>(p + (size_t)(s + j) * d.stride);
#pragma unroll
            for (int j = 0; j < 8; ++j) { c[j & 3].x += v[j].x; c[j & 3].y += v[j].y; c[j & 3].z += v[j].z; c[j & 3].w += v[j].w; }
        }
        float4 v[7];
#pragma unroll
        for (int j = 0; j < 7; ++j) v[j] = s + j < s1 ? *reinterpret_cast<const float4*>(p + (size_t)(s + j) * d.stride) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int j = 0; j < 7; ++j) { c[j & 3].x += v[j].x; c[j & 3].y += v[j].y; c[j & 3].z += v[j].z; c[j & 3].w += v[j].w; }
        float4 r = make_float4((c[0].x + c[1].x) + (c[2].x + c[3].x), (c[0].y + c[1].y) + (c[2].y + c[3].y),
                               (c[0].z + c[1].z) + (c[2].z + c[3].z), (c[0].w + c[1].w) + (c[2].w + c[3].w));
#pragma unroll
        for (int o = 1; o < LANES; o <<= 1) {
            r.x += __shfl_xor(r.x, o); r.y += __shfl_xor(r.y, o); r.z += __shfl_xor(r.z, o); r.w += __shfl_xor(r.w, o);
        }
        if (part) return;
        if (d.rscale) {                           // (row_len is a multiple of 4 on this path: the four outputs share a row)
            const float f = d.rscale[i / d.row_len];
            r.x *= f; r.y *= f; r.z *= f; r.w *= f;
        }
        float4* o = reinterpret_cast<float4*>(d.dst + i);
        if (d.accumulate) { const float4 q = *o; r.x += q.x; r.y += q.y; r.z += q.z; r.w += q.w; }
        *o = r;
        return;
    }
    for (int64_t e = i; e < i + 4 && e < d.n + d.nb; ++e) {
        float acc = 0.f;
        for (int s = s0; s < s1; ++s) acc += d.part[(size_t)s * d.stride + e];
#pragma unroll
        for (int o = 1; o < LANES; o <<= 1) acc += __shfl_xor(acc, o);
        if (part) continue;
        if (e < d.n) {
            if (d.rscale) acc *= d.rscale[e / d.row_len];
            d.dst[e] = d.accumulate ? d.dst[e] + acc : acc;
        } else {
            const int c = (int)(e - d.n);
            d.db[c] = d.accumulate ? d.db[c] + acc : acc;
        }
    }
}

__global__ void __launch_bounds__(256) wgrad_reduce_batch(ReduceBatchArgs a) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int k = 0;                                    // (a block never straddles two reductions)
    while (k + 1 < a.count && (int64_t)blockIdx.x * 256 >= a.first[k + 1]) ++k;
    const int lanes = reduce_lanes(a.d[k].splits);
    if (lanes == 16) reduce_one<16>(a.d[k], t - a.first[k]);
    else if (lanes == 4) reduce_one<4>(a.d[k], t - a.first[k]);
    else reduce_one<1>(a.d[k], t - a.first[k]);
}

hipError_t launch_reduce_batch(const ReduceDesc* d, int count, hipStream_t st) {
    for (int done = 0; done < count;) {
        ReduceBatchArgs a{};
        int64_t tot = 0;
        int k = 0;
        for (; k < LPM_REDUCE_BATCH && done + k < count; ++k) {
            a.d[k] = d[done + k];
            a.first[k] = tot;
            // a thread per four outputs, whole blocks per reduction: a block never straddles two of them
            tot += (((a.d[k].n + a.d[k].nb + 3) / 4 * reduce_lanes(a.d[k].splits) + 255) / 256) * 256;
        }
        a.first[k] = tot;
        a.count = k;
        done += k;
        if (tot == 0) continue;
        hipLaunchKernelGGL(wgrad_reduce_batch, dim3((unsigned)(tot / 256)), dim3(256), 0, st, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// The same reduction for a short output vector (a first layer's few thousand weights) and many partials:
// 8 lanes share one output, each adds a contiguous eighth of the partials in order, and the eight sums are
// added in lane order -- a fixed order, with 8 loads in flight per output instead of one.
__global__ void __launch_bounds__(256) wgrad_reduce_short(const float* __restrict__ part, size_t stride, int splits,
                                                          float* __restrict__ dst, int64_t n, float* __restrict__ db, int nb,
                                                          const float* __restrict__ rscale, int row_len, int accumulate) {
    __shared__ float red[8][32];
    const int o = threadIdx.x & 31, l = threadIdx.x >> 5;
    const int64_t i = (int64_t)blockIdx.x * 32 + o;
    float acc = 0.f;
    if (i < n + nb) {
        const int per = (splits + 7) / 8;
        const int s1 = min(splits, (l + 1) * per);
        for (int s = l * per; s < s1; ++s) acc += part[(size_t)s * stride + i];
    }
    red[l][o] = acc;
    __syncthreads();
    if (l != 0 || i >= n + nb) return;
    float v = red[0][o];
#pragma unroll
    for (int k = 1; k < 8; ++k) v += red[k][o];
    if (i < n) {
        if (rscale) v *= rscale[i / row_len];
        dst[i] = accumulate ? dst[i] + v : v;
    } else {
        const int c = (int)(i - n);
        db[c] = accumulate ? db[c] + v : v;
    }
}

// Weight gradient of an image-input layer (Cin*Kh*Kw <= 64): one N tile holds every (tap, channel) index.
bool mfma_wgrad_flat_ok(const ConvGeom& g) { return g.K() <= 64 && g.Cout % 8 == 0 && fits32(g); }

static WgradPlan plan_wgrad_flat(const ConvGeom& g) {
    WgradPlan pl{};
    const int64_t R = g.rows_out();
    pl.bk = R >= 1024 ? 128 : 64;
    pl.rt_total = (int)((R + pl.bk - 1) / pl.bk);
    pl.co_tiles = (g.Cout + 63) / 64;
    // the 2-byte gathers make a pixel tile slow (about 2 us), so blocks take as few as two of them
    int s = std::min(std::min(512 / pl.co_tiles, std::max(1, pl.rt_total / 2)), 256);
    pl.rt_per = (pl.rt_total + s - 1) / s;
    pl.splits = (pl.rt_total + pl.rt_per - 1) / pl.rt_per;
    return pl;
}

size_t mfma_wgrad_flat_ws_bytes(const ConvGeom& g) {
    const WgradPlan pl = plan_wgrad_flat(g);
    return pl.splits > 1 ? (size_t)pl.splits * ((size_t)g.Cout * g.K() + g.Cout) * sizeof(float) : 0;
}

hipError_t mfma_conv_wgrad_flat(const ConvGeom& g, const void* x, const void* dz, float* dw, float* dbias,
                                const float* rscale, int accumulate, void* ws, hipStream_t st) {
    const WgradPlan pl = plan_wgrad_flat(g);
    WgradArgs a{};
    a.X = (const uint16_t*)x; a.DZ = (const uint16_t*)dz;
    a.out = pl.splits > 1 ? (float*)ws : dw;
    a.Cout = g.Cout; a.Cin = g.K(); a.KhKw = 1; a.Kw = g.Kw;
    a.Kh = g.Kh; a.D = g.D; a.Do = g.Do; a.pad_d = g.pad_d;
    a.x_cin = g.Cin; a.x_taps = g.taps();
    a.H = g.H; a.W = g.W; a.Ho = g.Ho; a.Wo = g.Wo; a.stride = g.stride; a.pad = g.pad;
    a.R = (int)g.rows_out();
    a.db = dbias; a.rscale = rscale;
    a.part_stride = (size_t)g.Cout * g.K() + g.Cout;
    a.dz_bytes = (unsigned)(g.rows_out() * g.Cout * 2); a.x_bytes = (unsigned)(g.rows_in() * g.Cin * 2);
    a.rt_total = pl.rt_total; a.rt_per_split = pl.rt_per; a.splits = pl.splits;
    a.accumulate = accumulate;
    a.co_tiles = pl.co_tiles; a.ci_tiles = 1;
    const dim3 grid((unsigned)pl.co_tiles, 1, pl.splits);
    if (pl.bk == 128) hipLaunchKernelGGL((wgrad_kernel<64, 64, 128, true>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((wgrad_kernel<64, 64, 64, true>), grid, dim3(256), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || pl.splits == 1) return e;
    const int64_t n = (int64_t)g.Cout * g.K();
    const int nb = dbias ? g.Cout : 0;
    hipLaunchKernelGGL(wgrad_reduce_short, dim3((unsigned)((n + nb + 31) / 32)), dim3(256), 0, st, (const float*)ws,
                       a.part_stride, pl.splits, dw, n, dbias, nb, rscale, g.K(), accumulate);
    return hipGetLastError();
}

}  // namespace lpm
