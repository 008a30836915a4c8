// Convolutions whose channel counts do not come in 16-byte chunks -- an image or volume of one to three channels, a first
// layer's six feature maps -- on the matrix cores: forward (eq. 1), stride-1 data gradient (eq. 9) and weight gradient (eq. 8)
// of bfloat16 and float layers, two- and three-dimensional, fp32 accumulation.
//
// The reduction is too short (27 terms for a 3x3 filter over RGB) and its elements too scattered for tiles in LDS: a lane
// gathers its operand straight from memory, element by element, through the L1 cache, where a pixel's neighbours have
// already brought its line in.  Every element is one load whose offset is a sum of two terms, one of the pixel and one of
// (tap, channel); a bit mask per pixel says which taps meet the image, and the others get an offset past the buffer's end
// and read as zero.  What bounds these layers then is the traffic of their other tensor and, for small launches, one memory
// latency per operand.  Measured per launch in a training step (us, the vector-ALU or register-staged kernel before -> this):
// forward 4 x 224^2 x 3 -> 64: 70 -> 29, 16 x 32^2 x 3 -> 64: 13.8 -> 9.9, 2 x 32^3 x 1 -> 32: 60 -> 9.3, float 8 x 32^2 x 3: 18 -> 9;
// weight gradient 4 x 224^2: 42 + 5 (its own reduction) -> 22, 16 x 32^2: 15.3 + 5.4 -> 10, float 8 x 32^2: 58 -> 10.
#include "contraction.h"
#include <algorithm>

namespace lpm {

constexpr unsigned NO_TAP = 1u << 31;          // a bit that no pixel's mask has (filters are less than 8 deep)

template <typename E> struct Gathered;         // one lane's 16-byte operand
template <> struct Gathered<bf16_t> {
    static constexpr int N = 8;
    unsigned short e[8];
    __device__ __forceinline__ void load(int i, __amdgpu_buffer_rsrc_t r, unsigned off) { e[i] = (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0); }
    __device__ __forceinline__ float value(int i) const { return bf2f(e[i]); }
    __device__ __forceinline__ uint4 pack() const {
        return make_uint4(e[0] | ((unsigned)e[1] << 16), e[2] | ((unsigned)e[3] << 16), e[4] | ((unsigned)e[5] << 16), e[6] | ((unsigned)e[7] << 16));
    }
};
template <> struct Gathered<float> {
    static constexpr int N = 4;
    unsigned e[4];
    __device__ __forceinline__ void load(int i, __amdgpu_buffer_rsrc_t r, unsigned off) { e[i] = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0); }
    __device__ __forceinline__ float value(int i) const { return __uint_as_float(e[i]); }
    __device__ __forceinline__ uint4 pack() const { return make_uint4(e[0], e[1], e[2], e[3]); }
};

// c += a * b over the 2 * Gathered<E>::N reduction values of one operand pair (any fixed order of them, the same for both)
template <typename E>
__device__ __forceinline__ void mma(f32x16& c, const uint4& a, const uint4& b) {
    if constexpr (sizeof(E) == 2) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    } else {
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    }
}

// offset (elements) of reduction index k = (tap, channel) from its pixel's tap (0,0,0), and the tap's mask bits
template <int SG>
__device__ __forceinline__ int2 tap_entry(int k, int K, const IgemmArgs& p) {
    if (k >= K) return make_int2(0, (int)NO_TAP);
    const int t = div_by(k, p.dCc), c = k - t * p.Ci, td = div_by(t, p.dKhw), r = t - td * (p.Kh * p.Kw), th = div_by(r, p.dKw), tw = r - th * p.Kw;
    return make_int2(SG * ((td * p.Hi + th) * p.Wi + tw) * p.Ci + c, (int)((1u << (24 + td)) | (1u << (12 + th)) | (1u << tw)));
}
// offset (elements) of row `row`'s tap (0,0,0) and the taps that meet the tensor (none past the last row)
template <bool FWD, bool WIN = false>
__device__ __forceinline__ int2 pixel_entry(const IgemmArgs& p, int row) {
    const bool ok = row < p.M;
    const int rr = ok ? row : 0;
    int n, hq, wq, dq = 0;
    if (WIN) {
        const WinPixel x = win_pixel(p, rr);
        n = x.n; hq = x.h; wq = x.w;
    } else {
        const int t = div_by(rr, p.dWr);
        wq = rr - t * p.Wr;
        n = div_by(t, p.dHr);
        hq = t - n * p.Hr;
    }
    if (p.Dr > 1) { const int ns = div_by(n, p.dDr); dq = n - ns * p.Dr; n = ns; }
    int h0, w0, d0;
    unsigned m;
    if (FWD) {
        h0 = hq * p.stride - p.pad; w0 = wq * p.stride - p.pad; d0 = dq * p.stride - p.pad_d;
        m = (tap_bits(max(0, -d0), min(p.Kd, p.Di - d0)) << 24) | (tap_bits(max(0, -h0), min(p.Kh, p.Hi - h0)) << 12) |
            tap_bits(max(0, -w0), min(p.Kw, p.Wi - w0));
    } else {
        h0 = hq + p.pad; w0 = wq + p.pad; d0 = dq + p.pad_d;
        m = (tap_bits(max(0, d0 - p.Di + 1), min(p.Kd, d0 + 1)) << 24) | (tap_bits(max(0, h0 - p.Hi + 1), min(p.Kh, h0 + 1)) << 12) |
            tap_bits(max(0, w0 - p.Wi + 1), min(p.Kw, w0 + 1));
    }
    return make_int2((((n * p.Di + d0) * p.Hi + h0) * p.Wi + w0) * p.Ci, ok ? (int)m : 0);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* q, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q), 0, bytes, 0x00020000);
}

// Forward and data gradient.  The filter bank lies in LDS, K-contiguous and padded with zeros.
// KSPLIT false: a wavefront takes 32 rows and NT * 32 output channels at a time and walks the row tiles with the stride of the
// grid, so the bank is staged once; the next tile's first loads are requested before this one's epilogue.  KSPLIT true, for
// launches of too few row tiles to fill the card: the four wavefronts of a block share a tile, each with a quarter of the
// reduction, and add their sums through LDS.
template <typename E, int NT, int MODE, bool KSPLIT>
__global__ void __launch_bounds__(256, MODE == MODE_DGRAD ? 2 : 3) gather_gemm(const IgemmArgs p, const int ksteps, const int tiles, const FastDiv dKp, const FastDiv dRows) {
    typedef Gathered<E> G;
    constexpr int ES = sizeof(E), EPC = G::N, KS = 2 * EPC, PIECE = 32 * (NT * 32 + 4);
    constexpr bool FWD = MODE != MODE_DGRAD;
    typedef Epilogue<E, 1, NT, MODE> Ep;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, rl = lane & 31, half = lane >> 5;
    const int Kp = ksteps * KS, pitch = Kp + EPC, taps = p.Kd * p.Kh * p.Kw, K = taps * p.Ci, n0 = blockIdx.y * (NT * 32);
    int2* tab = reinterpret_cast<int2*>(lds);
    E* bank = reinterpret_cast<E*>(lds + Kp * 8);
    float* pieces = reinterpret_cast<float*>(lds + Kp * 8 + NT * 32 * pitch * ES);
    float* piece = pieces + wave * PIECE;
    for (int k = tid; k < Kp; k += 256) tab[k] = tap_entry<FWD ? 1 : -1>(k, K, p);
    const E* w = (const E*)p.B;
    // (rows past the last output channel are not filled: what they add up to is not stored.  With them LeNet's data gradient, six rows
    // of 32, took 15.5 us instead of 10.7, its forward pass 7.6 instead of 6.8.)
    const int rows = min(p.N, NT * 32);
    for (int i0 = tid; i0 < rows * Kp; i0 += 8 * 256) {             // eight elements' loads in flight
        float v[8];
        int at[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * 256;
            int n, k, c = 0;
            int64_t o;
            if (FWD) {                       // w [N][K]
                n = div_by(i, dKp); k = i - n * Kp;
                o = (int64_t)(n0 + n) * K + k;
            } else {                         // w [Ci][taps][N], K = (tap, channel of the gathered tensor)
                k = div_by(i, dRows); n = i - k * rows;
                const int t = div_by(k, p.dCc);
                c = k - t * p.Ci;
                o = ((int64_t)c * taps + t) * p.N + n0 + n;
            }
            at[u] = n * pitch + k;
            const bool in = i < rows * Kp;
            if (!in) at[u] = -1;
            v[u] = in && n0 + n < p.N && k < K ? ld(w, o) : 0.f;
            if (!FWD && p.kscale && in && k < K) v[u] *= p.kscale[c];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) if (at[u] >= 0) st(bank, at[u], v[u]);
    }
    __syncthreads();
    const __amdgpu_buffer_rsrc_t rs = rsrc(p.A, p.a_bytes);
    const int ks0 = KSPLIT ? wave * ((ksteps + 3) / 4) : 0, ks1 = KSPLIT ? min(ksteps, ks0 + (ksteps + 3) / 4) : ksteps;
    int2 px;
    G g[4];                                  // four steps' loads in flight
    auto gather = [&](G& d, int ks) __attribute__((always_inline)) {
        const int4* e = reinterpret_cast<const int4*>(tab + ks * KS + half * EPC);
#pragma unroll
        for (int i = 0; i < EPC; i += 2) {
            const int4 v = e[i >> 1];
            d.load(i, rs, ((unsigned)px.y & (unsigned)v.y) == (unsigned)v.y ? (unsigned)(px.x + v.x) * ES : OOB);
            d.load(i + 1, rs, ((unsigned)px.y & (unsigned)v.w) == (unsigned)v.w ? (unsigned)(px.x + v.z) * ES : OOB);
        }
    };
    auto first = [&](int t) __attribute__((always_inline)) {
        px = pixel_entry<FWD, MODE == MODE_FWD_POOL>(p, t * 32 + rl);
#pragma unroll
        for (int i = 0; i < 4; ++i) if (ks0 + i < ks1) gather(g[i], ks0 + i);
    };
    const int step = KSPLIT ? gridDim.x : gridDim.x * 4;
    int t = KSPLIT ? blockIdx.x : blockIdx.x * 4 + wave;
    if (t < tiles) first(t);
    for (; t < tiles; t += step) {
        f32x16 acc[NT];
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[n][i] = 0.f;
        for (int ks = ks0; ks < ks1; ks += 4) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (ks + i < ks1) {
                    const uint4 b = g[i].pack();
#pragma unroll
                    for (int n = 0; n < NT; ++n)
                        mma<E>(acc[n], *reinterpret_cast<const uint4*>(bank + (n * 32 + rl) * pitch + (ks + i) * KS + half * EPC), b);
                }
                if (ks + 4 + i < ks1) gather(g[i], ks + 4 + i);
            }
        }
        if (t + step < tiles) first(t + step);
        if (KSPLIT) __syncthreads();         // (the pieces of the tile before)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<float4*>(piece + rl * (NT * 32 + 4) + n * 32 + q * 8 + half * 4) =
                    make_float4(acc[n][4 * q], acc[n][4 * q + 1], acc[n][4 * q + 2], acc[n][4 * q + 3]);
        if (KSPLIT) {
            __syncthreads();
            for (int i = tid; i < PIECE; i += 256) pieces[i] = (pieces[i] + pieces[PIECE + i]) + (pieces[2 * PIECE + i] + pieces[3 * PIECE + i]);
            __syncthreads();
            if (wave) continue;
        } else {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        Ep ep;
        ep.load(p, t * 32, n0, p.M, lane, 0, 0, 0, 0, 0, 0);
        ep.store(p, piece, t * 32, n0, p.M, lane, 0, 0, 0, 0, 0, 0);
    }
}

// --------------------------------------------------------------------------------------------------
// Weight gradient: dW[co][k] = sum over pixels of dz[pixel][co] * x[pixel + k].  A block takes 256 pixels at a time, a
// wavefront 64 of them, and holds a CT*32 x KT*32 part of dW; the wavefronts' parts are added through LDS at the end, the
// blocks' by the batched reduction.  Here the (tap, channel) term of an offset belongs to the lane, the pixels' terms come
// from LDS.
struct GwArgs {
    IgemmArgs p;             // geometry of the forward pass (A = x)
    const void* DZ;
    float* out;              // dW, or the partials base when splits > 1
    float* db;
    const float* rscale;
    size_t part_stride;
    unsigned dz_bytes;
    int chunks, per_split, splits, k_tiles, accumulate;
};

template <typename E, int CT, int KT>
__global__ void __launch_bounds__(256) gather_wgrad(const GwArgs a) {
    typedef Gathered<E> G;
    constexpr int ES = sizeof(E), EPC = G::N, KS = 2 * EPC, NW = CT * KT;
    const IgemmArgs& p = a.p;
    __shared__ __attribute__((aligned(16))) int2 px[2][256];
    __shared__ float red[2][NW * 1024];
    __shared__ float bred[4][CT * 32];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, rl = lane & 31, half = lane >> 5;
    const int kt = blockIdx.y % a.k_tiles, ct = blockIdx.y / a.k_tiles, k0 = kt * KT * 32, co0 = ct * CT * 32;
    const int K = p.Kd * p.Kh * p.Kw * p.Ci;
    const __amdgpu_buffer_rsrc_t rx = rsrc(p.A, p.a_bytes), rz = rsrc(a.DZ, a.dz_bytes);
    int2 ke[KT];
    unsigned ce[CT];
#pragma unroll
    for (int i = 0; i < KT; ++i) ke[i] = tap_entry<1>(k0 + i * 32 + rl, K, p);
#pragma unroll
    for (int i = 0; i < CT; ++i) ce[i] = co0 + i * 32 + rl < p.N ? (unsigned)(co0 + i * 32 + rl) : OOB;
    f32x16 acc[CT][KT];
    float bs[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        bs[c] = 0.f;
#pragma unroll
        for (int k = 0; k < KT; ++k)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[c][k][i] = 0.f;
    }
    const int c0 = blockIdx.x * a.per_split, c1 = min(a.chunks, c0 + a.per_split);
    px[0][tid] = pixel_entry<true>(p, c0 * 256 + tid);
    for (int ch = c0, b = 0; ch < c1; ++ch, b ^= 1) {
        __syncthreads();
        if (ch + 1 < c1) px[b ^ 1][tid] = pixel_entry<true>(p, (ch + 1) * 256 + tid);
        auto gather = [&](G (&gz)[CT], G (&gx)[KT], int s) __attribute__((always_inline)) {
            const int q = wave * 64 + s * KS + half * EPC;
            const unsigned row = (unsigned)(ch * 256 + q);
            const int4* e = reinterpret_cast<const int4*>(&px[b][q]);
#pragma unroll
            for (int i = 0; i < EPC; i += 2) {
                const int4 v = e[i >> 1];
#pragma unroll
                for (int k = 0; k < KT; ++k) {
                    gx[k].load(i, rx, ((unsigned)v.y & (unsigned)ke[k].y) == (unsigned)ke[k].y ? (unsigned)(v.x + ke[k].x) * ES : OOB);
                    gx[k].load(i + 1, rx, ((unsigned)v.w & (unsigned)ke[k].y) == (unsigned)ke[k].y ? (unsigned)(v.z + ke[k].x) * ES : OOB);
                }
#pragma unroll
                for (int c = 0; c < CT; ++c) {       // (rows past the last one lie past the buffer's end)
                    gz[c].load(i, rz, ce[c] == OOB ? OOB : ((row + i) * (unsigned)p.N + ce[c]) * ES);
                    gz[c].load(i + 1, rz, ce[c] == OOB ? OOB : ((row + i + 1) * (unsigned)p.N + ce[c]) * ES);
                }
            }
        };
        constexpr int STEPS = 64 / KS;
        G gz[2][CT], gx[2][KT];
        gather(gz[0], gx[0], 0);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            if (s + 1 < STEPS) gather(gz[(s + 1) & 1], gx[(s + 1) & 1], s + 1);
            uint4 fz[CT], fx[KT];
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                fz[c] = gz[s & 1][c].pack();
#pragma unroll
                for (int i = 0; i < EPC; ++i) bs[c] += gz[s & 1][c].value(i);
            }
#pragma unroll
            for (int k = 0; k < KT; ++k) fx[k] = gx[s & 1][k].pack();
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int k = 0; k < KT; ++k) mma<E>(acc[c][k], fz[c], fx[k]);
        }
    }
    // wavefronts 2 and 3 hand over to 0 and 1, then 1 to 0
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        bs[c] += __shfl_xor(bs[c], 32);
        if (half == 0) bred[wave][c * 32 + rl] = bs[c];
    }
#pragma unroll
    for (int step = 2; step > 0; step >>= 1) {
        if (wave >= step && wave < 2 * step) {
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int k = 0; k < KT; ++k)
#pragma unroll
                    for (int i = 0; i < 16; ++i) red[wave - step][(c * KT + k) * 1024 + i * 64 + lane] = acc[c][k][i];
        }
        __syncthreads();
        if (wave < step) {
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int k = 0; k < KT; ++k)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[c][k][i] += red[wave][(c * KT + k) * 1024 + i * 64 + lane];
        }
        __syncthreads();
    }
    if (wave) return;
    const int64_t total = (int64_t)p.N * K;
    float* out = a.out + (a.splits > 1 ? (size_t)blockIdx.x * a.part_stride : 0);
    if (a.db && kt == 0 && half == 0) {
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int co = co0 + c * 32 + rl;
            if (co >= p.N) continue;
            const float v = (bred[0][c * 32 + rl] + bred[1][c * 32 + rl]) + (bred[2][c * 32 + rl] + bred[3][c * 32 + rl]);
            if (a.splits > 1) out[total + co] = v;
            else a.db[co] = a.accumulate ? a.db[co] + v : v;
        }
    }
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        const int kk = k0 + k * 32 + rl;
        if (kk >= K) continue;
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int co = co0 + c * 32 + (i >> 2) * 8 + half * 4 + (i & 3);
                if (co >= p.N) continue;
                const size_t o = (size_t)co * K + kk;
                float v = acc[c][k][i];
                if (a.splits == 1 && a.rscale) v *= a.rscale[co];
                if (a.splits == 1 && a.accumulate) v += out[o];
                out[o] = v;
            }
    }
}

// --------------------------------------------------------------------------------------------------
// 31-bit element counts and offsets (a pixel's tap (0,0,0) may lie before the tensor), byte offsets below 4 GiB with the rows
// that a last tile reaches past the end, masks of 7 / 12 / 12 bits
static bool gather_fits(int dtype, const ConvGeom& g) {
    const int64_t es = dtype == LPM_BF16 ? 2 : 4, e31 = (int64_t)1 << 31, lim = ((int64_t)1 << 32) - 1;
    const int64_t halo = (((int64_t)g.Kd * g.H + g.Kh) * g.W + g.Kw) * g.Cin, halo_o = (((int64_t)g.Kd * g.Ho + g.Kh) * g.Wo + g.Kw) * g.Cout;
    return g.Kd < 8 && g.Kh <= 12 && g.Kw <= 12 && g.rows_in() * g.Cin + halo < e31 && (g.rows_out() + 256) * g.Cout + halo_o < e31 &&
           (g.rows_in() * g.Cin + halo) * es < lim && ((g.rows_out() + 256) * g.Cout + halo_o) * es < lim && (int64_t)g.Cout * g.K() < e31;
}
static int gather_steps(int es, int64_t K) { const int ks = 32 / es; return (int)((K + ks - 1) / ks); }
static size_t gather_lds(int es, int nt, int ksteps) {
    const size_t Kp = (size_t)ksteps * (32 / es);
    return Kp * 8 + nt * 32 * (Kp * es + 16) + 4 * 32 * (nt * 32 + 4) * 4;
}
// The bank (with its table and the staging of the epilogue) has to leave room for two blocks per CU; fewer than a few hundred
// rows are a handful of wavefronts, each with the latency of the whole reduction -- the kernels that share an output between lanes
// are faster there.
static bool gather_shape_ok(int dtype, int64_t rows, int N, int64_t K) {
    const int es = dtype == LPM_BF16 ? 2 : 4;
    return rows >= 256 && K <= 1024 && gather_lds(es, N > 32 ? 2 : 1, gather_steps(es, K)) <= 80 * 1024;
}
bool gather_fwd_ok(int dtype, const ConvGeom& g) { return gather_fits(dtype, g) && gather_shape_ok(dtype, g.rows_out(), g.Cout, g.K()); }
bool gather_dgrad_ok(int dtype, const ConvGeom& g) {
    return g.stride == 1 && gather_fits(dtype, g) && gather_shape_ok(dtype, g.rows_in(), g.Cin, (int64_t)g.taps() * g.Cout);
}
bool gather_wgrad_ok(int dtype, const ConvGeom& g) { return gather_fits(dtype, g); }

// whether the forward kernel can also store the 2x2 max-pooling of its output: its rows then go by pooling window, so that a window's
// four are next to each other in a tile (two launches less for LeNet: at 128
// samples a micro-batch 476 -> 455 us per step, at 8 355 -> 344, where two runs differ by 2 %)
bool gather_fwd_pools(const ConvGeom& g) { return !g.is3d() && !(g.Ho & 1) && !(g.Wo & 1); }

static void fill_geom(IgemmArgs& a) {
    a.Di = std::max(a.Di, 1); a.Dr = std::max(a.Dr, 1); a.Kd = std::max(a.Kd, 1);
    a.dWr = fast_div(a.Wr); a.dHr = fast_div(a.Hr); a.dDr = fast_div(a.Dr); a.dCc = fast_div(a.Ci);
    a.dKhw = fast_div(a.Kh * a.Kw); a.dKw = fast_div(a.Kw);
}

template <typename E, int NT, int MODE, bool KSPLIT>
static hipError_t go(const IgemmArgs& a, int ksteps, int tiles, hipStream_t st) {
    static DeviceSet done;
    const hipError_t attr = allow_lds(gather_gemm<E, NT, MODE, KSPLIT>, 80 * 1024, done);
    if (attr != hipSuccess) return attr;
    const int blocks = KSPLIT ? tiles : std::min((tiles + 3) / 4, 1536);
    launch_last(gather_gemm<E, NT, MODE, KSPLIT>, dim3((unsigned)blocks, (unsigned)((a.N + NT * 32 - 1) / (NT * 32))), dim3(256),
                       gather_lds(sizeof(E), NT, ksteps), st, a, ksteps, tiles, fast_div(ksteps * (32 / (int)sizeof(E))), fast_div(std::min(a.N, NT * 32)));
    return hipGetLastError();
}
template <typename E, int NT, int MODE>
static hipError_t go(const IgemmArgs& a, hipStream_t st) {
    const int ksteps = gather_steps(sizeof(E), (int64_t)a.Kd * a.Kh * a.Kw * a.Ci), tiles = (a.M + 31) / 32;
    if (tiles <= 256 && ksteps >= 4) return go<E, NT, MODE, true>(a, ksteps, tiles, st);       // less than a block per CU
    return go<E, NT, MODE, false>(a, ksteps, tiles, st);
}
template <int MODE>
static hipError_t run(int dtype, IgemmArgs& a, hipStream_t st) {
    fill_geom(a);
    if (MODE == MODE_FWD_POOL) { a.dWr = fast_div(a.Wr / 2); a.dHr = fast_div(a.Hr / 2); }
    if (dtype == LPM_BF16) return a.N > 32 ? go<bf16_t, 2, MODE>(a, st) : go<bf16_t, 1, MODE>(a, st);
    return a.N > 32 ? go<float, 2, MODE>(a, st) : go<float, 1, MODE>(a, st);
}

hipError_t gather_conv_fwd(int dtype, const ConvGeom& g, const void* x, const void* w, const float* scale, const float* bias,
                           const void* add, int relu, void* y, hipStream_t st, void* pool_y) {
    if (pool_y && (add || !gather_fwd_pools(g))) return hipErrorInvalidValue;
    IgemmArgs a{};
    a.A = x; a.B = w; a.C = y;
    a.scale = scale; a.bias = bias; a.add = add; a.relu = relu;
    a.M = (int)g.rows_out(); a.N = g.Cout;
    a.Hi = g.H; a.Wi = g.W; a.Di = g.D; a.Ci = g.Cin; a.Hr = g.Ho; a.Wr = g.Wo; a.Dr = g.Do;
    a.Kh = g.Kh; a.Kw = g.Kw; a.Kd = g.Kd; a.stride = g.stride; a.pad = g.pad; a.pad_d = g.pad_d;
    a.a_bytes = (unsigned)(g.rows_in() * g.Cin * (dtype == LPM_BF16 ? 2 : 4));
    if (pool_y) {
        a.fwd_pool = (uint16_t*)pool_y;
        return run<MODE_FWD_POOL>(dtype, a, st);
    }
    return run<MODE_FWD>(dtype, a, st);
}

// w: [Cout][taps][Cin] as it lies; dzscale (may be NULL) multiplies channel co of dz
hipError_t gather_conv_dgrad(int dtype, const ConvGeom& g, const void* dz, const float* dzscale, const void* w, void* dx, int accumulate,
                             const void* mask, const float* mscale, hipStream_t st) {
    IgemmArgs a{};
    a.A = dz; a.B = w; a.C = dx;
    a.add = accumulate ? dx : nullptr; a.mask = mask; a.mscale = mscale; a.kscale = dzscale;
    a.M = (int)g.rows_in(); a.N = g.Cin;
    a.Hi = g.Ho; a.Wi = g.Wo; a.Di = g.Do; a.Ci = g.Cout; a.Hr = g.H; a.Wr = g.W; a.Dr = g.D;
    a.Kh = g.Kh; a.Kw = g.Kw; a.Kd = g.Kd; a.stride = 1; a.pad = g.pad; a.pad_d = g.pad_d;
    a.a_bytes = (unsigned)(g.rows_out() * g.Cout * (dtype == LPM_BF16 ? 2 : 4));
    return run<MODE_DGRAD>(dtype, a, st);
}

struct GwPlan { int ct, kt, co_tiles, k_tiles, chunks, per, splits; };
static GwPlan plan_gather_wgrad(const ConvGeom& g) {
    GwPlan pl{};
    pl.ct = g.Cout > 32 ? 2 : 1;
    pl.kt = g.K() > 32 ? 2 : 1;
    pl.co_tiles = (g.Cout + pl.ct * 32 - 1) / (pl.ct * 32);
    pl.k_tiles = (int)((g.K() + pl.kt * 32 - 1) / (pl.kt * 32));
    pl.chunks = (int)((g.rows_out() + 255) / 256);
    // two blocks per CU to hide the loads' latency; every pixel range costs a pass over dW in the reduction
    const int64_t base = (int64_t)pl.co_tiles * pl.k_tiles, out_bytes = ((int64_t)g.Cout * g.K() + g.Cout) * 4;
    int64_t sp = std::min<int64_t>(pl.chunks, std::max<int64_t>(1, 512 / base));
    sp = std::min<int64_t>(sp, std::max<int64_t>(1, (64ll << 20) / out_bytes));
    pl.per = (int)((pl.chunks + sp - 1) / sp);
    pl.splits = (pl.chunks + pl.per - 1) / pl.per;
    return pl;
}
static size_t gw_stride(const ConvGeom& g) { return ((size_t)g.Cout * g.K() + g.Cout + 3) & ~(size_t)3; }
size_t gather_wgrad_ws_bytes(const ConvGeom& g) {
    const GwPlan pl = plan_gather_wgrad(g);
    return pl.splits > 1 ? (size_t)pl.splits * gw_stride(g) * sizeof(float) : 0;
}

template <typename E>
static void launch_gw(const GwPlan& pl, const GwArgs& a, hipStream_t st) {
    const dim3 grid((unsigned)pl.splits, (unsigned)(pl.co_tiles * pl.k_tiles));
    if (pl.ct == 2 && pl.kt == 2) hipLaunchKernelGGL((gather_wgrad<E, 2, 2>), grid, dim3(256), 0, st, a);
    else if (pl.ct == 2) hipLaunchKernelGGL((gather_wgrad<E, 2, 1>), grid, dim3(256), 0, st, a);
    else if (pl.kt == 2) hipLaunchKernelGGL((gather_wgrad<E, 1, 2>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((gather_wgrad<E, 1, 1>), grid, dim3(256), 0, st, a);
}

hipError_t gather_conv_wgrad(int dtype, const ConvGeom& g, const void* x, const void* dz, float* dw, float* dbias, const float* rscale,
                             int accumulate, void* ws, hipStream_t st, ReduceDesc* deferred) {
    const int es = dtype == LPM_BF16 ? 2 : 4;
    const GwPlan pl = plan_gather_wgrad(g);
    GwArgs a{};
    IgemmArgs& p = a.p;
    p.A = x;
    p.M = (int)g.rows_out(); p.N = g.Cout;
    p.Hi = g.H; p.Wi = g.W; p.Di = g.D; p.Ci = g.Cin; p.Hr = g.Ho; p.Wr = g.Wo; p.Dr = g.Do;
    p.Kh = g.Kh; p.Kw = g.Kw; p.Kd = g.Kd; p.stride = g.stride; p.pad = g.pad; p.pad_d = g.pad_d;
    p.a_bytes = (unsigned)(g.rows_in() * g.Cin * es);
    fill_geom(p);
    a.DZ = dz; a.dz_bytes = (unsigned)(g.rows_out() * g.Cout * es);
    a.out = pl.splits > 1 ? (float*)ws : dw;
    a.db = dbias; a.rscale = rscale; a.part_stride = gw_stride(g);
    a.chunks = pl.chunks; a.per_split = pl.per; a.splits = pl.splits; a.k_tiles = pl.k_tiles; a.accumulate = accumulate;
    if (dtype == LPM_BF16) launch_gw<bf16_t>(pl, a, st); else launch_gw<float>(pl, a, st);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || pl.splits == 1) return e;
    const int64_t n = (int64_t)g.Cout * g.K();
    const ReduceDesc d{(const float*)ws, a.part_stride, pl.splits, dw, n, dbias, dbias ? g.Cout : 0, rscale, (int)g.K(), accumulate};
    if (deferred) { *deferred = d; return hipSuccess; }
    return launch_reduce_batch(&d, 1, st);
}

}  // namespace lpm
