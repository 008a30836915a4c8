// One-head self-attention over the positions of a sample -- the "self-attention layer" of the residual self-attention
// block in the method's first use case (3D-ResAttNet), read as scaled dot-product attention:
//   x [m][P][3C] holds queries | keys | values per position (made by the 1x1 convolution in front of the layer)
//   S[i][j] = q_i . k_j / sqrt(C);   A = softmax over j;   y_i = sum_j A[i][j] v_j                    (forward, eq. 1)
//   dv_j = sum_i A[i][j] dy_i;  dA[i][j] = dy_i . v_j;  dS = A (dA - rowsum(A dA));
//   dq_i = sum_j dS[i][j] k_j / sqrt(C);  dk_j = sum_i dS[i][j] q_i / sqrt(C)                        (backward, eq. 9)
// Sizes here are small (P up to a few hundred positions after the last down-sampling stage, C up to a few hundred
// channels: well under a GFLOP per sample).  bf16 layers of whole 8-channel chunks run on the matrix cores, 16 queries (keys)
// per block; float layers and other channel counts on the vector ALU, with the row being worked on in LDS.  No atomics: the
// order of every sum is fixed, so results do not depend on scheduling.  The backward pass recomputes the scores (nothing
// but the layer input is kept from the forward pass) in two kernels: one per block of queries (dq, and the row statistics
// max, sum, rowsum(A dA)), one per block of keys (dk, dv), which needs those statistics.
#include "lpm_internal.h"
#include "elem.h"

namespace lpm {

constexpr int ATT_QB = 8;        // queries (keys) per block
constexpr int ATT_LIMIT = 1000;  // C + P: the key-block kernel keeps 8 x (2C + 2P) floats in LDS (under 64 KiB)

bool attn_ok(int32_t P, int32_t C) { return P > 0 && C > 0 && P + C <= ATT_LIMIT; }
size_t attn_bwd_ws_bytes(int32_t m, int32_t P) { return (size_t)m * P * 3 * sizeof(float); }

__device__ inline float att_wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ inline float att_wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// eight consecutive elements of a row (the caller has checked that rows start at multiples of eight elements)
__device__ __forceinline__ void att_ld8(const float* p, float (&v)[8]) {
    const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void att_ld8(const bf16_t* p, float (&v)[8]) {
    const uint4 w = *reinterpret_cast<const uint4*>(p);
    const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) { v[2 * k] = bf2f((uint16_t)(ww[k] & 0xffffu)); v[2 * k + 1] = bf2f((uint16_t)(ww[k] >> 16)); }
}

// acc[i] += sum_c row[c] * mat[i][c] for the ATT_QB rows of mat (LDS, [ATT_QB][C]); the row is read 8 channels at a
// time where C allows (a thread walking its row two bytes at a time was the slowest part of these kernels)
template <typename T>
__device__ __forceinline__ void att_row_dots(const T* __restrict__ row, int C, const float* mat, float (&acc)[ATT_QB]) {
    int c = 0;
    if ((C & 7) == 0) {
        for (; c < C; c += 8) {
            float v[8];
            att_ld8(row + c, v);
#pragma unroll
            for (int i = 0; i < ATT_QB; ++i) {
                const float4 m0 = *reinterpret_cast<const float4*>(mat + i * C + c), m1 = *reinterpret_cast<const float4*>(mat + i * C + c + 4);
                acc[i] = fmaf(v[0], m0.x, acc[i]); acc[i] = fmaf(v[1], m0.y, acc[i]); acc[i] = fmaf(v[2], m0.z, acc[i]); acc[i] = fmaf(v[3], m0.w, acc[i]);
                acc[i] = fmaf(v[4], m1.x, acc[i]); acc[i] = fmaf(v[5], m1.y, acc[i]); acc[i] = fmaf(v[6], m1.z, acc[i]); acc[i] = fmaf(v[7], m1.w, acc[i]);
            }
        }
        return;
    }
    for (; c < C; ++c) {
        const float v = ld(row, c);
#pragma unroll
        for (int i = 0; i < ATT_QB; ++i) acc[i] = fmaf(v, mat[i * C + c], acc[i]);
    }
}

// The per-block score tiles live in LDS position-major: tile[j * ATT_QB + i] for position j and the block's row i, so the
// eight values of one position are one 32-byte read.

// scores of the block's queries against every key, into sc[P][QB]; qs[QB][C] holds the queries times 1/sqrt(C)
template <typename T>
__device__ __forceinline__ void att_scores(const T* __restrict__ xs, int P, int C, const float* qs, float* sc) {
    for (int j = threadIdx.x; j < P; j += blockDim.x) {
        float acc[ATT_QB];
#pragma unroll
        for (int i = 0; i < ATT_QB; ++i) acc[i] = 0.f;
        att_row_dots(xs + (int64_t)j * 3 * C + C, C, qs, acc);
#pragma unroll
        for (int i = 0; i < ATT_QB; ++i) sc[j * ATT_QB + i] = acc[i];
    }
}

// per query row of the block: maximum and sum of exp (one wavefront per row at a time); sc becomes the softmax
__device__ __forceinline__ void att_softmax_rows(int P, int nq, float* sc, float* rmax, float* rsum) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    for (int i = wave; i < nq; i += nw) {
        float mx = -INFINITY;
        for (int j = lane; j < P; j += 64) mx = fmaxf(mx, sc[j * ATT_QB + i]);
        mx = att_wave_max(mx);
        float se = 0.f;
        for (int j = lane; j < P; j += 64) { const float e = expf(sc[j * ATT_QB + i] - mx); sc[j * ATT_QB + i] = e; se += e; }
        se = att_wave_sum(se);
        const float inv = 1.f / se;
        for (int j = lane; j < P; j += 64) sc[j * ATT_QB + i] *= inv;
        if (lane == 0) { rmax[i] = mx; rsum[i] = se; }
    }
}

// out[i][c] = sum_j tile[j][i] * rows[j][c] over all positions j, for the block's rows i < n_rows and all channels c:
// a thread owns a channel and ATT_QB / NP of the rows (NP parts of the block share a channel when C is small), so one
// element of rows[j] feeds that many multiply-adds.  f(i, c, value) stores.
template <int NP, typename T, typename F>
__device__ __forceinline__ void att_mix(const float* tile, const T* __restrict__ rows, int64_t row_stride, int P, int C, int n_rows, F&& f) {
    constexpr int QPP = ATT_QB / NP;
    const int cols = blockDim.x / NP, part = threadIdx.x / cols, i0 = part * QPP;
    for (int c = threadIdx.x - part * cols; c < C; c += cols) {
        float acc[QPP];
#pragma unroll
        for (int i = 0; i < QPP; ++i) acc[i] = 0.f;
        // Sixteen positions per trip, their loads issued together before the first is used: one memory latency per sixteen
        // positions (left to itself the compiler keeps four loads in flight; asked to unroll further it chains the
        // 2-byte loads through one register and waits for each).
        int j = 0;
        for (; j + 16 <= P; j += 16) {
            T raw[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) raw[k] = rows[(int64_t)(j + k) * row_stride + c];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const float v = ld(raw, k);
#pragma unroll
                for (int i = 0; i < QPP; ++i) acc[i] = fmaf(tile[(j + k) * ATT_QB + i0 + i], v, acc[i]);
            }
        }
        for (; j < P; ++j) {
            const float v = ld(rows, (int64_t)j * row_stride + c);
#pragma unroll
            for (int i = 0; i < QPP; ++i) acc[i] = fmaf(tile[j * ATT_QB + i0 + i], v, acc[i]);
        }
#pragma unroll
        for (int i = 0; i < QPP; ++i) if (i0 + i < n_rows) f(i0 + i, c, acc[i]);
    }
}

template <typename T, int NP>
__global__ void __launch_bounds__(256) attn_fwd_kernel(int P, int C, const T* __restrict__ x, T* __restrict__ y) {
    extern __shared__ __attribute__((aligned(16))) float lds[];
    float* qs = lds;                    // [QB][C]
    float* sc = lds + ATT_QB * C;       // [P][QB]
    __shared__ float rmax[ATT_QB], rsum[ATT_QB];
    const int n = blockIdx.y, i0 = blockIdx.x * ATT_QB, nq = min(ATT_QB, P - i0);
    const T* xs = x + (int64_t)n * P * 3 * C;
    const float scale = rsqrtf((float)C);
    for (int e = threadIdx.x; e < ATT_QB * C; e += blockDim.x) {
        const int i = e / C, c = e - i * C;
        qs[e] = i < nq ? ld(xs, (int64_t)(i0 + i) * 3 * C + c) * scale : 0.f;
    }
    __syncthreads();
    att_scores(xs, P, C, qs, sc);
    __syncthreads();
    att_softmax_rows(P, nq, sc, rmax, rsum);
    __syncthreads();
    att_mix<NP>(sc, xs + 2 * C, 3 * C, P, C, nq, [&](int i, int c, float v) { st(y, ((int64_t)n * P + i0 + i) * C + c, v); });
}

// per block of queries: dq, and per query row (max, sum of exp, sum_j A dA) into stats [m][P][3]
template <typename T, int NP>
__global__ void __launch_bounds__(256) attn_bwd_q_kernel(int P, int C, const T* __restrict__ x, const T* __restrict__ dy,
                                                         T* __restrict__ dx, int accumulate, float* __restrict__ stats) {
    extern __shared__ __attribute__((aligned(16))) float lds[];
    float* qs = lds;                           // [QB][C] queries / sqrt(C)
    float* gs = qs + ATT_QB * C;               // [QB][C] dy rows
    float* sc = gs + ATT_QB * C;               // [P][QB] A, then dS
    float* da = sc + ATT_QB * P;               // [P][QB] dA
    __shared__ float rmax[ATT_QB], rsum[ATT_QB];
    const int n = blockIdx.y, i0 = blockIdx.x * ATT_QB, nq = min(ATT_QB, P - i0);
    const T* xs = x + (int64_t)n * P * 3 * C;
    const T* gy = dy + (int64_t)n * P * C;
    const float scale = rsqrtf((float)C);
    for (int e = threadIdx.x; e < ATT_QB * C; e += blockDim.x) {
        const int i = e / C, c = e - i * C;
        qs[e] = i < nq ? ld(xs, (int64_t)(i0 + i) * 3 * C + c) * scale : 0.f;
        gs[e] = i < nq ? ld(gy, (int64_t)(i0 + i) * C + c) : 0.f;
    }
    __syncthreads();
    att_scores(xs, P, C, qs, sc);
    // dA[i][j] = dy_i . v_j
    for (int j = threadIdx.x; j < P; j += blockDim.x) {
        float acc[ATT_QB];
#pragma unroll
        for (int i = 0; i < ATT_QB; ++i) acc[i] = 0.f;
        att_row_dots(xs + (int64_t)j * 3 * C + 2 * C, C, gs, acc);
#pragma unroll
        for (int i = 0; i < ATT_QB; ++i) da[j * ATT_QB + i] = acc[i];
    }
    __syncthreads();
    att_softmax_rows(P, nq, sc, rmax, rsum);
    __syncthreads();
    {   // rowsum(A dA), then dS = A (dA - rowsum) in place of A
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
        for (int i = wave; i < nq; i += nw) {
            float r = 0.f;
            for (int j = lane; j < P; j += 64) r = fmaf(sc[j * ATT_QB + i], da[j * ATT_QB + i], r);
            r = att_wave_sum(r);
            for (int j = lane; j < P; j += 64) sc[j * ATT_QB + i] *= (da[j * ATT_QB + i] - r);
            if (lane == 0) {
                float* s3 = stats + ((int64_t)n * P + i0 + i) * 3;
                s3[0] = rmax[i]; s3[1] = rsum[i]; s3[2] = r;
            }
        }
    }
    __syncthreads();
    att_mix<NP>(sc, xs + C, 3 * C, P, C, nq, [&](int i, int c, float v) {
        const int64_t o = ((int64_t)n * P + i0 + i) * 3 * C + c;
        v *= scale;
        st(dx, o, accumulate ? v + ld(dx, o) : v);
    });
}

// per block of keys: dk and dv
template <typename T, int NP>
__global__ void __launch_bounds__(256) attn_bwd_kv_kernel(int P, int C, const T* __restrict__ x, const T* __restrict__ dy,
                                                          T* __restrict__ dx, int accumulate, const float* __restrict__ stats) {
    extern __shared__ __attribute__((aligned(16))) float lds[];
    float* ks = lds;                           // [QB][C] keys / sqrt(C)
    float* vs = ks + ATT_QB * C;               // [QB][C] values
    float* aa = vs + ATT_QB * C;               // [P][QB] A[i][j] for the block's keys j, all queries i
    float* ds = aa + ATT_QB * P;               // [P][QB] dS[i][j]
    const int n = blockIdx.y, j0 = blockIdx.x * ATT_QB, nk = min(ATT_QB, P - j0);
    const T* xs = x + (int64_t)n * P * 3 * C;
    const T* gy = dy + (int64_t)n * P * C;
    const float scale = rsqrtf((float)C);
    for (int e = threadIdx.x; e < ATT_QB * C; e += blockDim.x) {
        const int j = e / C, c = e - j * C;
        ks[e] = j < nk ? ld(xs, (int64_t)(j0 + j) * 3 * C + C + c) * scale : 0.f;
        vs[e] = j < nk ? ld(xs, (int64_t)(j0 + j) * 3 * C + 2 * C + c) : 0.f;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < P; i += blockDim.x) {
        float s[ATT_QB], d[ATT_QB];
#pragma unroll
        for (int j = 0; j < ATT_QB; ++j) { s[j] = 0.f; d[j] = 0.f; }
        att_row_dots(xs + (int64_t)i * 3 * C, C, ks, s);
        att_row_dots(gy + (int64_t)i * C, C, vs, d);
        const float* s3 = stats + ((int64_t)n * P + i) * 3;
        const float mx = s3[0], inv = 1.f / s3[1], r = s3[2];
#pragma unroll
        for (int j = 0; j < ATT_QB; ++j) {
            const float a = expf(s[j] - mx) * inv;
            aa[i * ATT_QB + j] = a;
            ds[i * ATT_QB + j] = a * (d[j] - r);
        }
    }
    __syncthreads();
    att_mix<NP>(aa, gy, C, P, C, nk, [&](int j, int c, float v) {
        const int64_t o = ((int64_t)n * P + j0 + j) * 3 * C + 2 * C + c;
        st(dx, o, accumulate ? v + ld(dx, o) : v);
    });
    att_mix<NP>(ds, xs, 3 * C, P, C, nk, [&](int j, int c, float v) {
        const int64_t o = ((int64_t)n * P + j0 + j) * 3 * C + C + c;
        v *= scale;
        st(dx, o, accumulate ? v + ld(dx, o) : v);
    });
}

// ---- matrix cores --------------------------------------------------------------------------------
// A block of eight wavefronts takes 16 rows (queries; keys in the kernel that makes dk and dv).  Scores against all positions
// and dA are products of bf16 rows that lie channel-contiguous in memory: the block's rows from LDS, the others straight from
// memory, fp32 accumulation, the result in LDS (16 x P floats).  The sums over positions (A V, dS K, A' dy, dS' q) read that
// fp32 tile as their first operand: split into three bf16 terms, which carry all 24 bits of it, so its precision is what it
// was on the vector ALU.  The other operand has the position as its reduction index, outermost in memory: a lane loads two
// neighbouring channels of eight positions and sorts them into an operand of even and one of odd channels -- a lane then
// ends with eight consecutive channels of a row.
// What bounds them is one pass over K and V per block at the rate a CU loads (and for small P the chain of the phases).
// 2 samples, P = 512, C = 128 (us): forward 45 -> 19, backward 60 + 92 -> 26 + 25; P = 64, C = 256: 38 + 48 -> 13 + 13 backward.
constexpr int AM_T = 512, AM_W = 8, AM_R = 16;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct AmShape {
    int P, C, Pp, Cp, tp, rp;       // positions, channels, rounded up to 32 and 128; LDS pitches of a score tile (floats) and of the staged rows (elements)
    __host__ __device__ AmShape(int P_, int C_) : P(P_), C(C_), Pp((P_ + 31) & ~31), Cp((C_ + 127) & ~127), tp(Pp + 4), rp(Cp + 8) {}
    __host__ __device__ size_t tile_bytes() const { return (size_t)AM_R * tp * 4; }
    __host__ __device__ size_t rows_bytes() const { return (size_t)AM_R * rp * 2; }
};
constexpr size_t AM_RED = AM_W * 64 * 8 * 4;      // partial sums of am_mix

// the block's 16 rows into LDS, zeros past the last one
__device__ __forceinline__ void am_stage(const AmShape& s, uint16_t* dst, const bf16_t* src, int64_t stride, int row0) {
    const int per = s.Cp >> 3;
    for (int i = threadIdx.x; i < AM_R * per; i += AM_T) {
        const int r = i / per, c = (i - r * per) * 8;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (row0 + r < s.P && c < s.C) v = *reinterpret_cast<const uint4*>(src + (row0 + r) * stride + c);
        *reinterpret_cast<uint4*>(dst + r * s.rp + c) = v;
    }
}

// tile[r][j] = mul * sum_c rows[r][c] * mat[j][c] for every position j (columns past the last one hold finite values)
__device__ __forceinline__ void am_products(const AmShape& s, const uint16_t* rows, const bf16_t* mat, int64_t stride, float mul, float* tile) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l = lane & 15, g = lane >> 4;
    const int groups = s.Cp >> 7, tiles = s.Pp >> 4, n = wave < tiles ? (tiles - wave + AM_W - 1) / AM_W * groups : 0;
    // items: 128 channels of 16 positions; the next item's loads are in flight while one is multiplied
    uint4 v[4], nx[4];
    int lj = wave * 16, lc = g * 8;
    auto load = [&]() __attribute__((always_inline)) {
        const bf16_t* b = mat + (int64_t)min(lj + l, s.P - 1) * stride;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            nx[u] = make_uint4(0, 0, 0, 0);
            if (lc + u * 32 < s.C) nx[u] = *reinterpret_cast<const uint4*>(b + lc + u * 32);
        }
        lc += 128;
        if (lc >= s.Cp) { lc = g * 8; lj += AM_W * 16; }
    };
    if (n > 0) load();
    int j0 = wave * 16, c = 0;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int it = 0; it < n; ++it) {
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = nx[u];
        if (it + 1 < n) load();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint4 a = *reinterpret_cast<const uint4*>(rows + l * s.rp + c + u * 32 + g * 8);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v[u]), __builtin_bit_cast(bf16x8, a), acc, 0, 0, 0);
        }
        c += 128;
        if (c == s.Cp) {
            *reinterpret_cast<float4*>(tile + l * s.tp + j0 + g * 4) = make_float4(acc[0] * mul, acc[1] * mul, acc[2] * mul, acc[3] * mul);
            acc = f32x4{0.f, 0.f, 0.f, 0.f};
            c = 0;
            j0 += AM_W * 16;
        }
    }
}

// softmax of the tile's rows in place, zeros in the columns past the last position; f(row, max, sum) on one lane per row
template <typename F>
__device__ __forceinline__ void am_softmax(const AmShape& s, float* tile, F&& f) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int r = wave; r < AM_R; r += AM_W) {
        float* t = tile + r * s.tp;
        float mx = -INFINITY;
        for (int j = lane; j < s.P; j += 64) mx = fmaxf(mx, t[j]);
        mx = att_wave_max(mx);
        float se = 0.f;
        for (int j = lane; j < s.P; j += 64) { const float e = expf(t[j] - mx); t[j] = e; se += e; }
        se = att_wave_sum(se);
        const float inv = 1.f / se;
        for (int j = lane; j < s.Pp; j += 64) t[j] = j < s.P ? t[j] * inv : 0.f;
        if (lane == 0) f(r, mx, se);
    }
}

// f(r, c, v): v[8] = sum over positions j of tile[r][j] * mat[j][c .. c + 7], r < 16, c = 0, 8, .. < C.  A unit of work is 32
// channels over a range of positions, one per wavefront where there are few channels (the ranges' sums meet in red).
template <typename F>
__device__ __forceinline__ void am_mix(const AmShape& s, const float* tile, const bf16_t* mat, int64_t stride, float* red, F&& f) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l = lane & 15, g = lane >> 4;
    const int nc = (s.C + 31) >> 5, parts = nc <= AM_W ? AM_W / nc : 1, steps = s.Pp >> 5, per = (steps + parts - 1) / parts;
    for (int u = wave; u < nc * parts || (parts > 1 && u < AM_W); u += AM_W) {
        const int cg = u % nc, part = u / nc;
        const bool work = part < parts;
        f32x4 even = {0.f, 0.f, 0.f, 0.f}, odd = {0.f, 0.f, 0.f, 0.f};
        const bf16_t* b = mat + min(cg * 32 + 2 * l, s.C - 2);
        const int k1 = work ? min(steps, (part + 1) * per) : 0;
        unsigned w[8], nw[8];
        auto load = [&](int k) __attribute__((always_inline)) {
            const int j = k * 32 + g * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e) nw[e] = *reinterpret_cast<const unsigned*>(b + (int64_t)min(j + e, s.P - 1) * stride);
#pragma unroll
            for (int e = 0; e < 8; ++e) if (j + e >= s.P) nw[e] = 0u;
        };
        if (part * per < k1) load(part * per);
        for (int k = part * per; k < k1; ++k) {
            const int j0 = k * 32 + g * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e) w[e] = nw[e];
            if (k + 1 < k1) load(k + 1);
            const float4 lo = *reinterpret_cast<const float4*>(tile + l * s.tp + j0), hi = *reinterpret_cast<const float4*>(tile + l * s.tp + j0 + 4);
            float x[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
            unsigned ev[4], od[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                ev[e] = __builtin_amdgcn_perm(w[2 * e + 1], w[2 * e], 0x05040100u);
                od[e] = __builtin_amdgcn_perm(w[2 * e + 1], w[2 * e], 0x07060302u);
            }
            const bf16x8 ve = __builtin_bit_cast(bf16x8, make_uint4(ev[0], ev[1], ev[2], ev[3])), vo = __builtin_bit_cast(bf16x8, make_uint4(od[0], od[1], od[2], od[3]));
#pragma unroll
            for (int term = 0; term < 3; ++term) {      // x = three bf16 terms; the remainders are exact
                unsigned q[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    q[e] = pack_bf16x2(x[2 * e], x[2 * e + 1]);
                    x[2 * e] -= __uint_as_float(q[e] << 16);
                    x[2 * e + 1] -= __uint_as_float(q[e] & 0xffff0000u);
                }
                const bf16x8 vx = __builtin_bit_cast(bf16x8, make_uint4(q[0], q[1], q[2], q[3]));
                even = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ve, vx, even, 0, 0, 0);
                odd = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vo, vx, odd, 0, 0, 0);
            }
        }
        float v[8] = {even[0], odd[0], even[1], odd[1], even[2], odd[2], even[3], odd[3]};
        if (parts > 1) {                   // (u < AM_W: every wavefront is here once)
            __syncthreads();               // (the sums of an earlier call have been read)
#pragma unroll
            for (int e = 0; e < 8; ++e) red[(u * 8 + e) * 64 + lane] = v[e];
            __syncthreads();
            if (part) continue;
            for (int q = 1; q < parts; ++q)
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] += red[((u + q * nc) * 8 + e) * 64 + lane];
        }
        const int c = cg * 32 + g * 8;
        if (c < s.C) f(l, c, v);
    }
}

__device__ __forceinline__ void am_store8(bf16_t* o, float (&v)[8], int accumulate) {
    if (accumulate) {
        float t[8];
        att_ld8(o, t);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += t[e];
    }
    *reinterpret_cast<uint4*>(o) = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
}

__global__ void __launch_bounds__(AM_T) attn_fwd_mm(int P, int C, const bf16_t* __restrict__ x, bf16_t* __restrict__ y) {
    extern __shared__ __attribute__((aligned(16))) unsigned char am_lds[];
    const AmShape s(P, C);
    float* tile = reinterpret_cast<float*>(am_lds);
    float* red = reinterpret_cast<float*>(am_lds + s.tile_bytes());
    uint16_t* rows = reinterpret_cast<uint16_t*>(am_lds + s.tile_bytes() + AM_RED);
    const int n = blockIdx.y, i0 = blockIdx.x * AM_R;
    const bf16_t* xs = x + (int64_t)n * P * 3 * C;
    am_stage(s, rows, xs, 3 * C, i0);
    __syncthreads();
    am_products(s, rows, xs + C, 3 * C, rsqrtf((float)C), tile);
    __syncthreads();
    am_softmax(s, tile, [](int, float, float) {});
    __syncthreads();
    am_mix(s, tile, xs + 2 * C, 3 * C, red, [&](int r, int c, float (&v)[8]) {
        if (i0 + r < P) am_store8(y + ((int64_t)n * P + i0 + r) * C + c, v, 0);
    });
}

__global__ void __launch_bounds__(AM_T) attn_bwd_q_mm(int P, int C, const bf16_t* __restrict__ x, const bf16_t* __restrict__ dy,
                                                      bf16_t* __restrict__ dx, int accumulate, float* __restrict__ stats) {
    extern __shared__ __attribute__((aligned(16))) unsigned char am_lds[];
    const AmShape s(P, C);
    float* sc = reinterpret_cast<float*>(am_lds);
    float* da = reinterpret_cast<float*>(am_lds + s.tile_bytes());
    float* red = reinterpret_cast<float*>(am_lds + 2 * s.tile_bytes());
    uint16_t* qs = reinterpret_cast<uint16_t*>(am_lds + 2 * s.tile_bytes() + AM_RED);
    uint16_t* gs = qs + AM_R * s.rp;
    __shared__ float rmax[AM_R], rsum[AM_R];
    const int n = blockIdx.y, i0 = blockIdx.x * AM_R;
    const bf16_t* xs = x + (int64_t)n * P * 3 * C;
    const bf16_t* gy = dy + (int64_t)n * P * C;
    const float scale = rsqrtf((float)C);
    am_stage(s, qs, xs, 3 * C, i0);
    am_stage(s, gs, gy, C, i0);
    __syncthreads();
    am_products(s, qs, xs + C, 3 * C, scale, sc);
    am_products(s, gs, xs + 2 * C, 3 * C, 1.f, da);
    __syncthreads();
    am_softmax(s, sc, [&](int r, float mx, float se) { rmax[r] = mx; rsum[r] = se; });
    // rowsum(A dA), then dS = A (dA - rowsum) in place of A (a wavefront's own rows: no barrier in between)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = wave; i < AM_R; i += AM_W) {
        float* t = sc + i * s.tp;
        const float* d = da + i * s.tp;
        float r = 0.f;
        for (int j = lane; j < P; j += 64) r = fmaf(t[j], d[j], r);
        r = att_wave_sum(r);
        for (int j = lane; j < P; j += 64) t[j] *= d[j] - r;
        if (lane == 0 && i0 + i < P) {
            float* s3 = stats + ((int64_t)n * P + i0 + i) * 3;
            s3[0] = rmax[i]; s3[1] = rsum[i]; s3[2] = r;
        }
    }
    __syncthreads();
    am_mix(s, sc, xs + C, 3 * C, red, [&](int r, int c, float (&v)[8]) {
        if (i0 + r >= P) return;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] *= scale;
        am_store8(dx + ((int64_t)n * P + i0 + r) * 3 * C + c, v, accumulate);
    });
}

__global__ void __launch_bounds__(AM_T) attn_bwd_kv_mm(int P, int C, const bf16_t* __restrict__ x, const bf16_t* __restrict__ dy,
                                                       bf16_t* __restrict__ dx, int accumulate, const float* __restrict__ stats) {
    extern __shared__ __attribute__((aligned(16))) unsigned char am_lds[];
    const AmShape s(P, C);
    float* aa = reinterpret_cast<float*>(am_lds);                          // [key][query] A
    float* ds = reinterpret_cast<float*>(am_lds + s.tile_bytes());         // dS
    float* red = reinterpret_cast<float*>(am_lds + 2 * s.tile_bytes());
    uint16_t* ks = reinterpret_cast<uint16_t*>(am_lds + 2 * s.tile_bytes() + AM_RED);
    uint16_t* vs = ks + AM_R * s.rp;
    const int n = blockIdx.y, j0 = blockIdx.x * AM_R;
    const bf16_t* xs = x + (int64_t)n * P * 3 * C;
    const bf16_t* gy = dy + (int64_t)n * P * C;
    const float scale = rsqrtf((float)C);
    am_stage(s, ks, xs + C, 3 * C, j0);
    am_stage(s, vs, xs + 2 * C, 3 * C, j0);
    __syncthreads();
    am_products(s, ks, xs, 3 * C, scale, aa);
    am_products(s, vs, gy, C, 1.f, ds);
    __syncthreads();
    for (int i = threadIdx.x; i < s.Pp; i += AM_T) {
        const float* s3 = stats + ((int64_t)n * P + min(i, P - 1)) * 3;
        const float mx = s3[0], inv = 1.f / s3[1], r = s3[2];
#pragma unroll
        for (int j = 0; j < AM_R; ++j) {
            const float a = i < P ? expf(aa[j * s.tp + i] - mx) * inv : 0.f, d = ds[j * s.tp + i];
            aa[j * s.tp + i] = a;
            ds[j * s.tp + i] = i < P ? a * (d - r) : 0.f;
        }
    }
    __syncthreads();
    am_mix(s, aa, gy, C, red, [&](int r, int c, float (&v)[8]) {
        if (j0 + r < P) am_store8(dx + ((int64_t)n * P + j0 + r) * 3 * C + 2 * C + c, v, accumulate);
    });
    am_mix(s, ds, xs, 3 * C, red, [&](int r, int c, float (&v)[8]) {
        if (j0 + r >= P) return;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] *= scale;
        am_store8(dx + ((int64_t)n * P + j0 + r) * 3 * C + C + c, v, accumulate);
    });
}

static bool am_ok(int dtype, int C) { return dtype == LPM_BF16 && C % 8 == 0; }
// The backward kernels at P + C = ATT_LIMIT, where few channels beside many positions take the most: 149 KB
constexpr int AM_LDS = 160 * 1024 - 256;
static_assert(2 * AM_R * ((ATT_LIMIT + 31) / 32 * 32 + 4) * 4 + 2 * AM_R * (128 + 8) * 2 + (int)AM_RED <= AM_LDS &&
              2 * AM_R * (32 + 4) * 4 + 2 * AM_R * ((ATT_LIMIT + 127) / 128 * 128 + 8) * 2 + (int)AM_RED <= AM_LDS, "the score tiles and staged rows fit");
template <typename K>
static hipError_t am_prepare(K kernel, DeviceSet& done) { return allow_lds(kernel, AM_LDS, done); }

// parts of a block that share a channel in att_mix: as many as leave every thread a channel
static int att_parts(int C) { return C <= 32 ? 8 : C <= 64 ? 4 : C <= 128 ? 2 : 1; }
#define LPM_ATT_NP(NP_, ...)                                       \
    do {                                                           \
        if ((NP_) == 8) { constexpr int NP = 8; __VA_ARGS__; }     \
        else if ((NP_) == 4) { constexpr int NP = 4; __VA_ARGS__; } \
        else if ((NP_) == 2) { constexpr int NP = 2; __VA_ARGS__; } \
        else { constexpr int NP = 1; __VA_ARGS__; }                \
    } while (0)

hipError_t launch_attn_fwd(int dtype, int32_t m, int32_t P, int32_t C, const void* x, void* y, hipStream_t st) {
    if (!attn_ok(P, C)) return hipErrorInvalidValue;
    if (am_ok(dtype, C)) {
        static DeviceSet done;
        const hipError_t attr = am_prepare(attn_fwd_mm, done);
        if (attr != hipSuccess) return attr;
        const AmShape s(P, C);
        hipLaunchKernelGGL(attn_fwd_mm, dim3((unsigned)((P + AM_R - 1) / AM_R), (unsigned)m), dim3(AM_T), s.tile_bytes() + s.rows_bytes() + AM_RED, st, P, C,
                           (const bf16_t*)x, (bf16_t*)y);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)((P + ATT_QB - 1) / ATT_QB), (unsigned)m);
    const size_t lds = (size_t)ATT_QB * (C + P) * sizeof(float);
    const int np = att_parts(C);
    if (dtype == LPM_BF16) LPM_ATT_NP(np, hipLaunchKernelGGL((attn_fwd_kernel<bf16_t, NP>), grid, dim3(256), lds, st, P, C, (const bf16_t*)x, (bf16_t*)y));
    else LPM_ATT_NP(np, hipLaunchKernelGGL((attn_fwd_kernel<float, NP>), grid, dim3(256), lds, st, P, C, (const float*)x, (float*)y));
    return hipGetLastError();
}

hipError_t launch_attn_bwd(int dtype, int32_t m, int32_t P, int32_t C, const void* x, const void* dy, void* dx, int accumulate,
                           void* ws, hipStream_t st) {
    if (!attn_ok(P, C) || !ws) return hipErrorInvalidValue;
    if (am_ok(dtype, C)) {
        static DeviceSet done_q, done_kv;
        const hipError_t aq = am_prepare(attn_bwd_q_mm, done_q), akv = am_prepare(attn_bwd_kv_mm, done_kv);
        if (aq != hipSuccess || akv != hipSuccess) return aq != hipSuccess ? aq : akv;
        const AmShape s(P, C);
        const dim3 grid((unsigned)((P + AM_R - 1) / AM_R), (unsigned)m);
        const size_t lds = 2 * s.tile_bytes() + 2 * s.rows_bytes() + AM_RED;
        hipLaunchKernelGGL(attn_bwd_q_mm, grid, dim3(AM_T), lds, st, P, C, (const bf16_t*)x, (const bf16_t*)dy, (bf16_t*)dx, accumulate, (float*)ws);
        launch_last(attn_bwd_kv_mm, grid, dim3(AM_T), lds, st, P, C, (const bf16_t*)x, (const bf16_t*)dy, (bf16_t*)dx, accumulate, (const float*)ws);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)((P + ATT_QB - 1) / ATT_QB), (unsigned)m);
    const size_t lds = (size_t)ATT_QB * (2 * C + 2 * P) * sizeof(float);
    const int np = att_parts(C);
    if (dtype == LPM_BF16) {
        LPM_ATT_NP(np, hipLaunchKernelGGL((attn_bwd_q_kernel<bf16_t, NP>), grid, dim3(256), lds, st, P, C, (const bf16_t*)x, (const bf16_t*)dy,
                                          (bf16_t*)dx, accumulate, (float*)ws));
        LPM_ATT_NP(np, launch_last(attn_bwd_kv_kernel<bf16_t, NP>, grid, dim3(256), lds, st, P, C, (const bf16_t*)x, (const bf16_t*)dy,
                                          (bf16_t*)dx, accumulate, (const float*)ws));
    } else {
        LPM_ATT_NP(np, hipLaunchKernelGGL((attn_bwd_q_kernel<float, NP>), grid, dim3(256), lds, st, P, C, (const float*)x, (const float*)dy,
                                          (float*)dx, accumulate, (float*)ws));
        LPM_ATT_NP(np, launch_last(attn_bwd_kv_kernel<float, NP>, grid, dim3(256), lds, st, P, C, (const float*)x, (const float*)dy,
                                          (float*)dx, accumulate, (const float*)ws));
    }
    return hipGetLastError();
}

}  // namespace lpm
