// Sums of partial results: the split pixel ranges of weight gradients, in one launch for all layers of a backward pass, and
// the split reduction of a fully connected data gradient with its epilogue.
#include "lpm_internal.h"
#include "elem.h"

namespace lpm {

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

// sums split-K partials in split order, then (+)= , mask and scale as the data gradient asks
__global__ void __launch_bounds__(256) splitk_epilogue(const float* __restrict__ part, int splits, int64_t MN, int N, int accumulate,
                                                       const uint16_t* __restrict__ mask, const float* __restrict__ mscale,
                                                       uint16_t* __restrict__ C) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= MN) return;
    float v = sum_partials(part, splits, MN, i);
    if (accumulate) v += bf2f(C[i]);
    if (mask && !(bf2f(mask[i]) > 0.f)) v = 0.f;
    if (mscale) v *= mscale[(unsigned)i % (unsigned)N];      // (the output has fewer than 2^31 elements)
    C[i] = f2bf(v);
}

hipError_t launch_splitk_epilogue(const float* part, int splits, int64_t MN, int N, int accumulate, const void* mask, const float* mscale,
                                  void* C, hipStream_t st) {
    launch_last(splitk_epilogue, dim3((unsigned)((MN + 255) / 256)), dim3(256), 0, st, part, splits, MN, N, accumulate,
                       (const uint16_t*)mask, mscale, (uint16_t*)C);
    return hipGetLastError();
}

// parts that the splits of a reduction are cut into
__host__ __device__ inline int reduce_lanes_log(int splits) { return splits > 64 ? 4 : splits > 16 ? 2 : 0; }
__host__ __device__ inline int reduce_lanes(int splits) { return 1 << reduce_lanes_log(splits); }

struct ReduceBatchArgs {
    ReduceDesc d[LPM_REDUCE_BATCH];
    int first[LPM_REDUCE_BATCH + 1];         // first block of every reduction, INT_MAX past the last
    FastDiv row[LPM_REDUCE_BATCH];           // outputs of a row
};

// A thread sums four consecutive outputs over its part of the splits with 16-byte loads, eight splits in flight (split s of the
// part goes to chain s % 4, the chains are added pairwise at the end: a fixed order).  With few splits the part is all of
// them; with many (a layer of few weights and many pixels) the block's threads form reduce_lanes() parts of 256 / lanes
// threads, each part a contiguous range of splits, and the parts' sums are added in order through LDS -- a part's threads
// read consecutive memory (one wavefront that took 16 splits of 16 outputs instead read 64-byte pieces: 53 us per micro-batch
// of VGG-16/224 against 26).
__global__ void __launch_bounds__(256) wgrad_reduce_batch(ReduceBatchArgs a) {
    __shared__ float4 red[256];
    int k = 0;                                    // (a block never straddles two reductions; a sum, not a search: no load waits for the one before)
#pragma unroll
    for (int j = 1; j < LPM_REDUCE_BATCH; ++j) k += (int)blockIdx.x >= a.first[j];
    const ReduceDesc& d = a.d[k];
    const int log = reduce_lanes_log(d.splits), lanes = 1 << log, tpp = 256 >> log, part = threadIdx.x >> (8 - log), o = threadIdx.x & (tpp - 1);
    const int64_t i = ((int64_t)((int)blockIdx.x - a.first[k]) * tpp + o) * 4, end = d.n + d.nb;
    const int per = (d.splits + lanes - 1) >> log, s0 = part * per, s1 = min(d.splits, s0 + per);
    const FastDiv rd = a.row[k];
    const bool small = end < ((int64_t)1 << 31);
    auto row_of = [&](int64_t e) __attribute__((always_inline)) { return small ? div_by((int)e, rd) : (int)(e / d.row_len); };
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i + 4 <= end && (d.stride & 3) == 0) {
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
        r = make_float4((c[0].x + c[1].x) + (c[2].x + c[3].x), (c[0].y + c[1].y) + (c[2].y + c[3].y),
                        (c[0].z + c[1].z) + (c[2].z + c[3].z), (c[0].w + c[1].w) + (c[2].w + c[3].w));
    } else if (i < end) {                         // the ragged end, and layers whose partials are not 16-byte aligned
        float t[4] = {0.f, 0.f, 0.f, 0.f};
        for (int s = s0; s < s1; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) if (i + e < end) t[e] += d.part[(size_t)s * d.stride + i + e];
        r = make_float4(t[0], t[1], t[2], t[3]);
    }
    if (lanes > 1) {
        red[threadIdx.x] = r;
        __syncthreads();
        if (part) return;
        for (int q = 1; q < lanes; ++q) {
            const float4 v = red[q * tpp + o];
            r.x += v.x; r.y += v.y; r.z += v.z; r.w += v.w;
        }
    }
    if (i + 4 <= d.n) {
        if (d.rscale) {
            const int row = row_of(i), left = d.row_len - (int)(i - (int64_t)row * d.row_len);      // outputs before the next row
            const float f = d.rscale[row];
            if (left >= 4) { r.x *= f; r.y *= f; r.z *= f; r.w *= f; }
            else {
                r.x *= f;
                r.y *= d.rscale[row_of(i + 1)]; r.z *= d.rscale[row_of(i + 2)]; r.w *= d.rscale[row_of(i + 3)];
            }
        }
        float4* out = reinterpret_cast<float4*>(d.dst + i);
        if (d.accumulate) { const float4 q = *out; r.x += q.x; r.y += q.y; r.z += q.z; r.w += q.w; }
        *out = r;
        return;
    }
    const float t[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (i + e >= end) break;
        if (i + e < d.n) {
            const float v = d.rscale ? t[e] * d.rscale[row_of(i + e)] : t[e];
            d.dst[i + e] = d.accumulate ? d.dst[i + e] + v : v;
        } else {
            const int c = (int)(i + e - d.n);
            d.db[c] = d.accumulate ? d.db[c] + t[e] : t[e];
        }
    }
}

hipError_t launch_reduce_batch(const ReduceDesc* d, int count, hipStream_t st) {
    for (int done = 0; done < count;) {
        ReduceBatchArgs a{};
        int tot = 0, k = 0;
        for (; k < LPM_REDUCE_BATCH && done + k < count; ++k) {
            a.d[k] = d[done + k];
            a.first[k] = tot;
            tot += (int)(((a.d[k].n + a.d[k].nb + 3) / 4 * reduce_lanes(a.d[k].splits) + 255) / 256);
        }
        for (int j = 0; j < k; ++j) a.row[j] = fast_div(a.d[j].row_len);
        for (int j = k; j <= LPM_REDUCE_BATCH; ++j) a.first[j] = 0x7fffffff;
        done += k;
        if (tot == 0) continue;
        if (done < count) hipLaunchKernelGGL(wgrad_reduce_batch, dim3((unsigned)tot), dim3(256), 0, st, a);
        else launch_last(wgrad_reduce_batch, dim3((unsigned)tot), dim3(256), 0, st, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lpm
