// Chooses the contraction kernel for a convolution / FC shape: matrix-core tiles where the channel counts come in 16-byte
// chunks (igemm.hip, wgrad.hip), matrix cores fed by per-element gathers where they do not (gather.hip: image inputs, a few
// feature maps), the shape-generic vector-ALU kernels for what is left (launches of a few thousand products, filters of more
// than 12 taps an axis, strided data gradients of ragged channels).
#include "lpm_internal.h"
#include <algorithm>

namespace lpm {

hipError_t conv_fwd_generic_launch(int dtype, const ConvGeom& g, const void* x, const void* w, const float* scale,
                                   const float* bias, const void* add, int relu, void* y, hipStream_t s);
hipError_t conv_dgrad_generic_launch(int dtype, const ConvGeom& g, const void* dz, const float* dzscale, const void* w, void* dx,
                                     int accumulate, const void* mask, const float* mscale, hipStream_t s);
hipError_t conv_wgrad_generic_launch(int dtype, const ConvGeom& g, const void* x, const void* dz, float* dw,
                                     int accumulate, void* ws, hipStream_t s);
size_t wgrad_generic_ws_bytes(const ConvGeom& g);

bool mfma_fwd_ok(int dtype, const ConvGeom& g);
bool mfma_dgrad_ok(int dtype, const ConvGeom& g);
size_t mfma_fwd_ws_bytes(int dtype, const ConvGeom& g);
size_t mfma_dgrad_ws_bytes(int dtype, const ConvGeom& g);
bool mfma_fwd_pools(int dtype, const ConvGeom& g);
hipError_t mfma_conv_fwd(int dtype, const ConvGeom& g, const void* x, const void* w, const float* scale, const float* bias,
                         const void* add, int relu, void* y, void* ws, bool ws_zeroed, hipStream_t st, void* pool_y,
                         HeldCall* hold, HeldCall* with);
hipError_t mfma_conv_dgrad(int dtype, const ConvGeom& g, const void* dz, const void* wt, void* dx, int accumulate, const void* mask,
                           const float* mscale, void* ws, bool ws_zeroed, hipStream_t st, const UnpoolDesc* unpool, const DgradSide* side, const float* kscale,
                           HeldCall* hold, HeldCall* with);
bool mfma_dgrad_kscale_ok(const ConvGeom& g);
bool wgrad_mm_ok(int dtype, const ConvGeom& g);
size_t wgrad_mm_ws_bytes(int dtype, const ConvGeom& g);
hipError_t wgrad_mm_launch(int dtype, const WgradTask& t, hipStream_t st);
hipError_t wgrad_mm_group(int dtype, const WgradTask* t, int n, hipStream_t st, ReduceDesc* red);

bool fc_skinny_ok(const ConvGeom& g);
size_t fc_dgrad_ws_bytes(const ConvGeom& g);
hipError_t fc_dgrad(const ConvGeom& g, const void* dz, const float* dzscale, const void* w, void* dx, int accumulate, const void* mask,
                    const float* mscale, void* ws, hipStream_t st);
hipError_t fc_wgrad(const ConvGeom& g, const void* x, const void* dz, float* dw, float* dbias, const float* rscale,
                    int accumulate, hipStream_t st);

bool gather_fwd_ok(int dtype, const ConvGeom& g);
bool gather_dgrad_ok(int dtype, const ConvGeom& g);
bool gather_wgrad_ok(int dtype, const ConvGeom& g);
size_t gather_wgrad_ws_bytes(const ConvGeom& g);
hipError_t gather_conv_fwd(int dtype, const ConvGeom& g, const void* x, const void* w, const float* scale, const float* bias,
                           const void* add, int relu, void* y, hipStream_t st, void* pool_y);
bool gather_fwd_pools(const ConvGeom& g);
hipError_t gather_conv_dgrad(int dtype, const ConvGeom& g, const void* dz, const float* dzscale, const void* w, void* dx, int accumulate,
                             const void* mask, const float* mscale, hipStream_t st);
hipError_t gather_conv_wgrad(int dtype, const ConvGeom& g, const void* x, const void* dz, float* dw, float* dbias, const float* rscale,
                             int accumulate, void* ws, hipStream_t st, ReduceDesc* deferred);

// A filter that covers its whole input makes one output pixel per sample: x is a matrix [m][K] and w [Cout][K] as they lie in
// memory, so the layer is a 1x1 convolution of K channels.  (As a convolution its data gradient would visit every tap for
// every input pixel, of which one is real; and the reduction need not be cut at the taps.)
static ConvGeom fc_view(const ConvGeom& g) {
    if (!g.covers_input()) return g;
    ConvGeom v{g.m, 1, 1, g.K(), 1, 1, g.Cout, 1, 1, 1, 0};
    return v;
}
// A float contraction of a few hundred thousand products (a fully connected layer at eight samples) is one or two tiles of the
// matrix-core kernel and takes the latency of its K loop, 7-8 us; a group of lanes per output element, 4 us.
static bool tiny_f32(int dtype, const ConvGeom& g) { return dtype == LPM_F32 && g.rows_out() * g.Cout * g.K() < ((int64_t)1 << 21); }
static bool fwd_mm(int dtype, const ConvGeom& g) { return mfma_fwd_ok(dtype, g) && !tiny_f32(dtype, g); }
static bool dgrad_mm(int dtype, const ConvGeom& g) { return mfma_dgrad_ok(dtype, g) && !tiny_f32(dtype, g); }

size_t fwd_ws_bytes(int dtype, const ConvGeom& g_) {
    const ConvGeom g = fc_view(g_);
    return fwd_mm(dtype, g) ? mfma_fwd_ws_bytes(dtype, g) : 0;
}
// A float data gradient takes the fully connected view unless its epilogue goes by the channels of x; bf16 reads the
// transposed weights, whose layout keeps the taps.
static bool f32_dgrad_viewed(const ConvGeom& g, const float* mscale, const DgradSide* side) { return !mscale && !side && dgrad_mm(LPM_F32, fc_view(g)); }

size_t dgrad_ws_bytes(int dtype, const ConvGeom& g) {
    size_t b = dgrad_mm(dtype, g) ? mfma_dgrad_ws_bytes(dtype, g) : 0;
    if (dtype == LPM_F32 && dgrad_mm(dtype, fc_view(g))) b = std::max(b, mfma_dgrad_ws_bytes(dtype, fc_view(g)));
    if (dtype == LPM_BF16 && fc_skinny_ok(g)) return std::max(LPM_COUNT_BYTES + fc_dgrad_ws_bytes(g), b);
    return b;
}
size_t wgrad_ws_bytes(int dtype, const ConvGeom& g) {
    if (dtype == LPM_BF16 && fc_skinny_ok(g)) return 0;
    if (wgrad_mm_ok(dtype, fc_view(g))) return wgrad_mm_ws_bytes(dtype, fc_view(g));
    if (gather_wgrad_ok(dtype, g)) return gather_wgrad_ws_bytes(g);
    return wgrad_generic_ws_bytes(g);
}

bool fwd_can_pool(int dtype, const ConvGeom& g) {
    if (fwd_mm(dtype, fc_view(g))) return mfma_fwd_pools(dtype, g);
    return gather_fwd_ok(dtype, g) && gather_fwd_pools(g);
}

hipError_t launch_conv_fwd(int dtype, const ConvGeom& g, const void* x, const void* w, const float* scale,
                           const float* bias, const void* add, int relu, void* y, void* ws, hipStream_t st, void* pool_y, bool ws_zeroed,
                           HeldCall* hold, HeldCall* with) {
    if (pool_y && !fwd_can_pool(dtype, g)) return hipErrorInvalidValue;      // callers ask fwd_can_pool first
    if (fwd_mm(dtype, fc_view(g))) return mfma_conv_fwd(dtype, fc_view(g), x, w, scale, bias, add, relu, y, ws, ws_zeroed, st, pool_y, hold, with);
    const hipError_t e = with ? run_held(*with, st) : hipSuccess;
    if (e != hipSuccess) return e;
    if (gather_fwd_ok(dtype, g)) return gather_conv_fwd(dtype, g, x, w, scale, bias, add, relu, y, st, pool_y);
    return conv_fwd_generic_launch(dtype, g, x, w, scale, bias, add, relu, y, st);
}

bool wgrad_fuses_bias(int dtype, const ConvGeom& g) { return wgrad_mm_ok(dtype, fc_view(g)) || gather_wgrad_ok(dtype, g) || (dtype == LPM_BF16 && fc_skinny_ok(g)); }

// whether the data gradient wants the [Cin][Kh][Kw][Cout] copy of the weights
bool dgrad_uses_wt(int dtype, const ConvGeom& g) { return dtype == LPM_BF16 && !fc_skinny_ok(g) && mfma_dgrad_ok(dtype, g); }

// the stride-1 MFMA data gradient can route its result through a following (in forward order: preceding) max-pooling, whole
// chunks of eight channels at a time.  At every size: with a pooling kernel of its own for gradients of more than 2^20 elements VGG-16/224 took
// 3373 / 3718 / 5522 us per step of four micro-batches of 3 / 4 / 8 images, without it 3346 / 3681 / 5483; VGG-16/CIFAR at 128 images
// 2235 / 2217.
bool dgrad_can_unpool(int dtype, const ConvGeom& g) {
    return dtype == LPM_BF16 && !g.is3d() && !fc_skinny_ok(g) && mfma_dgrad_ok(dtype, g) && g.stride == 1 && g.Cin % 8 == 0;
}

// the MFMA data gradient can take over the epilogue backward of a layer with a shortcut (DgradSide)
bool dgrad_has_side(int dtype, const ConvGeom& g) { return dtype == LPM_F32 ? dgrad_mm(dtype, g) : dgrad_uses_wt(dtype, g); }

// whether the data gradient can apply the layer's scale to a dz that does not carry it (bf16: through the transposed weights)
bool dgrad_scales_dz(int dtype, const ConvGeom& g) { return dtype == LPM_BF16 || mfma_dgrad_kscale_ok(g); }

hipError_t launch_conv_dgrad(int dtype, const ConvGeom& g, const void* dz, const void* w, const void* wt, void* dx,
                             int accumulate, const void* mask, const float* mscale, void* ws, hipStream_t st,
                             const UnpoolDesc* unpool, const DgradSide* side, const float* dzscale, bool ws_zeroed,
                             HeldCall* hold, HeldCall* with) {
    if (unpool && !(dgrad_can_unpool(dtype, g) && wt)) return hipErrorInvalidValue;      // callers ask dgrad_can_unpool first
    if (side && !(dgrad_has_side(dtype, g) && (wt || dtype == LPM_F32))) return hipErrorInvalidValue;          // ... and dgrad_has_side
    const bool skinny = dtype == LPM_BF16 && fc_skinny_ok(g);
    if (!skinny && dtype == LPM_BF16 && wt && mfma_dgrad_ok(dtype, g)) return mfma_conv_dgrad(dtype, g, dz, wt, dx, accumulate, mask, mscale, ws, ws_zeroed, st, unpool, side, nullptr, hold, with);
    if (dtype == LPM_F32 && f32_dgrad_viewed(g, mscale, side)) return mfma_conv_dgrad(dtype, fc_view(g), dz, w, dx, accumulate, mask, nullptr, ws, ws_zeroed, st, nullptr, nullptr, dzscale, hold, with);
    if (dtype == LPM_F32 && dgrad_mm(dtype, g)) return mfma_conv_dgrad(dtype, g, dz, w, dx, accumulate, mask, mscale, ws, ws_zeroed, st, nullptr, side, dzscale, hold, with);
    const hipError_t e = with ? run_held(*with, st) : hipSuccess;
    if (e != hipSuccess) return e;
    if (skinny) return fc_dgrad(g, dz, dzscale, w, dx, accumulate, mask, mscale, (char*)ws + LPM_COUNT_BYTES, st);
    if (gather_dgrad_ok(dtype, g)) return gather_conv_dgrad(dtype, g, dz, dzscale, w, dx, accumulate, mask, mscale, st);
    return conv_dgrad_generic_launch(dtype, g, dz, dzscale, w, dx, accumulate, mask, mscale, st);
}

static bool wgrad_mm_taken(int dtype, const ConvGeom& g) { return !(dtype == LPM_BF16 && fc_skinny_ok(g)) && wgrad_mm_ok(dtype, fc_view(g)); }
// the kernels that take one layer a launch
static hipError_t wgrad_other(int dtype, const WgradTask& t, hipStream_t st, ReduceDesc* deferred) {
    if (deferred) deferred->splits = 0;
    if (dtype == LPM_BF16 && fc_skinny_ok(t.g)) return fc_wgrad(t.g, t.x, t.dz, t.dw, t.db, t.rscale, t.accumulate, st);
    if (gather_wgrad_ok(dtype, t.g)) return gather_conv_wgrad(dtype, t.g, t.x, t.dz, t.dw, t.db, t.rscale, t.accumulate, t.ws, st, deferred);
    if (t.db || t.rscale) return hipErrorInvalidValue;      // callers ask wgrad_fuses_bias first
    return conv_wgrad_generic_launch(dtype, t.g, t.x, t.dz, t.dw, t.accumulate, t.ws, st);
}
hipError_t launch_conv_wgrad(int dtype, const WgradTask& t, hipStream_t st) {
    if (!wgrad_mm_taken(dtype, t.g)) return wgrad_other(dtype, t, st, nullptr);
    WgradTask v = t;
    v.g = fc_view(t.g);
    return wgrad_mm_launch(dtype, v, st);
}
hipError_t launch_wgrad_group(int dtype, const WgradTask* t, int n, hipStream_t st, ReduceDesc* red) {
    if (n > LPM_WGRAD_GROUP) return hipErrorInvalidValue;
    WgradTask mm[LPM_WGRAD_GROUP];
    ReduceDesc r[LPM_WGRAD_GROUP];
    int at[LPM_WGRAD_GROUP], k = 0;
    for (int i = 0; i < n; ++i) {
        if (wgrad_mm_taken(dtype, t[i].g)) {
            mm[k] = t[i];
            mm[k].g = fc_view(t[i].g);
            at[k++] = i;
        } else {
            const hipError_t e = wgrad_other(dtype, t[i], st, &red[i]);
            if (e != hipSuccess) return e;
        }
    }
    if (!k) return hipSuccess;
    const hipError_t e = wgrad_mm_group(dtype, mm, k, st, r);
    for (int i = 0; i < k; ++i) red[at[i]] = r[i];
    return e;
}

// Staging pays when one read-modify-write pass over dW moves several times the bytes of the staged operands.  Per step without it for
// convolutions / with it, in us: VGG-16/CIFAR 1976 / 1895, ResNet-18/CIFAR 3320 / 3265, VGG-16/224 6718 / 6669, volumetric 1759 / 1761.
bool wgrad_staged_ok(int dtype, const ConvGeom& g) {
    if (dtype != LPM_BF16) return false;
    if (fc_staged_ok(g)) return true;
    if (fc_skinny_ok(g) || !wgrad_mm_ok(dtype, fc_view(g))) return false;
    const int64_t dw_rmw = (int64_t)g.Cout * g.K() * 8, staged = (g.rows_in() * g.Cin + g.rows_out() * g.Cout) * 2;
    return (int64_t)g.Cout * g.K() >= 32768 && dw_rmw >= 6 * staged;
}

size_t wgrad_staged_ws_bytes(int dtype, const ConvGeom& g) {
    if (!wgrad_staged_ok(dtype, g) || fc_staged_ok(g)) return 0;
    size_t b = 0;
    for (int s = 1; s <= LPM_FC_STAGE_SLOTS; ++s) b = std::max(b, wgrad_ws_bytes(dtype, staged_geom(g, s)));
    return b;
}

}  // namespace lpm
