// A stage = one sub-module (a stack of consecutive layers) and its three operations
// F_{z,j}, B_{z,j}, U_z.  Host code only: validates, lays out buffers, enqueues kernels.
//
// Layer-wise Partitioning and Merging: sub-module z takes the activation of z-1 in the forward
// pass and the gradient of z+1 in the backward pass.  Problem Statement eqs. 1, 8, 9 define what
// each layer computes in the two passes; eq. 6 the update.
#include "lpm_internal.h"

#include <algorithm>
#include <new>

#include "stage.h"
#include <cmath>

using namespace lpm;

// Whether the layer's weight-gradient kernel can sum its bias gradient from dz: where dz carries a scale its column sum is
// not the bias gradient.
static bool bias_in_wgrad_ok(int dtype, const LayerRt& lr) {
    return wgrad_fuses_bias(dtype, lr.g) && (lr.dz_unscaled || !(lr.d.flags & LPM_SCALE));
}
// ... or the weight phase can sum it from dz in a kernel of its own
static bool bias_from_dz_ok(const LayerRt& lr) { return lr.dz_unscaled || !(lr.d.flags & LPM_SCALE); }

// Layers whose weight gradients share launches, and their operations at most (float: a sixteenth; a layer of more is on its own).  A
// launch costs some 10 us, and what layers share of it they gain; but none of them starts before the last one's dz is there, which a
// long launch no longer makes up for.  The layers go into as few groups as the limits allow, as even as these can be (filled one after the
// other: float ResNet-18 at 7 and 8 samples + 2 %).  Per step, in per cent of the time with 20 G operations:
//                                            none    10    20    25    30    40   any
//   R50 conv4_x, 16 samples a micro-batch     104   103   100   100   100   100   100
//   24 / 32 samples                       103/100 100/102 100  98/99  98/98  98/99  98/99
//   48 samples                                100    99   100    99    99    98    97
//   VGG-16/224, 4                             100   100   100   100   100   101   102
//   ResNet-18/CIFAR, 32                       107   100   100   100   100   100   100
//   width-48 ResNet, 13                       118   100   100   100   100   100   101
//   float ResNet-18, 8                        107   102   100   100   100   103   104
//   float ResNet-18, 9 / 12               104/103 101/101 100  97/98  97/95 100/96 100/98
// With 4 / 8 / 16 layers R50 conv4_x at 16 took 1710 / 1623 / 1655 us, ResNet-18/CIFAR 2921 / 2892 / 2907.
constexpr int32_t WG_LAYERS = 8;
constexpr double WG_WORK = 30e9;
static_assert(WG_LAYERS <= LPM_WGRAD_GROUP, "a launch takes that many");

static bool misaligned(const void* p) { return ((uintptr_t)p & 255u) != 0; }

extern "C" int32_t lpm_stage_create(const lpm_layer* layers, int32_t L, int32_t first, int32_t last,
                                    int32_t microbatch, int32_t dtype, lpm_stage** out) {
    if (!out) return fail(LPM_EINVAL, "out is NULL");
    *out = nullptr;
    if (dtype != LPM_F32 && dtype != LPM_BF16) return fail(LPM_EINVAL, "dtype must be LPM_F32 or LPM_BF16");
    if (microbatch <= 0) return fail(LPM_EINVAL, "microbatch must be positive");
    lpm_stage* s = new (std::nothrow) lpm_stage();
    if (!s) return fail(LPM_ENOMEM, "out of host memory");
    int32_t rc = validate_network(layers, L, s->net, s->shapes);
    if (rc) { delete s; return rc; }
    if (first < 0 || last > L || first >= last) { delete s; return fail(LPM_EINVAL, "stage range [%d,%d) is not inside the network", first, last); }
    s->first = first; s->last = last; s->m = microbatch; s->dtype = dtype; s->L = L;
    s->esz = dtype == LPM_BF16 ? 2 : 4;
    s->loss = s->net[last - 1].kind == LPM_SOFTMAX_CE;
    if (s->loss && last - first < 2) { delete s; return fail(LPM_ESHAPE, "the loss layer cannot form a stage on its own"); }
    // every tensor read from outside must be the stage input
    for (int32_t i = first; i < last; ++i) {
        const lpm_layer& l = s->net[i];
        if (l.src < first - 1 || (l.add_src != LPM_NONE && l.add_src < first - 1)) {
            delete s;
            return fail(LPM_ESHAPE, "layer %d reads a tensor produced before the stage input (%d)", i, first - 1);
        }
    }
    // no tensor of this stage other than its output may be read by a later layer
    for (int32_t i = last; i < L; ++i) {
        const lpm_layer& l = s->net[i];
        for (int32_t ref : {l.src, l.add_src}) {
            if (ref != LPM_NONE && ref >= first && ref < last - 1) {
                delete s;
                return fail(LPM_ESHAPE, "layer %d reads tensor %d across the stage boundary", i, ref);
            }
        }
    }

    // tensors first-1 .. last-1
    s->ten.resize((size_t)(last - first + 1));
    s->t_out = s->loss ? last - 2 : last - 1;
    size_t stash = 0, gws = 0;
    for (int32_t t = first - 1; t < last; ++t) {
        TensorRt& tr = s->T(t);
        tr.shape = s->shapes[(size_t)t + 1];
        tr.bytes = tr.shape.elems() * (size_t)microbatch * s->esz;
        if (t == first - 1) tr.loc = LOC_X;
        else if (t == s->t_out || (s->loss && t == last - 1)) tr.loc = LOC_Y;
        else {
            tr.loc = LOC_STASH;
            tr.stash_off = stash;
            stash += align_up(tr.bytes, 256);
            tr.g_off = gws;
            gws += align_up(tr.bytes, 256);
        }
    }
    if (s->loss) {
        s->dlogits_off = stash;
        stash += align_up(s->T(last - 2).bytes, 256);
    }
    s->stash_bytes = stash;

    s->lay.resize((size_t)(last - first));
    for (int32_t i = first; i < last; ++i) {
        LayerRt& lr = s->Ly(i);
        lr.d = s->net[i];
        const lpm_layer& l = lr.d;
        const Shape o = s->shapes[(size_t)i + 1];
        lr.g = ConvGeom{microbatch, l.h_in, l.w_in, l.cin, o.h, o.w, o.c, l.kh, l.kw, l.stride, l.pad};
        if (has_weights(l) && (l.d_in > 1 || l.kd > 1)) {          // a volumetric layer: the tensor heights are slices x rows
            lr.g.D = l.d_in; lr.g.Kd = l.kd; lr.g.pad_d = l.pad_d;
            lr.g.Do = (l.d_in + 2 * l.pad_d - l.kd) / l.stride + 1;
            lr.g.Ho = o.h / lr.g.Do;
        }
    }
    auto uses = [&](int32_t t, int& n_src, int& n_add) {
        n_src = n_add = 0;
        for (int32_t j = std::max(t + 1, first); j < last; ++j) { n_src += s->net[(size_t)j].src == t; n_add += s->net[(size_t)j].add_src == t; }
    };
    // The head: an average pooling whose only reader is a plain layer over its channels.
    for (int32_t i = first; i + 1 < last; ++i) {
        if (s->net[(size_t)i].kind != LPM_GAP || i == s->t_out) continue;
        LayerRt& fc = s->Ly(i + 1);
        int n_src, n_add;
        uses(i, n_src, n_add);
        if (n_src != 1 || n_add != 0 || !has_weights(fc.d) || fc.d.src != i || (fc.d.flags & (LPM_RELU | LPM_SCALE)) || fc.d.add_src != LPM_NONE) continue;
        if (fc.g.K() != fc.g.Cin || fc.g.rows_out() != microbatch) continue;
        const int32_t hw = s->net[(size_t)i].h_in * s->net[(size_t)i].w_in;
        fc.headed_fwd = head_ok(dtype, microbatch, hw, fc.g.Cin, fc.g.Cout, true);
        fc.headed_bwd = head_ok(dtype, microbatch, hw, fc.g.Cin, fc.g.Cout, false);
        if (fc.headed_fwd) s->Ly(i).head_fwd = i + 1;
        if (fc.headed_bwd) s->Ly(i).head_bwd = i + 1;
    }
    // parameters: trainable (W, bias per layer) first, frozen scales after
    size_t off = 0, lowp = 0, kws = 0, wws = 0, fws = 0, fcs = 0;
    for (int32_t i = first; i < last; ++i) {
        LayerRt& lr = s->Ly(i);
        const lpm_layer& l = lr.d;
        const Shape o = s->shapes[(size_t)i + 1];
        if (!has_weights(l)) {
            if (l.kind == LPM_ATTN) {
                if (!attn_ok(l.h_in * l.w_in, l.cout)) { delete s; return fail(LPM_ESHAPE, "layer %d: attention over %d positions of %d channels is outside the kernel's limits", i, l.h_in * l.w_in, l.cout); }
                kws = std::max(kws, align_up(LPM_COUNT_BYTES + attn_bwd_ws_bytes(microbatch, l.h_in * l.w_in), 256));
            }
            continue;
        }
        lr.w_count = (size_t)l.cout * taps_of(l) * l.cin;
        lr.w_off = off;
        off += align_up(lr.w_count, 64);
        if (l.flags & LPM_BIAS) { lr.b_off = off; off += align_up((size_t)l.cout, 64); }
        if (dtype == LPM_BF16) {
            lr.lowp_w_off = lr.w_off * 2;      // the bf16 copies mirror the float layout element for element
            if (!lr.headed_bwd && dgrad_uses_wt(dtype, lr.g)) { lr.lowp_wt_off = lowp; lowp += align_up(lr.w_count * 2, 256); }   // rebased below
        }
        // A scaled layer whose weight-gradient kernel also sums the bias gradient keeps dz free of the scale: the bias
        // gradient is then the plain column sum of dz (eq. 8 for the bias), whatever the scale's value -- zero included.
        lr.dz_unscaled = (l.flags & LPM_SCALE) && wgrad_fuses_bias(dtype, lr.g) && dgrad_scales_dz(dtype, lr.g);
        if (l.flags & (LPM_RELU | LPM_SCALE)) {          // needs its own dz buffer (it outlives the layer's turn)
            lr.dz_off = gws;
            gws += align_up(o.elems() * (size_t)microbatch * s->esz, 256);
        }
        lr.wws_off = wws;                        // every layer its own area: the reductions of a pass run in one launch
        wws += align_up(std::max({wgrad_ws_bytes(dtype, lr.g), wgrad_staged_ws_bytes(dtype, lr.g),
                                  epi_bwd_ws_bytes(lr.g.rows_out(), l.cout)}), 256);   // (a bias-only reduction runs here too)
        if (wgrad_staged_ok(dtype, lr.g)) {
            lr.fcs_x_off = fcs;  fcs += align_up((size_t)LPM_FC_STAGE_SLOTS * lr.g.rows_in() * lr.g.Cin * 2, 256);
            lr.fcs_dz_off = fcs; fcs += align_up((size_t)LPM_FC_STAGE_SLOTS * lr.g.rows_out() * lr.g.Cout * 2, 256);
        }
        const size_t dws = lr.headed_bwd ? 0 : dgrad_ws_bytes(dtype, lr.g);      // (of the passes that the head's kernels perform, nothing is kept ready)
        kws = std::max(kws, align_up(dws, 256));
        kws = std::max(kws, align_up(LPM_COUNT_BYTES + epi_bwd_ws_bytes(lr.g.rows_out(), l.cout), 256));
        if (dws) s->bwd_counts = true;
        if (!lr.headed_fwd) fws = std::max(fws, align_up(fwd_ws_bytes(dtype, lr.g), 256));
    }
    // Whether layer i's shortcut can take i's dz for its gradient instead of a copy: dz carries no scale, the shortcut is tensor a's
    // only one, and from then on the gradient of a is only read -- as the earlier contribution that the data gradient
    // of the block before adds in (a fused_side), or as the dz of a projection without ReLU and scale of its own.
    auto shares_dz = [&](int32_t i) {
        const LayerRt& lr = s->Ly(i);
        const int32_t a = lr.d.add_src;
        if (a == LPM_NONE || a < first || ((lr.d.flags & LPM_SCALE) && !lr.dz_unscaled)) return false;
        const LayerRt& ar = s->Ly(a);
        int n_src, n_add;
        uses(a, n_src, n_add);
        if (n_add != 1) return false;
        if (ar.fused_side) return n_src == 1;      // (another layer's data gradient would be added to the shared buffer)
        return n_src == 0 && has_weights(ar.d) && !(ar.d.flags & LPM_RELU) && ar.d.add_src == LPM_NONE && (!(ar.d.flags & LPM_SCALE) || ar.dz_unscaled);
    };
    // Epilogue-backward fusion: the first layer that reads a layer's output is the last to contribute to its gradient, and where it
    // reads it as its `src`, its backward kernel (data gradient / pooling backward) applies the ReLU mask and the scale itself and
    // writes dz directly; the bias gradient then comes out of the weight-gradient kernel.
    for (int32_t i = first; i < last; ++i) {
        LayerRt& lr = s->Ly(i);
        const lpm_layer& l = lr.d;
        if (!has_weights(l)) continue;
        if (i == s->t_out) {                   // its gradient arrives from outside the stage
            lr.shortcut_is_dz = shares_dz(i);
            continue;
        }
        if (!(l.flags & (LPM_RELU | LPM_SCALE))) continue;
        int n_src = 0, n_other = 0, n_add = 0;
        int32_t consumer = -1, first_add = last;
        for (int32_t j = i + 1; j < last; ++j) {
            const lpm_layer& c = s->net[j];
            if (c.src == i) {
                ((c.kind == LPM_SOFTMAX_CE || c.kind == LPM_ATTN) ? n_other : n_src)++;
                if (consumer < 0) consumer = j;
            }
            if (c.add_src == i) { ++n_add; first_add = std::min(first_add, j); }
        }
        if (n_src < 1 || n_other != 0) continue;
        if ((l.flags & LPM_BIAS) && !bias_from_dz_ok(lr)) continue;
        if (l.add_src != LPM_NONE || n_add > 0 || n_src > 1) {
            // Residual blocks.  The layer adds a shortcut, and / or later layers use its output as their shortcut, or a projection
            // of the next block reads it too: the layer that reads it first in layer order makes the last contribution in
            // the backward pass, and an MFMA data gradient can add the earlier ones, mask, and write both this layer's dz and the
            // shortcut's gradient.  (Of the blocks before a projection, instead of a pass of their own: width-48 ResNet 2437 -> 2405 us
            // per step, ResNet-18/CIFAR 2917 -> 2891.)  The global average pooling behind the last block masks, too,
            // where nothing is to be added and the shortcut shares the dz.
            const lpm_layer& c = s->net[(size_t)consumer];
            if (c.kind == LPM_GAP && n_add == 0 && n_src == 1 && shares_dz(i)) {
                lr.shortcut_is_dz = true;
                lr.fused_in = true;
                lr.fused_by = consumer;
                continue;
            }
            if (!has_weights(c) || first_add < consumer || !dgrad_has_side(dtype, s->Ly(consumer).g)) continue;
            lr.fused_side = true;
            lr.shortcut_is_dz = shares_dz(i);
        }
        lr.fused_in = true;
        lr.fused_by = consumer;
    }
    // ... and a projection shortcut: a scale-only layer (no ReLU, no shortcut of its own) whose output is read by
    // exactly one layer, as its shortcut, when that layer is fused_side: the shortcut gradient that layer's fused
    // epilogue writes is this layer's output gradient, and times this layer's scale it is this layer's dz.
    for (int32_t i = first; i < last; ++i) {
        LayerRt& lr = s->Ly(i);
        const lpm_layer& l = lr.d;
        if (!has_weights(l) || (l.flags & LPM_RELU) || !(l.flags & LPM_SCALE) || l.add_src != LPM_NONE) continue;
        if (i == s->t_out) continue;
        if ((l.flags & LPM_BIAS) && !bias_from_dz_ok(lr)) continue;
        int n_src = 0, n_add = 0;
        int32_t user = -1;
        for (int32_t j = i + 1; j < last; ++j) {
            if (s->net[(size_t)j].src == i) ++n_src;
            if (s->net[(size_t)j].add_src == i) { ++n_add; user = j; }
        }
        if (n_src != 0 || n_add != 1 || !s->Ly(user).fused_side || s->Ly(user).shortcut_is_dz) continue;
        lr.fused_in = true;
        lr.via_shortcut = true;
    }
    // The last contribution to the gradient of the stage's input, in the order of the backward pass: the first layer that reads
    // the input.  It can apply the ReLU mask of the tensor if it reads it as its source with a kernel that adds what is
    // there before it masks (max-pooling masks its own contribution only).
    if (first > 0) {
        int n_src, n_add;
        uses(first - 1, n_src, n_add);
        for (int32_t j = first; j < last; ++j) {
            const lpm_layer& l = s->net[(size_t)j];
            if (l.src != first - 1 && l.add_src != first - 1) continue;
            const bool adds = l.kind == LPM_CONV || l.kind == LPM_FC || l.kind == LPM_GAP;
            if (l.src == first - 1 && l.add_src != first - 1 && (adds || (l.kind == LPM_MAXPOOL2 && n_src + n_add == 1))) s->mask_layer = j;
            break;
        }
    }
    // Pooling-backward fusion: a 2x2 max-pooling (even input extent) whose output feeds exactly one layer, a
    // convolution whose data gradient runs on the stride-1 MFMA kernel: that kernel routes its result to the
    // window maxima itself and the gradient of the pooling output is never stored.
    for (int32_t i = first; i < last; ++i) {
        LayerRt& lr = s->Ly(i);
        const lpm_layer& l = lr.d;
        if (!has_weights(l) || l.src < first || s->net[(size_t)l.src].kind != LPM_MAXPOOL2) continue;
        const int32_t p = l.src;
        const lpm_layer& pl = s->net[(size_t)p];
        if (p == s->t_out || (pl.h_in & 1) || (pl.w_in & 1) || !dgrad_can_unpool(dtype, lr.g) || !dgrad_uses_wt(dtype, lr.g)) continue;
        int n_cons = 0;
        for (int32_t j = p + 1; j < last; ++j) n_cons += (s->net[(size_t)j].src == p) + (s->net[(size_t)j].add_src == p);
        if (n_cons != 1) continue;
        lr.unpool_of = p;
        s->Ly(p).unpooled = true;
    }
    // Pooling-forward fusion: a convolution whose output feeds a 2x2 max-pooling inside the stage and whose forward kernel can
    // store the pooled tensor as well (one kernel less per pool on the forward chain; the pooling layer's own input stays
    // stored, the backward pass needs it).
    for (int32_t i = first; i + 1 < last; ++i) {
        LayerRt& lr = s->Ly(i);
        const lpm_layer& l = lr.d;
        const lpm_layer& pl = s->net[(size_t)i + 1];
        if (!has_weights(l) || l.add_src != LPM_NONE || pl.kind != LPM_MAXPOOL2 || pl.src != i) continue;
        if ((pl.h_in & 1) || (pl.w_in & 1) || !fwd_can_pool(dtype, lr.g)) continue;
        lr.pool_fwd = i + 1;
        s->Ly(i + 1).pooled_fwd = true;
    }
    // A projection and the layer of the block that stands beside it do not read each other's results: forward, the projection
    // and the layer before it; backward, where the projection's dz is there with that of the layer that adds it, those two.
    // Small contractions share a launch then.
    for (int32_t i = first; i + 1 < last; ++i) {
        LayerRt& lr = s->Ly(i);
        LayerRt& nx = s->Ly(i + 1);
        if (!has_weights(lr.d) || !has_weights(nx.d) || nx.d.src == i || lr.headed_fwd || lr.headed_bwd) continue;
        lr.hold_fwd = nx.d.add_src != i && lr.pool_fwd < 0;
        int n_src, n_add;
        uses(i, n_src, n_add);
        // what a data gradient writes: the gradient of its source, and maybe that of the shortcut of the layer that made the source
        auto shortcut_of = [&](int32_t t) { return t >= first ? s->Ly(t).d.add_src : LPM_NONE; };
        const int32_t a0 = nx.d.src, a1 = shortcut_of(a0), b0 = lr.d.src, b1 = shortcut_of(b0);
        const bool apart = a0 != b0 && a1 != b0 && a0 != b1 && (a1 != b1 || a1 == LPM_NONE);
        nx.hold_bwd = nx.d.add_src == i && n_src == 0 && n_add == 1 && apart && nx.unpool_of < 0 && lr.unpool_of < 0 &&
                      lr.d.add_src == LPM_NONE && !(lr.d.flags & LPM_RELU) && (!(lr.d.flags & LPM_SCALE) || lr.dz_unscaled || lr.via_shortcut);
    }
    // Weight gradients are launched in groups of consecutive layers (the same groups in every form of the backward pass: what a
    // launch holds decides how its reductions are cut; WG_LAYERS, WG_WORK); next to the network's input, where the micro-batch waits for the
    // last weight gradient, one and two (us per step with none but the limits / one / one and two / one to four apart: R50 conv4_x at 16 samples
    // 1700 / 1689 / 1656 / 1687, ResNet-18/CIFAR at 32 1561 / 1553 / 1555 / 1552, width-48 ResNet 1837 / 1812 / 1814 / 1812, volumetric 1602 / 1620 /
    // 1622 / 1618).
    {
        std::vector<LayerRt*> ly;
        std::vector<double> w;
        for (int32_t i = first; i < last; ++i) {           // from the stage's input up: the backward pass ends there
            LayerRt& lr = s->Ly(i);
            if (!has_weights(lr.d)) continue;
            ly.push_back(&lr);
            w.push_back(2. * (double)lr.g.rows_out() * lr.g.Cout * lr.g.K() * (dtype == LPM_F32 ? 16 : 1));
        }
        const size_t n = ly.size();
        // the layer behind the group that begins at `at`: of no more than `layers`, and of no more than `most` operations or one layer
        auto next = [&](size_t at, size_t layers, double most) {
            double work = w[at];
            size_t k = at + 1;
            while (k < n && k - at < layers && work + w[k] <= most) work += w[k++];
            return k;
        };
        size_t from = 0;
        for (size_t layers = 1; first == 0 && layers <= 2 && from < n; ++layers) {
            ly[from]->wg_end = true;
            from = next(from, layers, WG_WORK);
        }
        auto groups = [&](double most, bool mark) {
            int c = 0;
            for (size_t at = from; at < n; at = next(at, WG_LAYERS, most), ++c) if (mark) ly[at]->wg_end = true;
            return c;
        };
        const int fewest = groups(WG_WORK, false);
        double even = WG_WORK;                             // the least limit that makes as few
        for (size_t i = from; i < n; ++i) {
            double sum = 0;
            for (size_t k = i; k < n && k - i < (size_t)WG_LAYERS; ++k) {
                sum += w[k];
                if (sum < even && groups(sum, false) == fewest) even = sum;
            }
        }
        groups(even, true);
    }
    s->n_trainable = off;
    if (dtype == LPM_BF16) {                   // transposed copies follow the mirrored region
        const size_t base = align_up(off * 2, 256);
        for (int32_t i = first; i < last; ++i)
            if (s->Ly(i).lowp_wt_off != NO) s->Ly(i).lowp_wt_off += base;
        lowp += base;
    }
    for (int32_t i = first; i < last; ++i) {
        LayerRt& lr = s->Ly(i);
        if (has_weights(lr.d) && (lr.d.flags & LPM_SCALE)) { lr.s_off = off; off += align_up((size_t)lr.d.cout, 64); }
    }
    s->n_params = off;
    s->lowp_bytes = lowp;
    // backward scratch: two copies of the gradient / dz area (a schedule alternates between them so the weight
    // phase of one micro-batch may still read its dz while the next data phase writes), then kernel scratch
    s->gws_bytes = gws;
    s->kws_off = 2 * gws;
    s->wws_off = 2 * gws + kws;
    for (int32_t i = first; i < last; ++i) {     // the staging areas follow the kernel scratch
        LayerRt& lr = s->Ly(i);
        if (lr.fcs_x_off != NO) { lr.fcs_x_off += 2 * gws + kws + wws; lr.fcs_dz_off += 2 * gws + kws + wws; }
    }
    s->bwd_ws = std::max<size_t>(2 * gws + kws + wws + fcs, 256);
    s->fwd_ws = std::max<size_t>(fws, 256);
    s->fwd_counts = fws > 0;
    *out = s;
    return LPM_OK;
}

lpm_stage::~lpm_stage() {
    if (ev_join) (void)hipEventDestroy(ev_join);
    if (ev_w2_fork) (void)hipEventDestroy(ev_w2_fork);
    if (ev_w2_join) (void)hipEventDestroy(ev_w2_join);
    for (hipEvent_t v : ev_layer) if (v) (void)hipEventDestroy(v);
}

// Borrows the side stream and creates the events on first use (needs a device; stage creation does not).
int32_t lpm_stage_prepare(lpm_stage* s) {
    if (s->side) return LPM_OK;
    hipStream_t st = nullptr;
    LPM_HIP(pooled_stream(next_side_stream_index(), &st));
    hipEvent_t ej = nullptr, e2f = nullptr, e2j = nullptr;
    hipError_t e = hipEventCreateWithFlags(&ej, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&e2f, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&e2j, hipEventDisableTiming);
    if (e != hipSuccess) {
        if (ej) (void)hipEventDestroy(ej);
        if (e2f) (void)hipEventDestroy(e2f);
        return hip_fail(e, "hipEventCreateWithFlags");
    }
    std::vector<hipEvent_t> evl((size_t)(s->last - s->first) * LPM_MAX_WINDOW, nullptr);
    for (int32_t i = s->first; i < s->last && e == hipSuccess; ++i) {
        if (!has_weights(s->Ly(i).d)) continue;
        for (int k = 0; k < LPM_MAX_WINDOW && e == hipSuccess; ++k)
            e = hipEventCreateWithFlags(&evl[(size_t)(i - s->first) * LPM_MAX_WINDOW + k], hipEventDisableTiming);
    }
    if (e != hipSuccess) {
        for (hipEvent_t v : evl) if (v) (void)hipEventDestroy(v);
        (void)hipEventDestroy(ej); (void)hipEventDestroy(e2f); (void)hipEventDestroy(e2j);
        return hip_fail(e, "hipEventCreateWithFlags");
    }
    s->ev_layer = std::move(evl);
    s->ev_join = ej;
    s->ev_w2_fork = e2f;
    s->ev_w2_join = e2j;
    s->side = st;
    return LPM_OK;
}

extern "C" int32_t lpm_stage_destroy(lpm_stage* s) {
    delete s;
    return LPM_OK;
}

extern "C" int32_t lpm_stage_sizes(const lpm_stage* s, size_t* param_bytes, size_t* lowp_bytes, size_t* grad_bytes,
                                   size_t* stash_bytes, size_t* fwd_ws_bytes_, size_t* bwd_ws_bytes,
                                   size_t* in_bytes, size_t* out_bytes) {
    if (!s) return fail(LPM_EINVAL, "stage is NULL");
    if (param_bytes) *param_bytes = std::max<size_t>(s->n_params * 4, 256);
    if (lowp_bytes) *lowp_bytes = s->lowp_bytes;
    if (grad_bytes) *grad_bytes = std::max<size_t>(s->n_trainable * 4, 256);
    if (stash_bytes) *stash_bytes = std::max<size_t>(s->stash_bytes, 256);
    if (fwd_ws_bytes_) *fwd_ws_bytes_ = s->fwd_ws;
    if (bwd_ws_bytes) *bwd_ws_bytes = s->bwd_ws;
    if (in_bytes) *in_bytes = s->T(s->first - 1).bytes;
    if (out_bytes) *out_bytes = s->T(s->t_out).bytes;
    return LPM_OK;
}

extern "C" int32_t lpm_stage_param_offset(const lpm_stage* s, int32_t layer, int32_t which, size_t* offset, size_t* count) {
    if (!s || !offset || !count) return fail(LPM_EINVAL, "NULL argument");
    if (layer < s->first || layer >= s->last) return fail(LPM_EINVAL, "layer %d is not in the stage", layer);
    const LayerRt& lr = s->Ly(layer);
    size_t o = NO, c = 0;
    if (which == 0) { o = lr.w_off; c = lr.w_count; }
    else if (which == 1) { o = lr.b_off; c = (size_t)lr.d.cout; }
    else if (which == 2) { o = lr.s_off; c = (size_t)lr.d.cout; }
    if (o == NO) return fail(LPM_EINVAL, "layer %d has no parameter tensor %d", layer, which);
    *offset = o; *count = c;
    return LPM_OK;
}

extern "C" int32_t lpm_stage_stash_offset(const lpm_stage* s, int32_t t, size_t* offset, size_t* bytes) {
    if (!s || !offset || !bytes) return fail(LPM_EINVAL, "NULL argument");
    if (t == -100) {
        if (!s->loss) return fail(LPM_EINVAL, "not a loss stage");
        *offset = s->dlogits_off; *bytes = s->T(s->last - 2).bytes;
        return LPM_OK;
    }
    if (t < s->first - 1 || t >= s->last || s->T(t).loc != LOC_STASH) return fail(LPM_EINVAL, "tensor %d is not in the stash", t);
    *offset = s->T(t).stash_off; *bytes = s->T(t).bytes;
    return LPM_OK;
}

extern "C" int32_t lpm_stage_grad_offset(const lpm_stage* s, int32_t t, size_t* offset, size_t* bytes) {
    if (!s || !offset || !bytes) return fail(LPM_EINVAL, "NULL argument");
    if (t < s->first - 1 || t >= s->last || s->T(t).loc != LOC_STASH) return fail(LPM_EINVAL, "tensor %d has no gradient in the scratch", t);
    *offset = s->T(t).g_off; *bytes = s->T(t).bytes;
    return LPM_OK;
}

// the update stores this layer's [Cin][Kh][Kw][Cout] copy itself
static bool update_transposes(const LayerRt& lr) { return lr.lowp_wt_off != NO && lr.d.cin % 4 == 0 && lr.d.cout % 4 == 0; }

// the [Cin][Kh][Kw][Cout] copies of every layer whose data gradient reads one, all in one launch; behind an update those that
// it has not stored
static hipError_t transpose_copies(const lpm_stage* s, const float* params, void* lowp, bool updated, hipStream_t st) {
    std::vector<TransposeDesc> d;
    for (int32_t i = s->first; i < s->last; ++i) {
        const LayerRt& lr = s->Ly(i);
        if (lr.lowp_wt_off != NO && !(updated && update_transposes(lr)))
            d.push_back(TransposeDesc{params + lr.w_off, (uint16_t*)((char*)lowp + lr.lowp_wt_off), lr.d.cout, taps_of(lr.d), lr.d.cin,
                                      lr.dz_unscaled ? params + lr.s_off : nullptr});
    }
    return d.empty() ? hipSuccess : launch_weight_transpose_batch(d.data(), (int)d.size(), st);
}

// the pieces of the trainable parameters: weights with a transposed copy, and everything between them
static std::vector<UpdateSeg> update_segments(const lpm_stage* s, const float* params, void* lowp) {
    std::vector<UpdateSeg> d;
    size_t at = 0;
    for (int32_t i = s->first; i < s->last; ++i) {
        const LayerRt& lr = s->Ly(i);
        if (!update_transposes(lr)) continue;
        if (lr.w_off > at) d.push_back(UpdateSeg{at, lr.w_off - at, nullptr, nullptr, 0, 0, 0});
        d.push_back(UpdateSeg{lr.w_off, lr.w_count, (uint16_t*)((char*)lowp + lr.lowp_wt_off), lr.dz_unscaled ? params + lr.s_off : nullptr,
                              lr.d.cout, taps_of(lr.d), lr.d.cin});
        at = lr.w_off + lr.w_count;
    }
    if (s->n_trainable > at) d.push_back(UpdateSeg{at, s->n_trainable - at, nullptr, nullptr, 0, 0, 0});
    return d;
}

extern "C" int32_t lpm_stage_sync_lowp(lpm_stage* s, const float* params, void* lowp, void* stream) {
    if (!s || !params) return fail(LPM_EINVAL, "NULL argument");
    if (s->dtype != LPM_BF16) return LPM_OK;
    if (!lowp) return fail(LPM_EINVAL, "lowp is NULL");
    if (misaligned(params) || misaligned(lowp)) return fail(LPM_EALIGN, "buffers must be 256-byte aligned");
    hipStream_t st = (hipStream_t)stream;
    LPM_HIP(launch_f32_to_bf16(params, (uint16_t*)lowp, s->n_trainable, st));
    LPM_HIP(transpose_copies(s, params, lowp, false, st));
    return LPM_OK;
}

namespace {
// Where tensor t lives for this call.
inline const void* tptr(const lpm_stage* s, int32_t t, const void* x, const void* y, const void* stash) {
    const TensorRt& tr = s->T(t);
    if (tr.loc == LOC_X) return x;
    if (tr.loc == LOC_Y) return y;
    return (const char*)stash + tr.stash_off;
}
}  // namespace

extern "C" int32_t lpm_stage_forward(lpm_stage* s, const void* x, void* y, const int32_t* labels, float* loss_accum,
                                     const float* params, const void* lowp, void* stash, void* fwd_ws,
                                     float loss_scale, void* stream) {
    return lpm_stage_forward_on(s, x, y, labels, loss_accum, params, lowp, stash, fwd_ws, loss_scale, stream, false);
}

// counts_zeroed: the caller has cleared the arrival counts at the head of fwd_ws (a schedule does so once per run)
int32_t lpm_stage_forward_on(lpm_stage* s, const void* x, void* y, const int32_t* labels, float* loss_accum, const float* params,
                             const void* lowp, void* stash, void* fwd_ws, float loss_scale, void* stream, bool counts_zeroed, hipEvent_t done) {
    if (!s || !x || !y || !params || !stash || !fwd_ws) return fail(LPM_EINVAL, "NULL argument");
    if (s->dtype == LPM_BF16 && !lowp) return fail(LPM_EINVAL, "lowp is NULL for a bf16 stage");
    if (s->loss && (!labels || !loss_accum)) return fail(LPM_EINVAL, "a loss stage needs labels and loss_accum");
    if (misaligned(x) || misaligned(y) || misaligned(params) || misaligned(stash) || misaligned(fwd_ws) ||
        (lowp && misaligned(lowp)))
        return fail(LPM_EALIGN, "device buffers must be 256-byte aligned");
    if (s->loss && (((uintptr_t)labels & 3u) || ((uintptr_t)loss_accum & 3u))) return fail(LPM_EALIGN, "labels / loss_accum must be 4-byte aligned");
    hipStream_t st = (hipStream_t)stream;
    if (s->fwd_counts && !counts_zeroed) LPM_HIP(launch_zero_counts(&fwd_ws, 1, st));
    HeldCall held;
    for (int32_t i = s->first; i < s->last; ++i) {
        const LayerRt& lr = s->Ly(i);
        const lpm_layer& l = lr.d;
        const void* in = tptr(s, l.src, x, y, stash);
        void* outp = const_cast<void*>(tptr(s, i, x, y, stash));
        if (!has_weights(l)) LPM_HIP(run_held(held, st));      // (a contraction's launcher sees to it)
        const bool ends = lr.head_fwd >= 0 ? lr.head_fwd == s->last - 1 : i == s->last - 1 && !lr.headed_fwd;      // its kernel is the pass's last
        StopEvent stop(ends ? done : nullptr, st);
        switch (l.kind) {
            case LPM_CONV:
            case LPM_FC: {
                if (lr.headed_fwd) break;            // done with the pooling it reads
                const void* w = s->dtype == LPM_BF16 ? (const void*)((const char*)lowp + lr.lowp_w_off)
                                                     : (const void*)(params + lr.w_off);
                const float* sc = lr.s_off != NO ? params + lr.s_off : nullptr;
                const float* bi = lr.b_off != NO ? params + lr.b_off : nullptr;
                const void* add = l.add_src != LPM_NONE ? tptr(s, l.add_src, x, y, stash) : nullptr;
                void* pooled = lr.pool_fwd >= 0 ? const_cast<void*>(tptr(s, lr.pool_fwd, x, y, stash)) : nullptr;
                LPM_HIP(launch_conv_fwd(s->dtype, lr.g, in, w, sc, bi, add, (l.flags & LPM_RELU) != 0, outp, fwd_ws, st, pooled, true,
                                        lr.hold_fwd && i + 1 < s->last ? &held : nullptr, &held));
                break;
            }
            case LPM_MAXPOOL2:
                if (lr.pooled_fwd) break;        // stored by the producer's forward kernel
                LPM_HIP(launch_maxpool_fwd(s->dtype, s->m, l.h_in, l.w_in, l.cin, in, outp, st));
                break;
            case LPM_GAP:
                if (lr.head_fwd >= 0) {
                    const LayerRt& fc = s->Ly(lr.head_fwd);
                    LPM_HIP(launch_head_fwd(s->dtype, s->m, l.h_in * l.w_in, l.cin, fc.g.Cout, in, outp,
                                            s->dtype == LPM_BF16 ? (const void*)((const char*)lowp + fc.lowp_w_off) : (const void*)(params + fc.w_off),
                                            fc.b_off != NO ? params + fc.b_off : nullptr, const_cast<void*>(tptr(s, lr.head_fwd, x, y, stash)), st));
                    break;
                }
                LPM_HIP(launch_gap_fwd(s->dtype, s->m, l.h_in * l.w_in, l.cin, in, outp, st));
                break;
            case LPM_ATTN:
                LPM_HIP(launch_attn_fwd(s->dtype, s->m, l.h_in * l.w_in, l.cout, in, outp, st));
                break;
            case LPM_SOFTMAX_CE:
                LPM_HIP(launch_softmax_ce(s->dtype, s->m, l.cin, in, labels, loss_scale, (char*)stash + s->dlogits_off,
                                          loss_accum, st));
                break;
        }
        LPM_HIP(stop.finish());
    }
    return LPM_OK;
}

extern "C" int32_t lpm_stage_backward(lpm_stage* s, const void* x, const void* y, const void* dy, void* dx,
                                      const float* params, const void* lowp, const void* stash, float* grads,
                                      int32_t accumulate, void* bwd_ws, void* stream) {
    return lpm_stage_backward_on(s, x, y, dy, dx, params, lowp, stash, grads, accumulate, bwd_ws, stream, nullptr, 0, LPM_PHASE_DATA | LPM_PHASE_WEIGHTS);
}

// B_{z,j} in two phases.  Data phase (on `stream`): everything the next stage down waits for -- epilogue
// backward, pooling backward, data gradients -- leaving every layer's dz in the backward scratch.  Weight
// phase: the weight (and fused bias) gradients, which nothing in the same pass reads, on `wstream`.
// wstream == stream: after the data phase, no event at all (fully serial); otherwise each weight gradient follows
// its layer's dz through an event and `stream` waits for the last of them (wstream == NULL: the stage's own side
// stream, the contract of lpm_stage_backward).
// phases: LPM_PHASE_DATA | LPM_PHASE_WEIGHTS as described; LPM_PHASE_DATA alone enqueues only the data
// phase; LPM_PHASE_WEIGHTS alone only the weight phase on wstream, with no event -- the caller has ordered
// wstream after the data phase (separate enqueue threads for the two).
// parity (0 / 1) selects the copy of the gradient / dz area in bwd_ws this pass uses.
// data_done (eager): an event for the end of the data phase; *data_point is the event to wait for, data_done or a layer's that
// stands at the same point.  weights_done: an event for the end of the weight phase on wstream.
// wpart (a weight phase by itself): its last group of layers, or the others, each with the sums of its own partial results.
// While `stream` is being captured the weight gradients stay on it and are taken out of its dependency
// frontier instead.
// wstream2 (with wstream, eager only): every other group of weight gradients of the phase runs on this second stream, forked from
// wstream at the start of the phase and joined back into it before the reduction of the partial sums.
int32_t lpm_stage_backward_on(lpm_stage* s, const void* x, const void* y, const void* dy, void* dx,
                              const float* params, const void* lowp, const void* stash, float* grads,
                              int32_t accumulate, void* bwd_ws, void* stream, void* wstream, int32_t parity,
                              int32_t phases, int32_t fc_slot, int32_t fc_flush, int32_t layer_slot, int32_t boundary, void* wstream2,
                              bool counts_zeroed, hipEvent_t data_done, hipEvent_t* data_point, hipEvent_t weights_done, int32_t wpart) {
    if ((boundary & LPM_MASK_DX) && !lpm_stage_can_mask_dx(s)) return fail(LPM_EINVAL, "internal: this stage cannot mask its input gradient");
    if ((boundary & LPM_DY_IS_DZ) && !lpm_stage_takes_dz(s)) return fail(LPM_EINVAL, "internal: this stage needs the gradient of its output");
    if (layer_slot >= LPM_MAX_WINDOW) return fail(LPM_EINVAL, "internal: layer event slot out of range");
    if (fc_slot >= LPM_FC_STAGE_SLOTS || fc_flush > LPM_FC_STAGE_SLOTS) return fail(LPM_EINVAL, "internal: staging slot out of range");
    if (!s || !x || !y || !params || !stash || !grads || !bwd_ws) return fail(LPM_EINVAL, "NULL argument");
    if (!s->loss && !dy) return fail(LPM_EINVAL, "dy is NULL for a stage that is not a loss stage");
    if (s->dtype == LPM_BF16 && !lowp) return fail(LPM_EINVAL, "lowp is NULL for a bf16 stage");
    if (misaligned(x) || misaligned(y) || misaligned(params) || misaligned(stash) || misaligned(grads) ||
        misaligned(bwd_ws) || (dy && misaligned(dy)) || (dx && misaligned(dx)) || (lowp && misaligned(lowp)))
        return fail(LPM_EALIGN, "device buffers must be 256-byte aligned");
    hipStream_t st = (hipStream_t)stream;
    const int32_t first = s->first, last = s->last;
    const bool acc = accumulate != 0;
    char* ws = (char*)bwd_ws;
    void* counts = ws + s->kws_off;              // data-gradient scratch: arrival counts first
    void* kws = ws + s->kws_off + LPM_COUNT_BYTES;
    void* wws = ws + s->wws_off;
    char* gw = ws + (parity ? s->gws_bytes : 0);
    int32_t prc = lpm_stage_prepare(s);
    if (prc) return prc;
    // While the caller's stream is being captured into a graph no second stream is involved: the weight
    // gradient nodes are taken out of the stream's dependency frontier instead (they depend on what came
    // before them and on the previous weight gradient, nothing later depends on them until the join).
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    LPM_HIP(hipStreamIsCapturing(st, &cap));
    const bool deferred = cap == hipStreamCaptureStatusNone;
    const bool do_data = (phases & LPM_PHASE_DATA) != 0, do_weights = (phases & LPM_PHASE_WEIGHTS) != 0;
    if (!deferred && !(do_data && do_weights)) return fail(LPM_EINVAL, "a captured backward pass cannot be split into phases");
    if (wpart != LPM_WEIGHTS_ALL && do_data) return fail(LPM_EINVAL, "internal: a weight phase in parts comes by itself");
    if (!do_data && (!do_weights || !wstream)) return fail(LPM_EINVAL, "internal: bad phase selection");
    if (do_data && s->bwd_counts && !counts_zeroed) LPM_HIP(launch_zero_counts(&counts, 1, st));
    // layer_slot >= 0 (the two phases come as separate calls with the same slot): the data phase records, per weight
    // layer that ends a group, the point in its stream where that layer's output gradient is final, and the weight phase waits for
    // that point before the group's weight gradients instead of for the end of the data phase
    const bool by_layer = layer_slot >= 0 && deferred && (do_data != do_weights);
    // Both phases in one call on two streams: each weight gradient is enqueued on the second stream as soon as the layer's output
    // gradient is final, and runs beside the rest of the data phase (width-48 ResNet at 13 samples, one micro-batch after the
    // other: 3.8 -> 3.5 ms per step; a kernel of such a step is too small to fill the card alone).
    hipStream_t wst = wstream ? (hipStream_t)wstream : s->side;
    const bool beside = deferred && do_data && do_weights && wst != st;
    std::vector<ReduceDesc> red;           // split weight gradients of this pass, reduced in one launch at its end
    // Points of the data phase that other streams wait for: per weight layer "its output gradient is final" (by_layer, beside),
    // and the end.  A point that follows a layer's last kernel with nothing in between is that kernel's stop event.
    const bool points = do_data && (by_layer || beside);
    auto layer_ev = [&](int32_t i) { return s->ev_layer[(size_t)(i - first) * LPM_MAX_WINDOW + (by_layer ? layer_slot : 0)]; };
    hipEvent_t at_point = nullptr;         // the event that stands at the data phase's present end, if one does
    auto point_after = [&](int32_t i) -> hipEvent_t {
        if (!do_data || !deferred) return nullptr;
        for (int32_t k = i - 1; k >= first; --k) {
            const LayerRt& q = s->Ly(k);
            if (has_weights(q.d)) {
                // (a layer without ReLU, scale or shortcut of its own launches nothing ahead of its weight gradient either)
                const bool plain = !(q.d.flags & LPM_RELU) && (!(q.d.flags & LPM_SCALE) || q.dz_unscaled) && q.d.add_src == LPM_NONE;
                if (!q.fused_in && !plain) return nullptr;
                if (points) return q.wg_end ? layer_ev(k) : nullptr;
                return k == first && q.d.src < first && !dx ? data_done : nullptr;
            }
            if (!(q.d.kind == LPM_MAXPOOL2 && q.unpooled)) return nullptr;
        }
        return data_done;
    };
    // bias_g != NULL: the layer's bias gradient is a plain column sum of bias_g that nothing in the data phase needs and its
    // weight-gradient kernel does not make; it runs in the weight phase, ahead of that kernel (scratch: the layer's own area)
    struct WgradJob { const LayerRt* lr; const void* xin; const void* dz; float* wdb; const float* sc; const void* bias_g; float* bias_db; };
    // The weight gradients of a group on stream q.  fc_slot = j >= 0 (of fc_flush = M micro-batches): a layer with staging areas
    // files its operands under slot j and contracts a group of slots at a time; the first group overwrites the accumulator.
    std::vector<WgradJob> jobs;            // the weight phase's layers, last layer first; a group's unless it is launched at the end
    auto run_group = [&](size_t from, size_t to, hipStream_t q) -> hipError_t {
        WgradTask t[LPM_WGRAD_GROUP];
        StageCopy copy[LPM_WGRAD_GROUP];
        ReduceDesc d[LPM_WGRAD_GROUP]{};
        int n = 0, nc = 0;
        hipError_t e;
        for (size_t k = from; k < to; ++k) {
            const WgradJob& j = jobs[k];
            const LayerRt& lr = *j.lr;
            if (j.bias_g && (e = launch_epilogue_bwd(s->dtype, lr.g.rows_out(), lr.d.cout, j.bias_g, nullptr, nullptr, nullptr, nullptr, 0,
                                                     j.bias_db, acc, (char*)wws + lr.wws_off, q)) != hipSuccess) return e;
            if (fc_slot >= 0 && lr.fcs_x_off != NO) copy[nc++] = StageCopy{lr.g, j.xin, j.dz, ws + lr.fcs_x_off, ws + lr.fcs_dz_off};
        }
        if (nc && (e = stage_operands(copy, nc, fc_slot, q)) != hipSuccess) return e;
        for (size_t k = from; k < to; ++k) {
            const WgradJob& j = jobs[k];
            const LayerRt& lr = *j.lr;
            float* dw = grads + lr.w_off;
            void* part = (char*)wws + lr.wws_off;
            if (!(fc_slot >= 0 && lr.fcs_x_off != NO)) {
                t[n++] = WgradTask{lr.g, j.xin, j.dz, dw, j.wdb, j.sc, acc, part};
                continue;
            }
            // Contract in groups of G micro-batches.  One group (G = M) touches dW once, but all of that work then sits
            // behind the last micro-batch, where nothing overlaps it; two groups leave half of it there.  Gradient
            // matrices of 64 MiB and more are bound by their own traffic and keep the single pass.
            const int32_t M = fc_flush;
            const int32_t G = ((size_t)lr.w_count * 4 >= ((size_t)64 << 20)) ? M : std::max(1, (M + 1) / 2);
            if ((fc_slot + 1) % G != 0 && fc_slot != M - 1) continue;
            const int32_t j0 = (fc_slot / G) * G, slots = fc_slot - j0 + 1;
            const char* xs = ws + lr.fcs_x_off + (size_t)j0 * lr.g.rows_in() * lr.g.Cin * 2;
            const char* dzs = ws + lr.fcs_dz_off + (size_t)j0 * lr.g.rows_out() * lr.g.Cout * 2;
            if (fc_staged_ok(lr.g)) {
                if ((e = fc_wgrad_staged(lr.g, xs, dzs, slots, dw, j.wdb, j.sc, j0 > 0, q)) != hipSuccess) return e;
            } else t[n++] = WgradTask{staged_geom(lr.g, slots), xs, dzs, dw, j.wdb, j.sc, j0 > 0, part};
        }
        if (n && (e = launch_wgrad_group(s->dtype, t, n, q, d)) != hipSuccess) return e;
        for (int k = 0; k < n; ++k) if (d[k].splits > 0) red.push_back(d[k]);
        return hipSuccess;
    };
    HeldCall held;                         // a data gradient that waits for the next layer's
    const void* head_dz = nullptr;         // the dz of a headed layer, for the pooling below it
    std::vector<hipGraphNode_t> wtail;     // capture: frontier left by the last weight gradient
    auto frontier = [&](std::vector<hipGraphNode_t>& out) -> hipError_t {
        hipStreamCaptureStatus stt;
        const hipGraphNode_t* deps = nullptr;
        size_t nd = 0;
        hipError_t e = hipStreamGetCaptureInfo_v2(st, &stt, nullptr, nullptr, &deps, &nd);
        if (e == hipSuccess) out.assign(deps, deps + nd);
        return e;
    };

    // gradient buffer of every tensor, and whether it already holds a contribution
    std::vector<void*> G((size_t)(last - first + 1), nullptr);
    std::vector<char> have((size_t)(last - first + 1), 0);
    auto gi = [&](int32_t t) { return (size_t)(t - (first - 1)); };
    // whether layer i's backward kernel writes the dz of the layer that made tensor t
    auto writes_dz = [&](int32_t i, int32_t t) { return t >= first && s->Ly(t).fused_in && s->Ly(t).fused_by == i; };
    for (int32_t t = first; t < last; ++t)
        if (s->T(t).loc == LOC_STASH) G[gi(t)] = gw + s->T(t).g_off;
    G[gi(first - 1)] = dx;
    int32_t top = last - 1;
    if (s->loss) {
        top = last - 2;
        G[gi(top)] = const_cast<char*>((const char*)stash) + s->dlogits_off;
    } else {
        G[gi(top)] = const_cast<void*>(dy);
    }
    have[gi(top)] = 1;

    for (int32_t i = top; i >= first; --i) {
        const LayerRt& lr = s->Ly(i);
        const lpm_layer& l = lr.d;
        const void* g = G[gi(i)];
        if (!have[gi(i)]) return fail(LPM_ESHAPE, "internal: tensor %d has no consumer", i);
        const bool want_src = (l.src >= first) || (dx != nullptr);
        // a data gradient that waits goes with this layer's, or before anything else is launched
        if (held.held && !(has_weights(l) && want_src && lr.unpool_of < 0)) {
            LPM_HIP(run_held(held, st));
            at_point = nullptr;
        }
        switch (l.kind) {
            case LPM_CONV:
            case LPM_FC: {
                const void* yout = tptr(s, i, x, y, stash);
                const float* sc = lr.s_off != NO ? params + lr.s_off : nullptr;
                const bool relu = (l.flags & LPM_RELU) != 0;
                float* dbias = lr.b_off != NO ? grads + lr.b_off : nullptr;
                const bool bias_in_wgrad = dbias && bias_in_wgrad_ok(s->dtype, lr);
                const void* dz = g;
                const void* bias_g = nullptr;
                if (lr.fused_in || (i == s->t_out && (boundary & LPM_DY_IS_DZ))) {
                    // written by the consumer's backward kernel; or the next stage applied this layer's ReLU mask to what it handed down
                    dz = lr.fused_in ? (const void*)(gw + lr.dz_off) : g;
                    if (dbias && !bias_in_wgrad) bias_g = dz;
                    if (!lr.fused_in && lr.shortcut_is_dz) {
                        G[gi(l.add_src)] = const_cast<void*>(dz);      // (only read from here on)
                        have[gi(l.add_src)] = 1;
                    }
                } else {
                    void* gadd = nullptr;
                    int gadd_acc = 0;
                    if (l.add_src != LPM_NONE && ((l.add_src >= first) || dx != nullptr)) {
                        gadd = G[gi(l.add_src)];
                        gadd_acc = have[gi(l.add_src)];
                        have[gi(l.add_src)] = 1;
                    }
                    const bool need_dz = relu || (sc && !lr.dz_unscaled);
                    if (!need_dz && !gadd && dbias && !bias_in_wgrad) {
                        bias_g = g;
                    } else if (need_dz || gadd || (dbias && !bias_in_wgrad)) {
                        at_point = nullptr;
                        if (do_data) LPM_HIP(launch_epilogue_bwd(s->dtype, lr.g.rows_out(), l.cout, g, relu ? yout : nullptr, lr.dz_unscaled ? nullptr : sc,
                                                    need_dz ? (void*)(gw + lr.dz_off) : nullptr, gadd, gadd_acc,
                                                    bias_in_wgrad ? nullptr : dbias, acc, kws, st));
                        if (need_dz) dz = gw + lr.dz_off;
                    }
                }
                if (points && lr.wg_end && at_point != layer_ev(i)) {
                    LPM_HIP(hipEventRecord(layer_ev(i), st));
                    at_point = layer_ev(i);
                }
                float* wdb = bias_in_wgrad ? dbias : nullptr;
                // where the gradient w.r.t. this layer's input goes: the producer's dz (fused) or the tensor's gradient
                void* gsrc = nullptr;
                int gsrc_acc = 0;
                const void* gmask = nullptr;
                const float* gmscale = nullptr;
                const bool want = (l.src >= first) || (dx != nullptr);
                UnpoolDesc unpool{};
                if (lr.unpool_of >= 0) {
                    // this layer's input is a max-pooling output nobody else reads: route the data gradient through the
                    // pooling to where the pooling backward would have written (the same choices as in the pooling case below)
                    const int32_t p = lr.unpool_of, q = s->Ly(p).d.src;
                    have[gi(p)] = 1;
                    if (q >= first || dx != nullptr) {
                        unpool.pool_x = tptr(s, q, x, y, stash);
                        unpool.dst = G[gi(q)];
                        unpool.accumulate = have[gi(q)];
                        if (writes_dz(p, q)) {
                            const LayerRt& pr = s->Ly(q);
                            unpool.dst = gw + pr.dz_off;
                            unpool.accumulate = 0;
                            unpool.mask = (pr.d.flags & LPM_RELU) != 0;
                            unpool.mscale = (pr.s_off != NO && !pr.dz_unscaled) ? params + pr.s_off : nullptr;
                        } else if (q == first - 1 && p == s->mask_layer && (boundary & LPM_MASK_DX)) {
                            unpool.mask = 1;
                        }
                        have[gi(q)] = 1;
                    }
                }
                DgradSide side{};
                bool use_side = false;
                if (want && lr.unpool_of < 0) {
                    if (writes_dz(i, l.src)) {
                        const LayerRt& pr = s->Ly(l.src);
                        gsrc = gw + pr.dz_off;
                        gmask = (pr.d.flags & LPM_RELU) ? tptr(s, l.src, x, y, stash) : nullptr;
                        gmscale = (pr.s_off != NO && !pr.dz_unscaled) ? params + pr.s_off : nullptr;
                        if (pr.fused_side) {
                            // the producer sits in a residual block: what its shortcut users have already put into its output
                            // gradient is added, and the masked sum is also the gradient of the producer's own shortcut
                            use_side = true;
                            side.earlier = have[gi(l.src)] ? G[gi(l.src)] : nullptr;
                            const int32_t a = pr.d.add_src;
                            if (pr.shortcut_is_dz) {
                                G[gi(a)] = gsrc;
                                have[gi(a)] = 1;
                            } else if (a != LPM_NONE && a >= first && s->Ly(a).via_shortcut) {
                                side.shortcut = gw + s->Ly(a).dz_off;           // the projection's dz
                                side.shortcut_scale = s->Ly(a).dz_unscaled ? nullptr : params + s->Ly(a).s_off;
                                have[gi(a)] = 1;
                            } else if (a != LPM_NONE && (a >= first || dx != nullptr)) {
                                side.shortcut = G[gi(a)];
                                side.shortcut_acc = have[gi(a)];
                                have[gi(a)] = 1;
                            }
                        }
                    } else {
                        gsrc = G[gi(l.src)];
                        gsrc_acc = have[gi(l.src)];
                        if (i == s->mask_layer && (boundary & LPM_MASK_DX)) gmask = x;      // ReLU backward of the previous stage's last layer
                    }
                    have[gi(l.src)] = 1;
                }
                const void* xin = tptr(s, l.src, x, y, stash);
                jobs.push_back(WgradJob{&lr, xin, dz, wdb, lr.dz_unscaled ? sc : nullptr, bias_g, bias_g ? dbias : nullptr});
                if (beside && lr.wg_end) {
                    LPM_HIP(hipStreamWaitEvent(wst, layer_ev(i), 0));
                    LPM_HIP(run_group(0, jobs.size(), wst));
                    jobs.clear();
                } else if (!deferred && lr.wg_end) {
                    std::vector<hipGraphNode_t> before;
                    LPM_HIP(frontier(before));
                    if (!wtail.empty())       // weight gradients share one scratch area: keep them in a chain
                        LPM_HIP(hipStreamUpdateCaptureDependencies(st, wtail.data(), wtail.size(), hipStreamAddCaptureDependencies));
                    LPM_HIP(run_group(0, jobs.size(), st));      // (the same kernels and sums as an eager pass, a reduction per group)
                    if (!red.empty()) LPM_HIP(launch_reduce_batch(red.data(), (int)red.size(), st));
                    red.clear();
                    jobs.clear();
                    LPM_HIP(frontier(wtail));
                    LPM_HIP(hipStreamUpdateCaptureDependencies(st, before.data(), before.size(), hipStreamSetCaptureDependencies));
                }
                if (want) {
                    const void* w = s->dtype == LPM_BF16 ? (const void*)((const char*)lowp + lr.lowp_w_off)
                                                         : (const void*)(params + lr.w_off);
                    const void* wt = (s->dtype == LPM_BF16 && lr.lowp_wt_off != NO)
                                         ? (const void*)((const char*)lowp + lr.lowp_wt_off) : nullptr;
                    const hipEvent_t ev = point_after(i);
                    StopEvent stop(ev, st);
                    if (lr.unpool_of >= 0) {
                        if (do_data && unpool.dst) LPM_HIP(launch_conv_dgrad(s->dtype, lr.g, dz, w, wt, nullptr, 0, nullptr, nullptr, counts, st, &unpool,
                                                                             nullptr, lr.dz_unscaled ? sc : nullptr, true));
                    } else if (lr.headed_bwd) {
                        head_dz = dz;            // (the pooling's kernel goes on from there)
                    } else if (do_data) {
                        const bool hold = lr.hold_bwd && i > first && (s->Ly(i - 1).d.src >= first || dx);
                        LPM_HIP(launch_conv_dgrad(s->dtype, lr.g, dz, w, wt, gsrc, gsrc_acc, gmask, gmscale, counts, st, nullptr,
                                                  use_side ? &side : nullptr, lr.dz_unscaled ? sc : nullptr, true, hold ? &held : nullptr, &held));
                    }
                    LPM_HIP(stop.finish());
                    at_point = ev;
                }
                break;
            }
            case LPM_MAXPOOL2:
            case LPM_GAP:
                if (lr.unpooled) break;          // done by the consumer's data gradient
                if (want_src || lr.head_bwd >= 0) {  // (a head's kernel stores the pooled tensor's gradient, too)
                    void* gsrc = G[gi(l.src)];
                    int gsrc_acc = have[gi(l.src)];
                    const void* gmask = nullptr;
                    const float* gmscale = nullptr;
                    if (writes_dz(i, l.src)) {
                        const LayerRt& pr = s->Ly(l.src);
                        gsrc = gw + pr.dz_off;
                        gsrc_acc = 0;
                        gmask = (pr.d.flags & LPM_RELU) ? tptr(s, l.src, x, y, stash) : nullptr;
                        gmscale = (pr.s_off != NO && !pr.dz_unscaled) ? params + pr.s_off : nullptr;
                        if (pr.shortcut_is_dz) {
                            G[gi(pr.d.add_src)] = gsrc;
                            have[gi(pr.d.add_src)] = 1;
                        }
                    } else if (i == s->mask_layer && (boundary & LPM_MASK_DX)) {
                        gmask = x;
                    }
                    const hipEvent_t ev = point_after(i);
                    StopEvent stop(ev, st);
                    if (do_data && l.kind == LPM_MAXPOOL2)
                        LPM_HIP(launch_maxpool_bwd(s->dtype, s->m, l.h_in, l.w_in, l.cin, tptr(s, l.src, x, y, stash),
                                                   tptr(s, i, x, y, stash), g, gsrc, gsrc_acc, gmask != nullptr, gmscale, st));
                    else if (do_data && lr.head_bwd >= 0) {
                        const LayerRt& fc = s->Ly(lr.head_bwd);
                        LPM_HIP(launch_head_bwd(s->dtype, s->m, l.h_in * l.w_in, l.cin, fc.g.Cout, head_dz,
                                                s->dtype == LPM_BF16 ? (const void*)((const char*)lowp + fc.lowp_w_off) : (const void*)(params + fc.w_off),
                                                const_cast<void*>(g), gsrc, gsrc_acc, gmask, gmscale, st));
                    } else if (do_data)
                        LPM_HIP(launch_gap_bwd(s->dtype, s->m, l.h_in * l.w_in, l.cin, g, gsrc, gsrc_acc, gmask, gmscale, st));
                    LPM_HIP(stop.finish());
                    at_point = ev;
                    have[gi(l.src)] = 1;
                }
                break;
            case LPM_ATTN:
                if (want_src) {
                    const hipEvent_t ev = point_after(i);
                    StopEvent stop(ev, st);
                    if (do_data)
                        LPM_HIP(launch_attn_bwd(s->dtype, s->m, l.h_in * l.w_in, l.cout, tptr(s, l.src, x, y, stash), g, G[gi(l.src)],
                                                have[gi(l.src)], kws, st));
                    LPM_HIP(stop.finish());
                    at_point = ev;
                    have[gi(l.src)] = 1;
                }
                break;
            default:
                return fail(LPM_ESHAPE, "internal: unexpected layer kind in backward");
        }
    }
    if (!wtail.empty())
        LPM_HIP(hipStreamUpdateCaptureDependencies(st, wtail.data(), wtail.size(), hipStreamAddCaptureDependencies));
    if (do_data && data_done) {
        if (!at_point) {
            LPM_HIP(hipEventRecord(data_done, st));
            at_point = data_done;
        }
        *data_point = at_point;
    }
    if (do_weights && (beside || !jobs.empty())) {
        size_t from = 0, to = jobs.size();
        if (wpart != LPM_WEIGHTS_ALL) {
            size_t last = to - 1;                 // the first layer of the last group
            while (last > 0 && !jobs[last - 1].lr->wg_end) --last;
            (wpart == LPM_WEIGHTS_LAST ? from : to) = last;
        }
        hipStream_t wst2 = (wstream && wstream2 && deferred && to - from > (size_t)WG_LAYERS) ? (hipStream_t)wstream2 : nullptr;
        if (wst2 == wst) wst2 = nullptr;
        if (wst2) {        // ordered after everything the phase's stream holds (the previous micro-batch's reduction reads the areas written now)
            LPM_HIP(hipEventRecord(s->ev_w2_fork, wst));
            LPM_HIP(hipStreamWaitEvent(wst2, s->ev_w2_fork, 0));
        }
        int groups = 0;
        for (size_t k = from; k < to; ++k) {
            if (!jobs[k].lr->wg_end) continue;
            hipStream_t q = (wst2 && (groups++ & 1)) ? wst2 : wst;
            if (by_layer)
                LPM_HIP(hipStreamWaitEvent(q, s->ev_layer[(size_t)(jobs[k].lr - &s->lay[0]) * LPM_MAX_WINDOW + layer_slot], 0));
            LPM_HIP(run_group(from, k + 1, q));
            from = k + 1;
        }
        if (wst2) {
            LPM_HIP(hipEventRecord(s->ev_w2_join, wst2));
            LPM_HIP(hipStreamWaitEvent(wst, s->ev_w2_join, 0));
        }
        const hipEvent_t end = beside ? s->ev_join : weights_done;
        StopEvent stop(end, wst);
        if (!red.empty()) LPM_HIP(launch_reduce_batch(red.data(), (int)red.size(), wst));
        LPM_HIP(stop.finish());
        if (beside) LPM_HIP(hipStreamWaitEvent(st, s->ev_join, 0));        // the caller's stream is ordered after every weight gradient
    } else if (do_weights && weights_done) {
        LPM_HIP(hipEventRecord(weights_done, wst));
    }
    return LPM_OK;
}

bool lpm_stage_can_mask_dx(const lpm_stage* s) { return s && s->mask_layer >= 0; }

bool lpm_stage_takes_dz(const lpm_stage* s) {
    if (!s || s->loss) return false;
    const int32_t i = s->t_out;
    if (i != s->last - 1) return false;
    const LayerRt& lr = s->Ly(i);
    const lpm_layer& l = lr.d;
    return has_weights(l) && (l.flags & LPM_RELU) && (!(l.flags & LPM_SCALE) || lr.dz_unscaled) && (l.add_src == LPM_NONE || lr.shortcut_is_dz);
}

extern "C" int32_t lpm_stage_update(lpm_stage* s, float* params, void* lowp, float* grads, float* momentum,
                                    float lr_, float mu, int32_t zero_grads, void* stream) {
    return lpm_stage_update_to(s, params, params, lowp, grads, momentum, lr_, mu, zero_grads, stream);
}

// U with the new weights written to another buffer than the one they are read from (params_out may equal
// params_in): the asynchronous update keeps two versions of a stage's weights.  Frozen scales are not touched.
int32_t lpm_stage_update_to(lpm_stage* s, const float* params_in, float* params, void* lowp, float* grads, float* momentum,
                            float lr_, float mu, int32_t zero_grads, void* stream) {
    if (!s || !params_in || !params || !grads || !momentum) return fail(LPM_EINVAL, "NULL argument");
    if (s->dtype == LPM_BF16 && !lowp) return fail(LPM_EINVAL, "lowp is NULL for a bf16 stage");
    if (misaligned(params_in) || misaligned(params) || misaligned(grads) || misaligned(momentum) || (lowp && misaligned(lowp)))
        return fail(LPM_EALIGN, "device buffers must be 256-byte aligned");
    hipStream_t st = (hipStream_t)stream;
    if (s->n_trainable == 0) return LPM_OK;
    const std::vector<UpdateSeg> d = update_segments(s, params, lowp);
    LPM_HIP(launch_sgd(d.data(), (int)d.size(), params_in, params, s->dtype == LPM_BF16 ? (uint16_t*)lowp : nullptr, grads, momentum, lr_, mu,
                       zero_grads, st));
    if (s->dtype == LPM_BF16) LPM_HIP(transpose_copies(s, params, lowp, true, st));
    return LPM_OK;
}

extern "C" int32_t lpm_stage_update_adam(lpm_stage* s, float* params, void* lowp, float* grads, float* m1, float* m2,
                                         float lr_, float beta1, float beta2, float eps, int32_t step, int32_t zero_grads,
                                         void* stream) {
    if (!s || !params || !grads || !m1 || !m2) return fail(LPM_EINVAL, "NULL argument");
    if (s->dtype == LPM_BF16 && !lowp) return fail(LPM_EINVAL, "lowp is NULL for a bf16 stage");
    if (step < 1 || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps >= 0.f))
        return fail(LPM_EINVAL, "Adam needs step >= 1, 0 <= beta < 1 and eps >= 0");
    if (misaligned(params) || misaligned(grads) || misaligned(m1) || misaligned(m2) || (lowp && misaligned(lowp)))
        return fail(LPM_EALIGN, "device buffers must be 256-byte aligned");
    if (s->n_trainable == 0) return LPM_OK;
    // bias corrections in double on the host: 1 - beta^t loses digits in float for beta close to 1
    const float inv_c1 = (float)(1.0 / (1.0 - std::pow((double)beta1, (double)step)));
    const float inv_c2 = (float)(1.0 / (1.0 - std::pow((double)beta2, (double)step)));
    hipStream_t st = (hipStream_t)stream;
    const std::vector<UpdateSeg> d = update_segments(s, params, lowp);
    LPM_HIP(launch_adam(d.data(), (int)d.size(), params, s->dtype == LPM_BF16 ? (uint16_t*)lowp : nullptr, grads, m1, m2, lr_, beta1, beta2,
                        eps, inv_c1, inv_c2, zero_grads, st));
    if (s->dtype == LPM_BF16) LPM_HIP(transpose_copies(s, params, lowp, true, st));
    return LPM_OK;
}
