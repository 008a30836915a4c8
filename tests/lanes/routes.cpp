// Looks into the library: which geometries the implicit-GEMM kernels take (op 0: forward, 1: data gradient), for tests of sizes no test
// can hold, which heads share a kernel, calls that wait for the next one's launch where no network makes them wait, and launches behind a stop event.
#include "lpm_internal.h"
#include "stage.h"

namespace lpm {
bool mfma_fwd_ok(int dtype, const ConvGeom& g);
bool mfma_dgrad_ok(int dtype, const ConvGeom& g);
}  // namespace lpm

extern "C" int lanes_takes(int op, int dtype, const lpm_conv_geom* q) {
    lpm::ConvGeom g{q->m, q->h, q->w, q->cin, (q->h + 2 * q->pad - q->kh) / q->stride + 1, (q->w + 2 * q->pad - q->kw) / q->stride + 1,
                    q->cout, q->kh, q->kw, q->stride, q->pad};
    return op == 0 ? lpm::mfma_fwd_ok(dtype, g) : lpm::mfma_dgrad_ok(dtype, g);
}

// whether an average pooling over hw positions of c channels shares a kernel with the layer of n outputs behind it
extern "C" int lanes_head(int dtype, int m, int hw, int c, int n, int fwd) { return lpm::head_ok(dtype, m, hw, c, n, fwd != 0); }

// layer i's contraction waits (forward, backward) although what follows need not be one that it can share a launch with
extern "C" void lanes_hold(lpm_stage* s, int i, int fwd, int bwd) {
    s->Ly(i).hold_fwd = fwd != 0;
    s->Ly(i).hold_bwd = bwd != 0;
}

// One contraction (op 0: forward, a = x; 1: data gradient, a = dz, w transposed) in a stage's order of sums, launched by itself -> lone, and twice in one
// launch, which goes in chunks across taps -> pair, pair2.
extern "C" int lanes_lone_and_paired(int op, const lpm_conv_geom* q, const void* a, const void* w, void* lone, void* pair, void* pair2, void* ws) {
    lpm::ConvGeom g{q->m, q->h, q->w, q->cin, q->h + 2 * q->pad - q->kh + 1, q->w + 2 * q->pad - q->kw + 1, q->cout, q->kh, q->kw, 1, q->pad};
    g.D = q->d; g.Kd = q->kd; g.pad_d = q->pad_d; g.Do = q->d + 2 * q->pad_d - q->kd + 1;
    auto run = [&](void* out, lpm::HeldCall* hold, lpm::HeldCall* with) {
        return op == 0 ? lpm::launch_conv_fwd(LPM_BF16, g, a, w, nullptr, nullptr, nullptr, 0, out, ws, nullptr, nullptr, false, hold, with)
                       : lpm::launch_conv_dgrad(LPM_BF16, g, a, w, w, out, 0, nullptr, nullptr, ws, nullptr, nullptr, nullptr, nullptr, false, hold, with);
    };
    lpm::HeldCall h;
    if (run(lone, nullptr, nullptr) != hipSuccess || run(pair, &h, nullptr) != hipSuccess || !h.held) return -1;
    return run(pair2, nullptr, &h) == hipSuccess && !h.held ? 0 : -1;
}

// two calls held in one place: what the second returns
extern "C" int lanes_hold_twice() {
    const lpm::ConvGeom g{2, 8, 8, 64, 8, 8, 64, 3, 3, 1, 1};
    lpm::HeldCall h;
    void* p = (void*)4096;
    if (lpm::launch_conv_fwd(LPM_BF16, g, p, p, nullptr, nullptr, nullptr, 0, p, p, nullptr, nullptr, true, &h) != hipSuccess || !h.held) return -1;
    return lpm::launch_conv_fwd(LPM_BF16, g, p, p, nullptr, nullptr, nullptr, 0, p, p, nullptr, nullptr, true, &h);
}

// the data gradient of an average pooling and the layer over its channels, m samples, under a stop event: launches that the event does not stand behind
extern "C" long lanes_behind_head(int dtype, int m, int hw, int c, int n) {
    hipEvent_t e = nullptr;
    (void)hipEventCreate(&e);
    const long before = lanes::launched();
    void* p = (void*)4096;
    {
        lpm::StopEvent stop(e, nullptr);
        if (lpm::launch_head_bwd(dtype, m, hw, c, n, p, p, p, p, 0, nullptr, nullptr, nullptr) != hipSuccess || stop.finish() != hipSuccess) return -1;
    }
    const long after = lanes::launched(), left = e->records == 1 && after > before ? after - e->behind : -1;
    (void)hipEventDestroy(e);
    return left;
}

// a forward pass with an event for its end: whether the event came with the pass's last kernel (1), after it as a packet of its own (0), or neither (-1)
extern "C" int lanes_forward_done(lpm_stage* s) {
    hipEvent_t e = nullptr;
    (void)hipEventCreate(&e);
    void* p = (void*)4096;
    const int32_t rc = lpm_stage_forward_on(s, p, p, nullptr, nullptr, (float*)p, p, p, p, 1.f, nullptr, true, e);
    const int how = rc == LPM_OK && e->records == 1 && e->behind == lanes::launched() ? e->with_kernel : -1;
    (void)hipEventDestroy(e);
    return how;
}
