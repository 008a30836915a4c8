// Which geometries the implicit-GEMM kernels take (op 0: forward, 1: data gradient), for tests of sizes no test can hold.
#include "lpm_internal.h"

namespace lpm {
bool mfma_fwd_ok(int dtype, const ConvGeom& g);
bool mfma_dgrad_ok(int dtype, const ConvGeom& g);
}  // namespace lpm

extern "C" int lanes_takes(int op, int dtype, const lpm_conv_geom* q) {
    lpm::ConvGeom g{q->m, q->h, q->w, q->cin, (q->h + 2 * q->pad - q->kh) / q->stride + 1, (q->w + 2 * q->pad - q->kw) / q->stride + 1,
                    q->cout, q->kh, q->kw, q->stride, q->pad};
    return op == 0 ? lpm::mfma_fwd_ok(dtype, g) : lpm::mfma_dgrad_ok(dtype, g);
}
