"""The update kernels store the transposed bf16 copies that the data gradients read: after an update every low-precision byte is
what lpm_stage_sync_lowp makes of the new parameters, at channel counts that fill no 64-wide tile, with and without biases and
scales, for filters that need the copies and layers that do not."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _layers():
    out, src = [], -1
    for cin, cout, k, stride, bias, scale in [(4, 8, 3, 1, True, False), (8, 72, 3, 1, False, True), (72, 136, 1, 1, True, False), (136, 64, 3, 2, False, True),
                                              (64, 24, 5, 1, True, True), (24, 6, 3, 1, True, False), (6, 16, 3, 1, False, False)]:
        h = 8 if len(out) <= 3 else 4
        out.append(dict(kind="conv", cin=cin, cout=cout, kh=k, kw=k, stride=stride, pad=k // 2, h_in=h, w_in=h, relu=True, bias=bias,
                        scale=scale, src=src, add_src=None, cut_after=False))
        src = len(out) - 1
    return out


@pytest.mark.parametrize("rule", ["sgd", "adam"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_update_keeps_every_copy(rule, dtype):
    import torch
    import paper_2207_11019_amd as lpm
    dt = lpm.BF16 if dtype == "bf16" else lpm.F32
    st = lpm.Stage(_layers(), 0, 7, 2, dt)
    gen = torch.Generator().manual_seed(11)
    n, total = st.grad_bytes // 4, st.param_bytes // 4
    p = torch.rand(total, generator=gen) + 0.25
    g, v, v2 = (torch.rand(n, generator=gen) * s for s in (1.0, 0.1, 0.01))
    dp, dg, dv, dv2 = p.cuda(), g.cuda(), v.cuda(), v2.cuda()
    lowp = [torch.zeros(max(st.lowp_bytes, 256), dtype=torch.uint8, device="cuda") for _ in range(2)] if dt == lpm.BF16 else [None, None]
    if rule == "sgd":
        st.update(dp, lowp[0], dg, dv, 0.05, 0.9, True)
        v = 0.9 * v + g
        p[:n] -= 0.05 * v
    else:
        st.update_adam(dp, lowp[0], dg, dv, dv2, 0.05, 0.9, 0.99, 1e-8, 3, True)
        v, v2 = 0.9 * v + 0.1 * g, 0.99 * v2 + 0.01 * g * g
        p[:n] -= 0.05 * (v / (1 - 0.9 ** 3)) / ((v2 / (1 - 0.99 ** 3)).sqrt() + 1e-8)
        np.testing.assert_allclose(dv2.cpu().numpy(), v2.numpy(), rtol=1e-5, atol=1e-6)
    if dt == lpm.BF16:
        st.sync_lowp(dp, lowp[1])
    torch.cuda.synchronize()
    np.testing.assert_allclose(dp.cpu().numpy(), p.numpy(), rtol=1e-5, atol=1e-6)
    np.testing.assert_allclose(dv.cpu().numpy(), v.numpy(), rtol=1e-5, atol=1e-6)
    assert not dg.any()
    if dt == lpm.BF16:
        assert lowp[0].any() and torch.equal(lowp[0], lowp[1])
