"""Layers on both sides of the size from which a step with a 16-bit copy and the variance's history takes the ratio pass and the update of large layers
in two kernels: the same bits as without a copy, where both are one kernel up to a larger share of such layers, and the copy is x rounded."""
import numpy as np
import pytest

from tests.refstep import HYPER

pytestmark = pytest.mark.gpu

T = 8192
LINE = 2 * 6144      # tiles


@pytest.mark.parametrize("tiles,two_kernels", [(LINE, False), (LINE + 2, True)])     # (one tile of the unaligned layer is not whole)
@pytest.mark.parametrize("period", [0, 2])
def test_same_bits_with_and_without_a_copy(tiles, two_kernels, period):
    import torch
    import paper_2104_06069_amd as ob
    from paper_2104_06069_amd.step import DeviceStep
    W = 1
    offsets = np.concatenate([[0], np.cumsum([tiles * T, 1000, tiles * T, 300 * T + 7, 4000 * T])])
    steps = [DeviceStep(offsets, W, 0, packed_momentum=True, fused_apply=True, deferred_error=True, deferred_variance=period, x_lp_dtype=lp, **HYPER)
             for lp in (torch.bfloat16, None)]
    gen = torch.Generator(device="cuda").manual_seed(3)
    n_pad, n = steps[0].n_pad, int(offsets[-1])
    rand = lambda s: torch.randn(n_pad, generator=gen, device="cuda").mul_(s)
    x, v = rand(0.02), rand(1e-4).abs_().add_(1e-8)
    x[n:] = 0
    v[n:] = 0
    words = [torch.randint(-2 ** 31, 2 ** 31, (steps[0].packed_all.numel(),), generator=gen, device="cuda", dtype=torch.int32) for _ in range(5)]
    names = []
    for ds in steps:
        ds.load_state(dict(x=x, m=torch.zeros_like(x), v_fresh=v, v_frozen=v, c_avg=np.full(5, 1.25, np.float32)))
        ds.m_is_packed, ds._cur = True, 1
        ds._pa[0].copy_(words[4])
        ds._ss[0].fill_(2e-3)
        for t in range(4):
            if t:
                ds.begin_step()
            ds.packed_all.copy_(words[t])
            ds.server_scales.fill_((1 + t) * 1e-3)
            ob.ob_lamb_profile_enable(ds.ctx, True)
            ds.ratios_apply(1e-2)
            names.append(set(ob.ob_lamb_profile_read(ds.ctx)))
            ob.ob_lamb_profile_enable(ds.ctx, False)
        ds.check_status()
    for t, got in enumerate(names):
        with_copy = t < 4
        if two_kernels and with_copy and period:
            assert "ratios_trail" not in got and {"ratios_big_hist", "decompress_apply"} <= got, (t, got)
        elif period:
            assert "ratios_trail" in got and "ratios_big_hist" not in got, (t, got)
    a, b = steps
    for k in ("x", "v_fresh", "r_prev", "coeff_c"):
        assert torch.equal(a.t[k], b.t[k]), k
    assert torch.equal(a.x_lp[:n], a.t["x"][:n].to(torch.bfloat16))
    assert not torch.equal(a.t["x"], x)
    for ds in steps:
        ds.close()
