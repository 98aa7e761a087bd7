"""The LAMB step's shorter square root and quotient against IEEE binary32 arithmetic (numpy), with the coefficients that the device
formed: the same bits for every mantissa of the variance, at the ends of the range that they take and beyond it."""
import numpy as np
import pytest

from tests.refstep import HYPER

pytestmark = pytest.mark.gpu

f32 = np.float32
T = 8192
V_EDGE = [0.0, 1e-45, 1.1754942e-38, 2.0 ** -96, np.nextafter(f32(2.0 ** -96), f32(0)), 2.0 ** 60, np.nextafter(f32(2.0 ** 60), f32(np.inf)), 3e38,
          np.inf, np.nan]
M_EDGE = [0.0, -0.0, 1e-45, -1e-38, 2.0 ** -80, np.nextafter(f32(2.0 ** -80), f32(0)), -2.0 ** 40, np.nextafter(f32(2.0 ** 40), f32(np.inf)), np.inf,
          np.nan]
LISTS = {"warmup_small": ([1 << 19] * 4, 0), "warmup_resident": ([1 << 21] * 4, 0), "warmup_trail": ([70 * T] * 3 + [66 * T + 256], 8)}


@pytest.mark.parametrize("wd,eta", [(0.0, 1e-6), (0.01, 2.0 ** -22), (0.0, 0.0)])
@pytest.mark.parametrize("kind", ["every_mantissa", "edges"])
@pytest.mark.parametrize("kernel", list(LISTS))
def test_update_is_ieee_arithmetic(kernel, kind, wd, eta):
    import torch
    import paper_2104_06069_amd as ob
    from paper_2104_06069_amd.step import DeviceStep
    sizes, cap = LISTS[kernel]
    off = np.concatenate([[0], np.cumsum(sizes)])
    n = int(off[-1])
    rng = np.random.default_rng(9)
    hyper = dict(HYPER, eta=eta, weight_decay=wd)
    ds = DeviceStep(off, 1, 0, fused_max_tiles=cap, **hyper)
    b1, b2 = f32(hyper["beta1"]), f32(hyper["beta2"])
    g = (rng.standard_normal(n, dtype=f32) * f32(1e-3)).astype(f32)
    m = (rng.standard_normal(n, dtype=f32) * f32(1e-4)).astype(f32)
    x = (rng.standard_normal(n, dtype=f32) * f32(0.02)).astype(f32)
    if kind == "every_mantissa":
        # (no gradient: the variance is beta2 times these)
        v = (np.arange(n, dtype=np.uint32) * np.uint32((1 << 24) // n) + np.uint32(0x3f800000)).view(f32)
        g[:] = 0
    else:                   # in some of the wavefronts' parts, so that both forms run
        v = np.abs(rng.standard_normal(n, dtype=f32)) * f32(1e-8)
        at = rng.integers(0, n // 4096, n // 20480) * 4096 + rng.integers(0, 256, n // 20480)
        v[at] = np.array(V_EDGE, f32)[rng.integers(0, len(V_EDGE), at.size)]
        m[at] = np.array(M_EDGE, f32)[rng.integers(0, len(M_EDGE), at.size)]
        g[at] = 0
    ds.load_state(dict(x=x, m=m, v_fresh=v))
    ob.ob_lamb_profile_enable(ds.ctx, True)
    lr = 1e-2
    ds.warmup_step(torch.from_numpy(np.concatenate([g, np.zeros(ds.n_pad - n, f32)])).to(ds.device), lr)
    got = {k: ds.get(k)[:n] for k in ("x", "m", "v_fresh")}
    c = ds.get("coeff_c")
    assert kernel in ob.ob_lamb_profile_read(ds.ctx)
    ds.close()
    with np.errstate(all="ignore"):
        mn = b1 * m + (f32(1) - b1) * g
        vn = b2 * v + (f32(1) - b2) * (g * g)
        u = mn / (np.sqrt(vn) + f32(eta))
        if wd:
            u = u + f32(wd) * x
        want = x - np.repeat(f32(lr) * c, sizes) * u
    for k, w in (("m", mn), ("v_fresh", vn), ("x", want)):
        same = (got[k].view(np.uint32) == w.view(np.uint32)) | (np.isnan(got[k]) & np.isnan(w))
        assert same.all(), (k, int((~same).sum()), int(np.argmin(same)))
