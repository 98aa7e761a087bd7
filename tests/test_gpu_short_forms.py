"""The shorter square root, quotient and maximum of quotients of the barrier kernels against IEEE binary32 arithmetic (numpy): the
same bits for every mantissa of v_frozen, at the ends of the range that they take and beyond it."""
import numpy as np
import pytest

from tests.refstep import HYPER

pytestmark = pytest.mark.gpu

f32 = np.float32
EDGE = [0.0, 1e-45, 1.1754942e-38, 2.0 ** -96, np.nextafter(f32(2.0 ** -96), f32(0)), np.nextafter(f32(2.0 ** -96), f32(1)), 1e-20,
        2.0 ** 59, 2.0 ** 60, np.nextafter(f32(2.0 ** 60), f32(np.inf)), 3e38, np.inf, np.nan]


def v_values(kind, n, rng):
    if kind == "every_mantissa":      # [1, 4): both parities of the exponent
        return np.arange(0x3f800000, 0x3f800000 + n, dtype=np.uint32).view(f32)
    v = np.abs(rng.standard_normal(n, dtype=f32)) * f32(1e-4) + f32(1e-8)
    if kind == "edges":               # in a tenth of the wavefronts' parts, so that both forms run
        at = rng.integers(0, n // 4096, n // 40960) * 4096 + rng.integers(0, 256, n // 40960)
        v[at] = np.array(EDGE, f32)[rng.integers(0, len(EDGE), at.size)]
    return v


@pytest.mark.parametrize("period", [0, 2])
@pytest.mark.parametrize("kind,scale,eta", [("every_mantissa", 1e-4, 1e-6), ("edges", 1e-4, 1e-6), ("edges", 3e-4, 0.0),
                                            ("edges", 1e-30, 1e-6), ("edges", 0.0, 1e-6), ("near_ties", 2e-4, 2.0 ** -22)])
def test_update_and_ratio_are_ieee_arithmetic(kind, scale, eta, period):
    import torch
    from paper_2104_06069_amd.step import DeviceStep
    n_l, L = 1 << 22, 4
    n = n_l * L
    rng = np.random.default_rng(5)
    hyper = dict(HYPER, eta=eta)
    ds = DeviceStep(np.arange(L + 1) * n_l, 1, 0, packed_momentum=True, fused_apply=True, deferred_variance=period, **hyper)
    vz = v_values(kind, n, rng)
    # layers whose largest quotient lies below the lower clip bound, inside and above the window
    with np.errstate(over="ignore"):
        vf = vz * np.repeat(np.array([2.5, 1.02, 0.95, 0.5], f32), n_l)
    if kind == "near_ties":           # quotients within a few units of the last place of each other
        vf = (vf.view(np.uint32) + rng.integers(0, 3, n, dtype=np.uint32)).view(f32)
    x = rng.standard_normal(n, dtype=f32) * f32(0.02)
    if kind == "every_mantissa":
        x[:] = 0
    bits = [rng.integers(0, 256, n // 8, dtype=np.uint8) for _ in range(2)]      # previous, new momentum
    s_prev, s_new = f32(scale * 1.1), f32(scale)
    c_avg = np.array([0.7, 1.3, 1.0, 0.9], f32)
    ds.load_state(dict(x=x, v_fresh=vf, v_frozen=vz, c_avg=c_avg))
    ds.m_is_packed = True
    ds._cur = 1
    for pair, b, s in ((0, bits[0], s_prev), (1, bits[1], s_new)):
        ds._pa[pair].copy_(torch.from_numpy(b.view(np.int32)))
        ds._ss[pair].fill_(float(s))
    lr = 1e-2
    ds.ratios_apply(lr)
    got = {k: ds.get(k) for k in ("x", "r_prev", "coeff_c", "v_fresh")}
    ds.close()
    with np.errstate(all="ignore"):
        b1, b2 = f32(hyper["beta1"]), f32(hyper["beta2"])
        omb1, omb2 = f32(1) - b1, f32(1) - b2
        bm = b1 * s_prev
        t = [omb2 * (g * g) for g in ((s_new - bm) / omb1, (s_new + bm) / omb1)]
        old, new = (np.unpackbits(b, bitorder="little") for b in bits)
        v = b2 * vf + np.where(old != new, t[1], t[0]).astype(f32)
        q = (vz / v).reshape(L, n_l)
        r = np.fmax(np.fmax.reduce(q, axis=1), f32(0))
        r = np.minimum(np.maximum(r, (f32(1) - f32(hyper["r_threshold"])) * f32(1)), (f32(1) + f32(hyper["r_threshold"])) * f32(1))
        r = np.minimum(np.maximum(r, f32(hyper["r_min"])), f32(hyper["r_max"]))
        c = r * c_avg
        u = np.where(new == 1, s_new, -s_new).astype(f32) / (np.sqrt(vz) + f32(eta))
        want = x - np.repeat(f32(lr) * c, n_l) * u
    for k, w in (("r_prev", r), ("coeff_c", c), ("v_fresh", v), ("x", want)):
        same = (got[k].view(np.uint32) == w.view(np.uint32)) | (np.isnan(got[k]) & np.isnan(w))
        assert same.all(), (k, int((~same).sum()), int(np.argmin(same)))
