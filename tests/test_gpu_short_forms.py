"""The shorter square root, quotient and maximum of quotients of the kernels that ob_lamb_ratios_apply and ob_lamb_ratios_apply_hist take
beyond the smallest lists, against IEEE binary32 arithmetic (numpy): the same bits for every mantissa of v_frozen, over all
exponents that they take, at the ends of that range and beyond it."""
import numpy as np
import pytest

from tests.refstep import HYPER

pytestmark = pytest.mark.gpu

f32 = np.float32
T = 8192
EDGE = [0.0, 1e-45, 1.1754942e-38, 2.0 ** -96, np.nextafter(f32(2.0 ** -96), f32(0)), np.nextafter(f32(2.0 ** -96), f32(1)), 1e-20,
        2.0 ** 59, 2.0 ** 60, np.nextafter(f32(2.0 ** 60), f32(np.inf)), 3e38, np.inf, np.nan]
# sizes, workers, fused_max_tiles, kernels of a call that rewrites the variance / has a history (256 CUs)
LISTS = {
    "barrier": ([1 << 22] * 4, 1, 0, {"ratios_apply_resident"}, {"ratios_apply_hist"}),
    "in_lds": ([1 << 22] * 3, 1, 0, {"ratios_apply_hist_lds"}, {"ratios_apply_hist_lds"}),
    # many elements outside the 8192-element tiles, most of them in 1024-element ones inside one layer
    "rest_update": ([3 * T + 5000 + i for i in range(130)], 2, 1 << 20, {"ratios_apply_hist"}, {"ratios_apply_hist"}),
    "trail": ([1200 * T, 77, 900 * T + 5], 3, 8, None, {"ratios_trail"}),
    "big_hist": ([2000 * T + 300, 3 * T], 2, 8, None, {"ratios_big_hist"}),
}


def v_values(kind, n, rng):
    if kind == "every_mantissa":      # [1, 4): both parities of the exponent; every one of them in lists of 2^24 elements or more
        step = max(1, (1 << 24) // n)
        return (np.arange(n, dtype=np.uint32) * np.uint32(step) % np.uint32(1 << 24) + np.uint32(0x3f800000)).view(f32)
    if kind == "every_exponent":      # [2^-96, 2^60]
        return rng.integers(0x0f800000, 0x5d800001, n, dtype=np.uint32).view(f32)
    v = np.abs(rng.standard_normal(n, dtype=f32)) * f32(1e-4) + f32(1e-8)
    if kind == "edges":               # in a tenth of the wavefronts' parts, so that both forms run
        at = rng.integers(0, n // 4096, n // 40960) * 4096 + rng.integers(0, 256, n // 40960)
        v[at] = np.array(EDGE, f32)[rng.integers(0, len(EDGE), at.size)]
    return v


CASES = [("barrier", kind, scale, eta, period, False) for period in (0, 2)
         for kind, scale, eta in [("every_mantissa", 1e-4, 1e-6), ("every_exponent", 1e-4, 1e-6), ("edges", 1e-4, 1e-6), ("edges", 3e-4, 0.0),
                                  ("edges", 1e-30, 1e-6), ("edges", 0.0, 1e-6), ("near_ties", 2e-4, 2.0 ** -22)]]
CASES += [(name, kind, scale, 1e-6, period, use_k) for name in list(LISTS)[1:] for period in (0, 2) if period or LISTS[name][3]
          for kind, scale, use_k in [("every_mantissa", 1e-4, False), ("edges", 3e-4, True)]]


@pytest.mark.parametrize("name,kind,scale,eta,period,use_k", CASES)
def test_update_and_ratio_are_ieee_arithmetic(name, kind, scale, eta, period, use_k):
    import torch
    import paper_2104_06069_amd as ob
    from paper_2104_06069_amd.step import DeviceStep
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the lists are ones for 256 CUs")
    sizes, W, cap = LISTS[name][:3]
    kernels = LISTS[name][4 if period else 3]
    L, n = len(sizes), sum(sizes)
    off = np.concatenate([[0], np.cumsum(sizes)])
    per_layer = lambda a: np.repeat(np.asarray(a, f32), sizes)
    rng = np.random.default_rng(5)
    hyper = dict(HYPER, eta=eta)
    k = rng.uniform(0.25, 4.0, L).astype(f32) if use_k else np.ones(L, f32)
    ds = DeviceStep(off, W, 0, packed_momentum=True, fused_apply=True, deferred_variance=period, mom_scale=k if use_k else None,
                    fused_max_tiles=cap, **hyper)
    vz = v_values(kind, n, rng)
    # layers whose largest quotient lies below the lower clip bound, inside and above the window
    with np.errstate(over="ignore"):
        vf = vz * per_layer(np.resize([2.5, 1.02, 0.95, 0.5], L))
    if kind == "near_ties":           # quotients within a few units of the last place of each other
        vf = (vf.view(np.uint32) + rng.integers(0, 3, n, dtype=np.uint32)).view(f32)
    x = rng.standard_normal(n, dtype=f32) * f32(0.02)
    if kind.startswith("every"):
        x[:] = 0
    bits = [rng.integers(0, 256, ds.n_pad // 8, dtype=np.uint8) for _ in range(2)]      # previous, new momentum
    s_prev, s_new = f32(scale * 1.1), f32(scale)
    c_avg = np.resize(np.array([0.7, 1.3, 1.0, 0.9], f32), L)
    pad = lambda a: np.concatenate([a, np.zeros(ds.n_pad - n, f32)])
    ds.load_state(dict(x=pad(x), v_fresh=pad(vf), v_frozen=pad(vz), c_avg=c_avg))
    ds.m_is_packed = True
    ds._cur = 1
    for pair, b, s in ((0, bits[0], s_prev), (1, bits[1], s_new)):
        ds._pa[pair].copy_(torch.from_numpy(b.view(np.int32)))
        ds._ss[pair].fill_(float(s))
    lr = 1e-2
    ob.ob_lamb_profile_enable(ds.ctx, True)
    ds.ratios_apply(lr)
    ran = set(ob.ob_lamb_profile_read(ds.ctx))
    got = {key: ds.get(key)[:m] for key, m in (("x", n), ("r_prev", L), ("coeff_c", L), ("v_fresh", n))}
    ob.ob_lamb_check_device_status(ds.ctx, ds.stream)
    ds.close()
    assert kernels <= ran and not (ran - kernels) & {"ratios_trail", "ratios_big_hist"}, ran
    assert name != "rest_update" or not ran & {"ratios_pass", "decompress_apply"}, ran
    with np.errstate(all="ignore"):
        b1, b2 = f32(hyper["beta1"]), f32(hyper["beta2"])
        omb1, omb2 = f32(1) - b1, f32(1) - b2
        s_k, bm = s_new / k, b1 * (s_prev / k)
        t = [omb2 * (g * g) for g in ((s_k - bm) / omb1, (s_k + bm) / omb1)]
        old, new = (np.unpackbits(b, bitorder="little")[:n] for b in bits)
        v = b2 * vf + np.where(old != new, per_layer(t[1]), per_layer(t[0]))
        q = vz / v
        r = np.fmax(np.fmax.reduceat(q, off[:-1]), f32(0))
        r = np.minimum(np.maximum(r, (f32(1) - f32(hyper["r_threshold"])) * f32(1)), (f32(1) + f32(hyper["r_threshold"])) * f32(1))
        r = np.minimum(np.maximum(r, f32(hyper["r_min"])), f32(hyper["r_max"]))
        c = r * c_avg
        u = np.where(new == 1, per_layer(s_k), -per_layer(s_k)) / (np.sqrt(vz) + f32(eta))
        want = x - per_layer(f32(lr) * c) * u
    for key, w in (("r_prev", r), ("coeff_c", c), ("v_fresh", v), ("x", want)):
        assert w.dtype == f32
        same = (got[key].view(np.uint32) == w.view(np.uint32)) | (np.isnan(got[key]) & np.isnan(w))
        assert same.all(), (key, int((~same).sum()), int(np.argmin(same)))
