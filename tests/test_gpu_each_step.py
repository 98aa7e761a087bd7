"""ob_lamb_ratios_apply with the momentum in its 1-bit form on lists that take ob_lamb_ratios_apply_hist's kernels with no
history: the variance array is up to date after every step, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.test_gpu_hard_values import config  # noqa: E402
from tests.test_gpu_parity import _need_gpu, assert_close, finish, kernels_of, start_pair  # noqa: E402
from tests.test_gpu_rest_update import step  # noqa: E402

pytestmark = pytest.mark.gpu

T = 8192
LISTS = {   # sizes, workers, the limit of the barrier kernel's layers, momentum scaling, 16-bit copy, a kernel that the list takes
    "rest_in_launch": ([900, 300 * T + 5, 1, 0, 3 * T], 3, 1 << 20, True, torch.bfloat16, "ratios_apply_hist"),
    "lds": ([130 * T] * 10 + [7], 1, 1 << 20, False, None, "ratios_apply_hist_lds"),
    "resident": ([200 * T, 900, 50 * T + 1], 2, 1 << 20, False, None, "ratios_apply_resident"),
    "trail": ([215 * T + 11] * 5 + [8 * T] * 40 + [62 * T + 1] * 22, 5, 8, False, None, "ratios_trail"),
}


@pytest.mark.parametrize("name", list(LISTS))
def test_steps(name):
    _need_gpu()
    import paper_2104_06069_amd as ob
    sizes, W, cap, use_k, lp, kernel = LISTS[name]
    cfg = config(name, sizes, W, use_k)
    st, ref, dev = start_pair(cfg, seed=61, two_pass=True, packed=True, fused=True, fused_max_tiles=cap, deferred=True)
    if lp is not None:
        dev.x_lp = torch.zeros(dev.n_pad, device=dev.device, dtype=lp)
    ob.ob_lamb_profile_enable(dev.ctx, True)
    for t in range(4):
        step(cfg, st, ref, dev, t, lambda g: dev.step(g, 1e-3))
        for k in ("x", "r_prev", "coeff_c"):
            assert_close(dev.get(k), ref.t[k], f"step {t}: {k}")
        assert_close(dev.t["v_fresh"].cpu().numpy(), ref.t["v_fresh"], f"step {t}: the array itself")
        if lp is not None:
            assert torch.equal(dev.x_lp[:dev.N].view(torch.int16), dev.t["x"][:dev.N].to(lp).view(torch.int16))
    assert kernel in kernels_of(dev)
    finish(dev)


@pytest.mark.parametrize("period", [0, 2])
def test_quotient_of_two_negative_variances(period):
    """No step makes one, but what the ratio of such a state was, it stays: their quotient is positive and counts."""
    _need_gpu()
    cfg = config("negative", [300 * T + 5, 3 * T, 40 * T], 1)
    st, ref, dev = start_pair(cfg, seed=62, two_pass=True, packed=True, fused=True, fused_max_tiles=1 << 20, deferred=True,
                              deferred_variance=period)
    for t in range(2):
        step(cfg, st, ref, dev, t, lambda g: dev.step(g, 1e-3))
    ref.t["v_fresh"][:] = 2 * ref.t["v_frozen"]  # every other ratio below what the clips raise it to ...
    ref.t["v_frozen"][7 * T] = -1.08
    ref.t["v_fresh"][7 * T] = -1.0               # ... and this one the largest of its layer
    ref.t["r_prev"][:] = 1.0
    for k in ("v_fresh", "v_frozen", "r_prev"):
        dev.load_state({k: ref.t[k]})
    step(cfg, st, ref, dev, 2, lambda g: dev.step(g, 1e-3))
    assert ref.t["r_prev"][0] > 1.05
    for k in ("r_prev", "coeff_c"):
        assert_close(dev.get(k), ref.t[k], k)
    finish(dev)
