"""Lists of few tiles, where the ratio pass outside the 8192-element tiles runs in the launch of the kernel with the
per-layer barrier (ob_lamb_ratios_apply_hist) and its segments arrive at that barrier: layers of one element and of
none, layers that only small tiles hold, in one tile or several, layers with one listed tile, with and without a
remainder, layers too large for the barrier, with a remainder and wholly in large tiles.  Against the oracle, bit for
bit; which launches a list takes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.test_gpu_parity import _need_gpu, finish, run_trajectory  # noqa: E402
from workloads.shapes import ParamList, padded_len  # noqa: E402

pytestmark = pytest.mark.gpu

T = 8192
LISTS = {   # sizes, workers, the limit of the barrier kernel's layers, ratio pass in the same launch
    "tiny_layers": ([1, 0, 1, 700, 1, 1, 3000, 0, 400 * T + 5, 1023, 1, 5000, 12 * T, 0], 3, None, True),
    "one_tile": ([T, 2 * T, T - 1, 1, T, 20_000, 500 * T], 1, None, True),
    "large_alone": ([1100 * T, 1100 * T, 3 * T], 1, None, True),
    "large_rest": ([77, 1100 * T + 9, 1, 300 * T], 5, None, True),
    "lowered": ([40 * T + 3, 5 * T + 1, 70 * T, 9 * T, 64], 2, 8, True),
    "all_inside": ([600 * T, 8 * T, 300 * T], 1, None, True),
    "many_tiles": ([1000 * T, 77] * 5 + [140 * T], 1, None, False),
}


@pytest.mark.parametrize("use_k", [False, True])
@pytest.mark.parametrize("name", list(LISTS))
def test_ratio_pass_in_the_barrier_kernels_launch(name, use_k):
    _need_gpu()
    import paper_2104_06069_amd as ob
    sizes, W, cap, one = LISTS[name]
    pl = ParamList(name, [(f"t{i}", s) for i, s in enumerate(sizes)])
    n_pad = padded_len(pl.N, W)
    cfg = dict(name=name, plist=pl, W=W, n_pad=n_pad, n_c=n_pad // W, grad="student_t3", steps=4, server_chunk=W - 1,
               use_k=use_k)
    ref, dev, stats = run_trajectory(cfg, 4, two_pass=True, packed=True, fused=True, warm_state=True, deferred=True,
                                     deferred_variance=2, check_every=2, fused_max_tiles=cap)
    assert stats["scale_ulp_steps"] == 0 and stats["word_mismatch_steps"] == 0
    for k in ("x", "m", "v_fresh", "err_worker", "err_server", "r_prev", "coeff_c"):
        assert np.array_equal(dev.get(k), ref.t[k]), k
    ob.ob_lamb_profile_enable(dev.ctx, True)
    dev.begin_step()
    dev.ratios_apply(1e-3)
    names = set(ob.ob_lamb_profile_read(dev.ctx))
    assert names & {"ratios_apply_hist", "ratios_apply_hist_lds"} and ("ratios_pass" in names) == (not one)
    finish(dev)
