"""ob_lamb_ratios_apply_hist on lists whose tiles keep v_frozen of most spans in LDS: those that fit on the device
at once only that way, and those of 24 to 70 million parameters.  Against the oracle bit for bit, with layers and
chunks that end anywhere; with momentum scaling and without."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.test_gpu_parity import _need_gpu, finish, run_trajectory  # noqa: E402
from workloads.shapes import ParamList, padded_len  # noqa: E402

pytestmark = pytest.mark.gpu

LISTS = {
    "one_round": ([7_813_632, 131_072, 256] + [262_144, 256] * 9 + [100_003, 1, 262_145, 700_001], 8),
    "rounds": ([6_000_003, 77, 5 * 8192 - 1, 0, 4_194_304, 1023, 3_300_001, 1, 7_000_000, 4_000_007], 7),
}


@pytest.mark.parametrize("use_k", [False, True])
@pytest.mark.parametrize("name", list(LISTS))
def test_variance_history_in_lds(name, use_k):
    _need_gpu()
    import paper_2104_06069_amd as ob
    sizes, W = LISTS[name]
    pl = ParamList(name, [(f"t{i}", s) for i, s in enumerate(sizes)])
    n_pad = padded_len(pl.N, W)
    cfg = dict(name=name, plist=pl, W=W, n_pad=n_pad, n_c=n_pad // W, grad="student_t3", steps=4, server_chunk=W - 1,
               use_k=use_k)
    ref, dev, stats = run_trajectory(cfg, 7, packed=True, fused=True, warm_state=True, deferred=True,
                                     deferred_variance=2, check_every=2)
    assert stats["scale_ulp_steps"] == 0 and stats["word_mismatch_steps"] == 0
    for k in ("x", "m", "v_fresh", "err_worker", "err_server", "r_prev", "coeff_c"):
        assert np.array_equal(dev.get(k), ref.t[k]), k
    ob.ob_lamb_profile_enable(dev.ctx, True)
    dev.begin_step()
    dev.ratios_apply(1e-3)
    assert "ratios_apply_hist" in set(ob.ob_lamb_profile_read(dev.ctx))
    finish(dev)
