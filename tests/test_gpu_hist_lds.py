"""ob_lamb_ratios_apply_hist on lists whose tiles keep v_frozen of most spans in LDS: those that fit on the device
at once only that way, and those of two to six rounds of the device's workgroups.  Against the oracle bit for bit,
with layers and chunks that end anywhere; with momentum scaling and without.  Which form a list takes, at the edges
of the rule."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.refstep import HYPER  # noqa: E402
from tests.test_gpu_parity import DeviceStep, _need_gpu, finish, run_trajectory  # noqa: E402
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
    assert "ratios_apply_hist_lds" in set(ob.ob_lamb_profile_read(dev.ctx))
    finish(dev)


# tiles of 8192 elements per tensor (one chunk: all of them inside their tensor), the form on 256 CUs
EDGES = [([640, 640], False), ([641, 640], True), ([768, 768], True), ([769, 768], False), ([853, 853, 853], False),
         ([854, 853, 853], True), ([768] * 12, True), ([768] * 11 + [769], False),
         # 24 to 70 M parameters of which few are listed (the first tensor is too large)
         ([3000, 1, 400], False), ([4000, 800, 800], False)]


@pytest.mark.parametrize("tiles,in_lds", EDGES)
def test_form_by_listed_tiles(tiles, in_lds):
    _need_gpu()
    import paper_2104_06069_amd as ob
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the edges are those of 256 CUs")
    offsets = np.concatenate([[0], np.cumsum(8192 * np.array(tiles))])
    dev = DeviceStep(offsets, 1, 0, two_pass=True, packed_momentum=True, fused_apply=True, deferred_error=True, deferred_variance=2,
                     **HYPER)
    assert ob.ob_lamb_fused_params(dev.ctx) == 8192 * sum(t for t in tiles if t < 1016)
    dev.m_is_packed = True      # (a state of zeros)
    ob.ob_lamb_profile_enable(dev.ctx, True)
    dev.begin_step()
    dev.ratios_apply(1e-3)
    took = set(ob.ob_lamb_profile_read(dev.ctx))
    assert ("ratios_apply_hist_lds" in took, "ratios_apply_hist" in took) == (in_lds, not in_lds), took
    finish(dev)
