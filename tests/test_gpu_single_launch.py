"""Lists whose tiles all fit on the device at once take ob_lamb_ratios_apply(_hist) and
ob_lamb_warmup_step as one launch each (k_ratios_apply_small, k_warmup_small) with tiles of 1024, 2048 or
4096 elements.  Against the oracle at the sizes where that can go wrong: tensors that end one element
before, at and after a tile's edge, empty and 1-element tensors, hundreds of tensors in one tile, the
smallest list, the largest of each tile size and the first one beyond them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.refstep import HYPER, RefStep  # noqa: E402
from tests.test_gpu_parity import DeviceStep, _need_gpu, assert_close, finish, run_trajectory  # noqa: E402
from workloads import Streams, gradient, init_state  # noqa: E402
from workloads.shapes import ParamList, padded_len  # noqa: E402

pytestmark = pytest.mark.gpu

EDGES = [1023, 1, 1024, 1025, 0, 2048, 4095, 4097, 0, 0, 3 * 8192 + 5, 1, 2, 3] + [5] * 300 + [8192, 2 * 8192 - 1]
LISTS = {
    "one": ([1], 1),
    "edges": (EDGES, 3),
    "edges_many_chunks": (EDGES, 61),
    "u1": (EDGES + [900_000, 64, 600_000], 2),            # 1.58e6 elements
    "u1_many": (EDGES + [115_001] * 13, 2),               # ... in tensors of few tiles
    "one_large": ([1_600_000], 2),                        # one tensor that meets every tile
    "u2": (EDGES + [1_300_000, 64, 500_000, 7], 5),       # 1.88e6
    "u4": (EDGES + [700_001, 64, 1_300_000, 1_000_000], 4),   # 3.08e6
    "u4_scaled": ([4097, 3, 8191, 1000] * 150 + [1_100_003], 3),   # 3.09e6: momentum scaling in tiles of several tensors
    "beyond": (EDGES + [1_700_001, 64, 2_300_000], 4),    # 4.08e6: the launches of the larger lists
    "one_in_whole_tiles": ([3_200_000], 4),               # ... a tensor that the barrier kernels take as a whole, too
}
LARGER = ("beyond", "one_in_whole_tiles")


def _cfg(name):
    sizes, W = LISTS[name]
    pl = ParamList(name, [(f"t{i}", s) for i, s in enumerate(sizes)])
    n_pad = padded_len(pl.N, W)
    return dict(name=name, plist=pl, W=W, n_pad=n_pad, n_c=n_pad // W, grad="student_t3", steps=3,
                server_chunk=W - 1, use_k=(name in ("edges", "u2", "u4_scaled")))


@pytest.mark.parametrize("period", [0, 3])
@pytest.mark.parametrize("name,max_tiles", [(n, None) for n in LISTS] + [("edges", 1 << 20), ("u2", 1 << 20)])
def test_ratios_apply_in_one_launch(name, max_tiles, period):
    """Bit for bit the oracle's state after every step; max_tiles: a limit (here a huge one) on the tiles
    per layer asks for the launches of the larger lists, on the same list."""
    _need_gpu()
    import paper_2104_06069_amd as ob
    cfg = _cfg(name)
    ref, dev, stats = run_trajectory(cfg, 7, packed=True, fused=True, warm_state=True, deferred=True,
                                     deferred_variance=period, fused_max_tiles=max_tiles, check_every=1)
    assert stats["scale_ulp_steps"] == 0 and stats["word_mismatch_steps"] == 0
    for k in ("x", "m", "v_fresh", "err_worker", "err_server", "r_prev", "coeff_c"):
        assert np.array_equal(dev.get(k), ref.t[k]), k
    ob.ob_lamb_profile_enable(dev.ctx, True)
    dev.begin_step()
    dev.ratios_apply(1e-3)
    took = set(ob.ob_lamb_profile_read(dev.ctx))
    assert ("ratios_apply_small" in took) == (name not in LARGER and max_tiles is None), took
    finish(dev)


@pytest.mark.parametrize("wd", [0.0, 0.01])
@pytest.mark.parametrize("name", list(LISTS))
def test_lamb_step_in_one_launch(name, wd):
    _need_gpu()
    import paper_2104_06069_amd as ob
    cfg = _cfg(name)
    pl, st = cfg["plist"], Streams(5)
    hyper = dict(HYPER, weight_decay=wd, c_min=1e-4)
    ref = RefStep(pl.offsets, cfg["W"], cfg["server_chunk"], **hyper)
    dev = DeviceStep(pl.offsets, cfg["W"], cfg["server_chunk"], **hyper)
    ref.load_state(init_state(st, cfg))
    dev.load_state(ref.t)
    ob.ob_lamb_profile_enable(dev.ctx, True)
    for t in range(3):
        g = gradient(st, cfg, t)
        ref.warmup_step(g, 1e-3)
        dev.warmup_step(torch.from_numpy(g).to(dev.device), 1e-3)
        for k in ("m", "v_fresh", "x", "coeff_c", "c_avg"):
            assert_close(dev.get(k), ref.t[k], f"step {t}: {k}")
    took = set(ob.ob_lamb_profile_read(dev.ctx))
    assert ("warmup_small" in took) == (name not in LARGER), took
    finish(dev)


# One tensor that meets every tile: its 1563 tiles of 1024 elements arrived at one counter, one after the other, in
# 27 us where the launches of the larger lists take 15 to 17.  Tensors that share tiles, with momentum scaling: 29 us
# against 24, most of it each element's own divisions by its tensor's coefficient.  One tensor in whole 8192-element
# tiles, all that the barrier kernel takes: 23 us against 20, twice as many arrivals.
@pytest.mark.parametrize("call", ["warmup_step", "ratios_apply"])
@pytest.mark.parametrize("sizes,W", [([900_000], 2), ([1_600_000], 2), ([90_000] * 24, 8), ([3_200_000], 4)])
def test_one_launch_is_no_slower_than_those_of_larger_lists(sizes, W, call):
    """Times of the kernels alone, in turn."""
    _need_gpu()
    import paper_2104_06069_amd as ob
    devs, us = [], [[], []]
    for max_tiles in (None, 1 << 20):
        dev = DeviceStep(np.concatenate([[0], np.cumsum(sizes)]), W, 0, two_pass=True, packed_momentum=True, fused_apply=True,
                         deferred_error=True, fused_max_tiles=max_tiles,
                         mom_scale=np.linspace(0.5, 2.0, len(sizes)).astype(np.float32), **HYPER)
        for k in ("x", "v_fresh", "v_frozen"):
            dev.t[k].fill_(1e-3)
        dev.m_is_packed = (call == "ratios_apply")      # (a state of constants)
        ob.ob_lamb_profile_enable(dev.ctx, True)
        devs.append(dev)
    g = torch.full((devs[0].n_pad,), 1e-3, device=devs[0].device)
    for rep in range(40):
        for dev, t in zip(devs, us):
            if call == "warmup_step":
                dev.warmup_step(g, 1e-3)
            else:
                dev.begin_step()
                dev.ratios_apply(1e-3)
            prof = ob.ob_lamb_profile_read(dev.ctx)
            t.append(sum(ms for ms, _ in prof.values()))
    one, several = (float(np.median(t[10:])) for t in us)
    assert one <= 1.1 * several, (one, several)
    for dev in devs:
        finish(dev)
