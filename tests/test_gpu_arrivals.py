"""Barriers whose arrivals are counted in one level or two: layers at the edges of the rule (256 and 257 tiles of the
barrier kernels, groups of 32 with a remainder of one, several such layers side by side, chunk ends that cut tiles
short), in the compression step, the LAMB step and their one-launch forms, against the oracle; every step counts
from the generation that the one before left."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.refstep import HYPER, RefStep  # noqa: E402
from tests.test_gpu_parity import DeviceStep, _need_gpu, assert_close, finish, run_trajectory  # noqa: E402
from workloads import Streams, gradient, init_state  # noqa: E402
from workloads.shapes import ParamList, padded_len  # noqa: E402

pytestmark = pytest.mark.gpu

T = 8192
LISTS = {   # sizes, workers
    "edges": ([256 * T, 257 * T, 289 * T, 3 * T], 1),
    "cut": ([321 * T + 5, 77, 288 * T, 1023, 600 * T], 7),
    "one_launch": ([270_001, 5, 2_200_000, 77], 3),     # tiles of 4096 elements, more than 512 of one layer
}


def _cfg(name, steps):
    sizes, W = LISTS[name]
    pl = ParamList(name, [(f"t{i}", s) for i, s in enumerate(sizes)])
    n_pad = padded_len(pl.N, W)
    return dict(name=name, plist=pl, W=W, n_pad=n_pad, n_c=n_pad // W, grad="student_t3", steps=steps, server_chunk=W - 1,
                use_k=False)


@pytest.mark.parametrize("name", list(LISTS))
def test_compression_steps(name):
    _need_gpu()
    ref, dev, stats = run_trajectory(_cfg(name, 5), 5, packed=True, fused=True, warm_state=True, deferred=True,
                                     deferred_variance=2, check_every=2)
    assert stats["scale_ulp_steps"] == 0 and stats["word_mismatch_steps"] == 0
    for k in ("x", "m", "v_fresh", "err_worker", "err_server", "r_prev", "coeff_c"):
        assert np.array_equal(dev.get(k), ref.t[k]), k
    finish(dev)


@pytest.mark.parametrize("name", list(LISTS))
def test_lamb_steps(name):
    _need_gpu()
    cfg, st = _cfg(name, 3), Streams(12)
    hyper = dict(HYPER, c_min=1e-4)
    ref = RefStep(cfg["plist"].offsets, cfg["W"], cfg["W"] - 1, **hyper)
    dev = DeviceStep(cfg["plist"].offsets, cfg["W"], cfg["W"] - 1, **hyper)
    ref.load_state(init_state(st, cfg))
    dev.load_state(ref.t)
    for t in range(3):
        g = gradient(st, cfg, t)
        ref.warmup_step(g, 1e-3)
        dev.warmup_step(torch.from_numpy(g).to(dev.device), 1e-3)
        for k in ("m", "v_fresh", "x", "coeff_c", "c_avg"):
            assert_close(dev.get(k), ref.t[k], f"step {t}: {k}")
    finish(dev)


def test_chunk_barrier():
    """The compression kernel with a chunk barrier, chunks of 257 and 289 of its 16384-element tiles."""
    _need_gpu()
    for tiles in (257, 289):
        n = tiles * 16384
        pl = ParamList("chunk", [("a", n), ("b", n - 1)])
        n_pad = padded_len(pl.N, 2)
        cfg = dict(name="chunk", plist=pl, W=2, n_pad=n_pad, n_c=n_pad // 2, grad="student_t3", steps=2, server_chunk=1,
                   use_k=False)
        ref, dev, stats = run_trajectory(cfg, 2, warm_state=True)
        assert stats["scale_ulp_steps"] == 0 and stats["word_mismatch_steps"] == 0
        assert np.array_equal(dev.get("err_worker"), ref.t["err_worker"])
        finish(dev)
