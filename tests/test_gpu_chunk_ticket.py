"""The scales of ob_lamb_compress_local and ob_lamb_server_reduce (deferred errors) with and without a launch of
their own, at the edges of the rules that choose: 64 and 65 tiles of a chunk (one or two levels of arrivals), 256
and 257, and the most of the worker's tiles for which its workgroups arrive.  Scales, words and state against the
oracle, and which launches ran (256 CUs)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.test_gpu_parity import _need_gpu, finish, run_trajectory  # noqa: E402
from workloads import gradient, Streams  # noqa: E402
from workloads.shapes import ParamList, padded_len  # noqa: E402

pytestmark = pytest.mark.gpu

#        workers, elements of a chunk, scale without a launch: worker, server
CASES = [(3, 64 * 1024, True, True), (3, 64 * 1024 + 256, True, True),
         (24, 256 * 1024, True, True), (25, 256 * 1024, False, False), (2, 256 * 1024 + 256, False, False),
         (160, 64 * 1024 - 256, True, True), (161, 64 * 1024, False, True)]


@pytest.mark.parametrize("W,n_c,worker,server", CASES)
def test_scales_with_and_without_a_launch(W, n_c, worker, server):
    _need_gpu()
    import paper_2104_06069_amd as ob
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        worker = server = None      # (the rules count the device's workgroup slots)
    n = W * n_c - 77
    pl = ParamList("ticket", [("a", n // 3), ("b", 5), ("c", n - n // 3 - 5)])
    assert padded_len(pl.N, W) == W * n_c
    cfg = dict(name="ticket", plist=pl, W=W, n_pad=W * n_c, n_c=n_c, grad="student_t3", steps=3, server_chunk=W - 1,
               use_k=False)
    ref, dev, stats = run_trajectory(cfg, 3, packed=True, fused=True, warm_state=True, deferred=True, check_every=1)
    assert stats["scale_ulp_steps"] == 0 and stats["word_mismatch_steps"] == 0
    ob.ob_lamb_profile_enable(dev.ctx, True)
    dev.begin_step()
    dev.step(torch.from_numpy(gradient(Streams(1), cfg, 9)).to(dev.device), 1e-3)
    took = set(ob.ob_lamb_profile_read(dev.ctx))
    if worker is not None:
        assert ("chunk_scale" not in took) == worker, took
        assert ("server_scale" not in took) == server, took
    finish(dev)
