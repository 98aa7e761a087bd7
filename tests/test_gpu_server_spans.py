"""ob_lamb_server_reduce with one, two and four 1024-element spans to a tile, at the edges of the rule (few workers,
long chunks) and with chunk ends that cut the last tile short: errors in deferred form (scale from the arrivals) and
in plain form (three kernels), against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.test_gpu_parity import _need_gpu, finish, run_trajectory  # noqa: E402
from workloads.shapes import ParamList, padded_len  # noqa: E402

pytestmark = pytest.mark.gpu

T = 1024
#        workers, elements of a chunk
CASES = [(1, 4096 * T), (2, 4096 * T + 256), (2, 4097 * T + 768), (2, 4095 * T), (1, 2048 * T + 1024 - 256), (7, 2047 * T),
         (7, 2048 * T + 512), (3, 4099 * T)]


@pytest.mark.parametrize("deferred", [True, False])
@pytest.mark.parametrize("W,n_c", CASES)
def test_server_reduce(W, n_c, deferred):
    _need_gpu()
    n = W * n_c - 77
    pl = ParamList("server", [("a", n // 3), ("b", 5), ("c", n - n // 3 - 5)])
    assert padded_len(pl.N, W) == W * n_c
    cfg = dict(name="server", plist=pl, W=W, n_pad=W * n_c, n_c=n_c, grad="student_t3", steps=2, server_chunk=W - 1,
               use_k=False)
    ref, dev, stats = run_trajectory(cfg, 2, two_pass=True, packed=True, fused=True, warm_state=True, deferred=deferred,
                                     check_every=1)
    assert stats["scale_ulp_steps"] == 0 and stats["word_mismatch_steps"] == 0
    assert np.array_equal(dev.get("err_server"), ref.t["err_server"])
    finish(dev)
