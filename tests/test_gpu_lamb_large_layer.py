"""ob_lamb_warmup_step in one pass on layers near the largest that its kernel takes (x of most spans waits in
LDS), against the oracle: layers below and beyond the limit, chunk ends that cut tiles short, 16-bit gradients."""
import pytest

torch = pytest.importorskip("torch")

from tests.refstep import HYPER, RefStep  # noqa: E402
from tests.test_gpu_parity import DeviceStep, _need_gpu, assert_close, finish  # noqa: E402
from workloads import Streams, gradient, init_state  # noqa: E402
from workloads.shapes import ParamList, padded_len  # noqa: E402

pytestmark = pytest.mark.gpu

LISTS = {   # sizes, workers, layers in one pass
    "one_layer": ([9_000_001, 77, 700_001], 3, 2),
    "cut_tiles": ([1023, 8_000_003, 4097, 500_009], 61, 2),
    "beyond": ([12_000_000, 8 * 8192 + 5, 8191], 2, 1),
}


@pytest.mark.parametrize("wd", [0.0, 0.01])
@pytest.mark.parametrize("grad", ["f32", "bf16"])
@pytest.mark.parametrize("name", list(LISTS))
def test_lamb_step_of_a_large_layer(name, grad, wd):
    _need_gpu()
    import paper_2104_06069_amd as ob
    sizes, W, n_fused = LISTS[name]
    pl, st = ParamList(name, [(f"t{i}", s) for i, s in enumerate(sizes)]), Streams(5)
    n_pad = padded_len(pl.N, W)
    cfg = dict(name=name, plist=pl, W=W, n_pad=n_pad, n_c=n_pad // W, grad="student_t3", steps=2, server_chunk=W - 1,
               use_k=False)
    hyper = dict(HYPER, weight_decay=wd, c_min=1e-4)
    ref, dev = RefStep(pl.offsets, W, W - 1, **hyper), DeviceStep(pl.offsets, W, W - 1, two_pass=True, **hyper)
    assert ob.ob_lamb_warmup_fused_layers(dev.ctx) == n_fused
    ref.load_state(init_state(st, cfg))
    dev.load_state(ref.t)
    for t in range(2):
        g = torch.from_numpy(gradient(st, cfg, t))
        if grad == "bf16":
            g = g.to(torch.bfloat16)
        ref.warmup_step(g.float().numpy(), 1e-3)
        dev.warmup_step(g.to(dev.device), 1e-3)
        for k in ("m", "v_fresh", "x", "coeff_c", "c_avg"):
            assert_close(dev.get(k), ref.t[k], f"step {t}: {k}")
    finish(dev)
