"""ob_lamb_warmup_step on layers that are too large for the kernel with the per-layer barrier: moments and update as
two kinds of workgroups of one launch (or of launches that end between them), against the oracle."""
import pytest

torch = pytest.importorskip("torch")

from tests.refstep import HYPER, RefStep  # noqa: E402
from tests.test_gpu_parity import DeviceStep, _need_gpu, assert_close, finish, kernels_of  # noqa: E402
from workloads import Streams, gradient, init_state  # noqa: E402
from workloads.shapes import ParamList, padded_len  # noqa: E402

pytestmark = pytest.mark.gpu

T = 8192
LISTS = {   # sizes, workers, fused_max_tiles, two_pass_warmup
    # fewer parts than the updates lag behind; layers next to ones of the other kernels; an empty one
    "two_layers": ([300, 64 * T + 5, 0, 65 * T - 1, 100_003, 3], 1, 8, False),
    # more parts than that, chunk ends that cut tiles and parts short, tensors that start anywhere
    "lagging": ([161 * T + 77 * i + 1 for i in range(6)] + [13], 61, 8, False),
    # a layer of more parts than are kept, in the default configuration
    "beyond_kept": ([17_500_003, 5000], 2, None, False),
    # no update waits: one group of layers, and two
    "one_group": ([70 * T + 9, 66 * T, 1234], 3, 8, True),
    "two_groups": ([9_000_001, 8_000_003, 70 * T], 7, 8, True),
}


def build(name, **more):
    sizes, W, cap, two_pass = LISTS[name]
    pl, st = ParamList(name, [(f"t{i}", s) for i, s in enumerate(sizes)]), Streams(6)
    n_pad = padded_len(pl.N, W)
    cfg = dict(name=name, plist=pl, W=W, n_pad=n_pad, n_c=n_pad // W, grad="student_t3", steps=3, server_chunk=W - 1,
               use_k=False)
    hyper = dict(HYPER, c_min=1e-4)
    ref = RefStep(pl.offsets, W, W - 1, **hyper)
    dev = DeviceStep(pl.offsets, W, W - 1, two_pass=True, two_pass_warmup=two_pass, fused_max_tiles=cap, **more, **hyper)
    ref.load_state(init_state(st, cfg))
    dev.load_state(ref.t)
    return ref, dev, lambda t: torch.from_numpy(gradient(st, cfg, t))


def compare(ref, dev, what):
    for k in ("m", "v_fresh", "x", "coeff_c", "c_avg"):
        assert_close(dev.get(k), ref.t[k], f"{what}: {k}")


@pytest.mark.parametrize("name,grad", [(n, "f32") for n in LISTS] + [("lagging", "bf16"), ("two_groups", "f16")])
def test_lamb_steps(name, grad):
    _need_gpu()
    import paper_2104_06069_amd as ob
    lp = {"f32": None, "bf16": torch.bfloat16, "f16": torch.float16}[grad]
    ref, dev, g_of = build(name, x_lp_dtype=lp)
    ob.ob_lamb_profile_enable(dev.ctx, True)
    for t in range(2):
        g = g_of(t) if lp is None else g_of(t).to(lp)
        ref.warmup_step(g.float().numpy(), 1e-3)
        dev.warmup_step(g.to(dev.device), 1e-3)
        compare(ref, dev, f"step {t}")
        if lp is not None:
            assert torch.equal(dev.x_lp[:dev.N], dev.t["x"][:dev.N].to(lp))
    assert "warmup_trail" in kernels_of(dev)
    finish(dev)


@pytest.mark.parametrize("name", ["lagging", "one_group"])
def test_lamb_step_replayed_from_a_captured_graph(name):
    """The counters and flags of the launches go round: every replay is the next step."""
    _need_gpu()
    ref, dev, g_of = build(name)
    g = g_of(0).to(dev.device)
    ref.warmup_step(g.cpu().numpy(), 1e-3)
    dev.warmup_step(g, 1e-3)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        dev.warmup_step(g, 1e-3)
    for t in range(1, 4):
        g.copy_(g_of(t))
        graph.replay()
        ref.warmup_step(g_of(t).numpy(), 1e-3)
        compare(ref, dev, f"replay {t}")
    finish(dev)


def test_expired_wait_is_reported_and_recovered():
    """With no polls allowed the updates take what they find (every access stays in bounds) and the status call says so; the
    context then takes two passes."""
    _need_gpu()
    import paper_2104_06069_amd as ob
    ref, dev, g_of = build("two_layers", spin_limit=0)
    dev.warmup_step(g_of(0).to(dev.device), 1e-3)
    with pytest.raises(ob.ObLambError) as e:
        ob.ob_lamb_check_device_status(dev.ctx, dev.stream)
    assert e.value.status == -4
    dev.load_state(ref.t)
    ob.ob_lamb_profile_enable(dev.ctx, True)
    ref.warmup_step(g_of(1).numpy(), 1e-3)
    dev.warmup_step(g_of(1).to(dev.device), 1e-3)
    compare(ref, dev, "after the expiry")
    assert "warmup_trail" not in kernels_of(dev)
    finish(dev)
