"""ob_lamb_ratios_apply_hist on lists with several layers that are too large for the kernel with the per-layer barrier: ratio
pass and update as two kinds of workgroups of one launch, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.test_gpu_hard_values import config  # noqa: E402
from tests.refstep import HYPER  # noqa: E402
from tests.test_gpu_parity import DeviceStep, _need_gpu, assert_close, finish, kernels_of, push_wire, start_pair, words_of  # noqa: E402
from workloads import foreign_server_chunks, foreign_worker_chunks, gradient  # noqa: E402

pytestmark = pytest.mark.gpu

T = 8192
LISTS = {   # sizes, workers (the barrier kernel's layers: up to 8 tiles; with enough tiles in none of the kernels' layers that the plain ratio
    # pass is a launch of its own, or no listed layer)
    # the second layer's tiles are fewer than what the updates lag behind; layers of the other kernels between them, an empty one
    "two_layers": ([300, 900 * T + 5, 0, 5 * T + 1, 150 * T - 1, 60 * T, 100_003, 50 * T, 55 * T, 3], 1),
    # chunk ends that cut tiles short, tensors that start anywhere; more tiles than that before the last one
    "lagging": ([330 * T + 77 * i + 1 for i in range(7)] + [13, 3 * T, 60 * T + 1, 59 * T, 58 * T], 61),
    # no layer of the barrier kernel
    "none_listed": ([520 * T, 600 * T + 4000], 3),
}


def build(name, use_k=False):
    sizes, W = LISTS[name]
    cfg = config(name, sizes, W, use_k)
    return (cfg,) + start_pair(cfg, seed=41, two_pass=True, packed=True, fused=True, fused_max_tiles=8, deferred=True,
                               deferred_variance=3)


def step(cfg, st, ref, dev, t, run):
    g = gradient(st, cfg, t)
    ref.set_foreign_in(*foreign_worker_chunks(st, cfg, t))
    ref.set_foreign_all(*foreign_server_chunks(st, cfg, t))
    dev.begin_step()
    push_wire(ref, dev)
    ref.step(g, 1e-3)
    run(torch.from_numpy(g).to(dev.device))
    assert np.array_equal(words_of(dev.packed_all), ref.bits_all)
    for k in ("x", "v_fresh", "r_prev", "coeff_c"):
        assert_close(dev.get(k), ref.t[k], f"step {t}: {k}")


@pytest.mark.parametrize("name,use_k,lp", [(n, False, None) for n in LISTS] + [("two_layers", True, None), ("lagging", True, torch.bfloat16)])
def test_steps(name, use_k, lp):
    _need_gpu()
    import paper_2104_06069_amd as ob
    cfg, st, ref, dev = build(name, use_k)
    if lp is not None:
        dev.x_lp = torch.zeros(dev.n_pad, device=dev.device, dtype=lp)
    off = cfg["plist"].offsets
    l = int(np.argmax(np.diff(off)))
    for k, v, o in (("v_frozen", 0.0, 3), ("v_frozen", np.inf, 9 * T), ("v_fresh", 0.0, 40 * T)):   # in the largest layer
        ref.t[k][off[l] + o] = v
    dev.load_state(ref.t)
    ob.ob_lamb_profile_enable(dev.ctx, True)
    for t in range(5):
        step(cfg, st, ref, dev, t, lambda g: dev.step(g, 1e-3))
        if lp is not None:
            assert torch.equal(dev.x_lp[:dev.N].view(torch.int16), dev.t["x"][:dev.N].to(lp).view(torch.int16))
    names = kernels_of(dev)
    assert "ratios_trail" in names and "ratios_big_hist" not in names, names
    finish(dev)


def test_steps_replayed_from_a_captured_graph():
    """The flags and counters of the launches go round: replays give what as many eager steps of a second context do."""
    _need_gpu()
    cfg, st, ref, dev = build("lagging")
    _, _, _, eager = build("lagging")
    P = dev.graph_period
    g = [torch.from_numpy(gradient(st, cfg, t)).to(dev.device) for t in range(P)]
    for d in (dev, eager):
        d.load_state(ref.t)
        for b in d._pa:
            b.copy_(g[0][:b.numel()].view(torch.int32))
        for b in d._ss:
            b.fill_(1e-4)
    def steps(d):
        for j in range(P):
            d.begin_step()
            d.step(g[j], 1e-3)
    for d in (dev, eager):
        d.step(g[0], 1e-3)
        steps(d)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            steps(dev)
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(3):
        for j in range(P):
            g[j].mul_(0.5).add_(1e-4)
        graph.replay()
        steps(eager)
        torch.cuda.synchronize()
        for k in ("x", "v_fresh", "r_prev", "coeff_c", "err_worker", "err_server"):
            assert torch.equal(dev.t[k], eager.t[k]), (rep, k)
    finish(dev)
    finish(eager)


def test_expired_wait_is_reported_and_recovered():
    """With no polls allowed the updates take what they find (every access stays in bounds) and the status call says so; the
    context then takes the kernels that wait for nothing."""
    _need_gpu()
    import paper_2104_06069_amd as ob
    cfg, st, ref, ok = build("none_listed")
    finish(ok)
    dev = DeviceStep(cfg["plist"].offsets, cfg["W"], cfg["server_chunk"], two_pass=True, packed_momentum=True, fused_apply=True,
                     fused_max_tiles=8, deferred_error=True, deferred_variance=3, spin_limit=0, **HYPER)
    dev.load_state(ref.t)
    for t in range(2):      # (the first one reads the dense momentum)
        dev.begin_step()
        dev.step(torch.from_numpy(gradient(st, cfg, t)).to(dev.device), 1e-3)
    with pytest.raises(ob.ObLambError) as e:
        ob.ob_lamb_check_device_status(dev.ctx, dev.stream)
    assert e.value.status == -4
    dev.load_state(ref.t)
    ob.ob_lamb_profile_enable(dev.ctx, True)
    for t in range(2, 4):
        step(cfg, st, ref, dev, t, lambda g: dev.step(g, 1e-3))
    assert "ratios_trail" not in kernels_of(dev)
    finish(dev)
