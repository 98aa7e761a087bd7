"""The update of the tiles outside the 8192-element ones in the last workgroups of k_ratios_apply_hist's launch, over the 16-bit copy,
replays of a captured graph, the lists that only this form takes into that launch, and a wait that expires."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.test_gpu_hard_values import config  # noqa: E402
from tests.refstep import HYPER  # noqa: E402
from tests.test_gpu_parity import DeviceStep, _need_gpu, assert_close, finish, kernels_of, push_wire, start_pair  # noqa: E402
from workloads import foreign_server_chunks, foreign_worker_chunks, gradient  # noqa: E402

pytestmark = pytest.mark.gpu

T = 8192
# layers of one element and of none, that end in a tile, that only small tiles hold, wholly inside listed tiles; ends of chunks
SMALL = [1, 0, 1, 700, 1, 1, 3000, 0, 40 * T + 5, 1023, 1, 300 * T, 12 * T, 0, 77, 5 * T + 1]
MANY = [200 * T + 3] * 28 + [64, 0, 900]      # 5600 listed tiles: more than 20 a CU (256 CUs)


def step(cfg, st, ref, dev, t, run):
    g = gradient(st, cfg, t)
    ref.set_foreign_in(*foreign_worker_chunks(st, cfg, t))
    ref.set_foreign_all(*foreign_server_chunks(st, cfg, t))
    dev.begin_step()
    push_wire(ref, dev)
    ref.step(g, 1e-3)
    run(torch.from_numpy(g).to(dev.device))


@pytest.mark.parametrize("sizes,W,use_k,lp", [(SMALL, 1, False, None), (SMALL, 7, True, torch.bfloat16), (SMALL, 3, False, torch.float16),
                                              (MANY, 2, False, None)], ids=["plain", "k_bf16", "f16", "many_tiles"])
def test_steps(sizes, W, use_k, lp):
    _need_gpu()
    import paper_2104_06069_amd as ob
    cfg = config("rest_update", sizes, W, use_k)
    st, ref, dev = start_pair(cfg, seed=51, two_pass=True, packed=True, fused=True, fused_max_tiles=1 << 20, deferred=True,
                              deferred_variance=2)
    if lp is not None:
        dev.x_lp = torch.zeros(dev.n_pad, device=dev.device, dtype=lp)
    ref.t["v_frozen"][cfg["plist"].offsets[6] + 5] = np.nan     # (the update's general path)
    dev.load_state(ref.t)
    for t in range(4):
        if t == 1:
            ob.ob_lamb_profile_enable(dev.ctx, True)
        step(cfg, st, ref, dev, t, lambda g: dev.step(g, 1e-3))
        for k in ("x", "r_prev", "coeff_c", "v_fresh"):
            assert_close(dev.get(k), ref.t[k], f"step {t}: {k}")
        if lp is not None:
            a, b = dev.x_lp[:dev.N], dev.t["x"][:dev.N].to(lp)
            assert torch.equal(a.isnan(), b.isnan())      # (which NaN: the formats leave it open)
            assert torch.equal(a.nan_to_num().view(torch.int16), b.nan_to_num().view(torch.int16))
    names = kernels_of(dev)
    assert names & {"ratios_apply_hist", "ratios_apply_hist_lds"} and not names & {"ratios_pass", "decompress_apply"}, names
    finish(dev)


def test_replayed_from_a_captured_graph():
    """The launch counts its launches itself: replays give what as many eager steps of a second context do."""
    _need_gpu()
    cfg = config("rest_update", SMALL, 3)
    pair = [start_pair(cfg, seed=52, two_pass=True, packed=True, fused=True, fused_max_tiles=1 << 20, deferred=True, deferred_variance=2)
            for _ in range(2)]
    st, (dev, eager) = pair[0][0], [p[2] for p in pair]
    P = dev.graph_period
    g = [torch.from_numpy(gradient(st, cfg, t)).to(dev.device) for t in range(P)]

    def steps(d):
        for j in range(P):
            d.begin_step()
            d.step(g[j], 1e-3)
    for d in (dev, eager):
        for b in d._ss:
            b.fill_(1e-4)
        steps(d)
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


@pytest.mark.parametrize("period", [0, 2])
def test_expired_wait_is_reported_and_recovered(period):
    """With no polls allowed the updates of the listed tiles and of the rest go on with what they find (every access stays in
    bounds) and the status call says so; the context then takes the kernels that wait for nothing."""
    _need_gpu()
    import paper_2104_06069_amd as ob
    cfg = config("rest_update", SMALL, 3)
    st, ref, ok = start_pair(cfg, seed=53, two_pass=True, packed=True, fused=True, fused_max_tiles=1 << 20, deferred=True,
                             deferred_variance=period)
    finish(ok)
    dev = DeviceStep(cfg["plist"].offsets, cfg["W"], cfg["server_chunk"], two_pass=True, packed_momentum=True, fused_apply=True,
                     fused_max_tiles=1 << 20, deferred_error=True, deferred_variance=period, spin_limit=0, **HYPER)
    dev.load_state(ref.t)
    for t in range(2):      # (the first one reads the dense momentum)
        dev.begin_step()
        if t == 1:
            ob.ob_lamb_profile_enable(dev.ctx, True)
        dev.step(torch.from_numpy(gradient(st, cfg, t)).to(dev.device), 1e-3)
    names = kernels_of(dev)
    assert names & {"ratios_apply_hist", "ratios_apply_hist_lds"} and not names & {"ratios_pass", "decompress_apply"}, names
    with pytest.raises(ob.ObLambError) as e:
        ob.ob_lamb_check_device_status(dev.ctx, dev.stream)
    assert e.value.status == -4
    dev.load_state(ref.t)
    for t in range(2, 4):
        step(cfg, st, ref, dev, t, lambda g: dev.step(g, 1e-3))
        for k in ("x", "r_prev", "coeff_c", "v_fresh"):
            assert_close(dev.get(k), ref.t[k], f"step {t}: {k}")
    names = kernels_of(dev)
    assert not names & {"ratios_apply_hist", "ratios_apply_hist_lds", "ratios_apply_resident", "ratios_trail"}, names
    finish(dev)
