"""DeviceStep.step() and the calls it stands for, without a device: a recording binding in place of the library."""
import pytest

torch = pytest.importorskip("torch")

from paper_2104_06069_amd import binding as ob  # noqa: E402
from paper_2104_06069_amd import step as step_module  # noqa: E402
from paper_2104_06069_amd.step import DeviceStep  # noqa: E402


def _bare(cls, fused, monkeypatch):
    """An object of cls with host buffers and no context; -> (it, names of the library calls it makes)."""
    ds = cls.__new__(cls)
    L, n_pad, W = 2, 2048, 2
    z = lambda n, dt=torch.float32: torch.zeros(n, dtype=dt)  # noqa: E731
    ds.ctx, ds.W, ds.c, ds.L, ds.n_pad, ds.n_c = None, W, 1, L, n_pad, n_pad // W
    ds.t = {k: z(n_pad) for k in ("x", "m", "v_fresh", "v_frozen", "err_worker")}
    ds.t.update(err_server=z(ds.n_c), mom_scale=None, **{k: z(L) for k in ("c_avg", "coeff_c", "r_prev")})
    ds.fold_gather, ds.deferred_error, ds.packed_momentum, ds.fused_apply = True, True, True, fused
    ds.packed_local, ds.packed_in = z(n_pad // 32, torch.int32), z(n_pad // 32, torch.int32)
    ds.scales_local, ds.scales_in = z(W), z(W)
    ds.srv_words, ds.srv_scale = z(ds.n_c // 32, torch.int32), z(1)
    ds._pa, ds._ss = [z(n_pad // 32, torch.int32) for _ in range(2)], [z(W) for _ in range(2)]
    ds._cur, ds.m_is_packed, ds.vf_period, ds._vf_pending = 0, True, 0, None
    ds.x_lp, ds.grad_scale, ds.status_interval, ds._steps_since_check = None, 1.0, 0, 0
    calls = []
    for name in ("compress_local", "server_reduce", "ratios_apply", "layer_ratios", "decompress_apply"):
        monkeypatch.setattr(step_module.ob, "ob_lamb_" + name, lambda ctx, state, *a, _n=name: calls.append((_n, state)))
    monkeypatch.setattr(cls, "stream", 0)
    return ds, calls


ORDER = {True: ["compress_local", "server_reduce", "ratios_apply"],
         False: ["compress_local", "server_reduce", "layer_ratios", "decompress_apply"]}


@pytest.mark.parametrize("fused", [True, False])
def test_step_makes_the_calls_in_order(fused, monkeypatch):
    ds, calls = _bare(type("Plain", (DeviceStep,), {}), fused, monkeypatch)
    ds.step(torch.zeros(ds.n_pad), 1e-3)
    assert [c[0] for c in calls] == ORDER[fused]
    for _, s in calls:
        assert s.x == ds.t["x"].data_ptr() and s.own_packed_in == ds.packed_in.data_ptr() + ds.n_c // 8


@pytest.mark.parametrize("where", ["subclass", "instance"])
@pytest.mark.parametrize("name", ["compress_local", "gather", "server_reduce", "ratios_apply", "layer_ratios",
                                  "decompress_apply"])
def test_step_goes_through_calls_that_a_program_replaced(name, where, monkeypatch):
    """A program's own compress_local(), gather(), ... runs as part of step(), and what it changes is what the
    calls after it see."""
    seen = []
    base = getattr(DeviceStep, name)

    def own(self, *a):
        seen.append(name)
        self.t["x"] = self.t["x"].clone()
        base(self, *a)

    cls = type("Own", (DeviceStep,), {name: own} if where == "subclass" else {})
    fused = name not in ("layer_ratios", "decompress_apply")
    ds, calls = _bare(cls, fused, monkeypatch)
    if where == "instance":
        setattr(ds, name, lambda *a: own(ds, *a))
    before = ds.t["x"]
    ds.step(torch.zeros(ds.n_pad), 1e-3)
    assert seen == [name] and [c[0] for c in calls] == ORDER[fused]
    first = {"compress_local": 0, "gather": 1, "server_reduce": 1, "ratios_apply": 2, "layer_ratios": 2, "decompress_apply": 3}[name]
    for i, (_, s) in enumerate(calls):
        assert s.x == (ds.t["x"] if i >= first else before).data_ptr(), i


def test_state_entries_that_a_program_took_out_or_put_in(monkeypatch):
    """With the momentum in its 1-bit form the dense array may be given back (its entry deleted or None), and
    pointers that the object does not fill itself may be put into the dict."""
    ds, calls = _bare(type("Plain", (DeviceStep,), {}), True, monkeypatch)
    del ds.t["m"], ds.t["mom_scale"]
    ds.fold_gather = ds.deferred_error = False
    ds.gather = lambda: None
    mine = torch.zeros(64)
    ds.t.update(own_packed_in=mine[:32], own_scale_in=mine[32:], err_packed=mine[4:])
    ds.step(torch.zeros(ds.n_pad), 1e-3)
    assert len(calls) == 3
    for _, s in calls:
        assert s.m is None and s.mom_scale is None and s.m_packed == ds._pa[1].data_ptr()
        assert s.own_packed_in == mine.data_ptr() and s.own_scale_in == mine.data_ptr() + 128
        assert s.err_packed == mine.data_ptr() + 16 and s.err_scales is None and s.srv_err_packed is None
    ds.t["x"] = None
    assert ds._state("commit").x is None and ds._state("commit").m_packed == ds._pa[0].data_ptr()
    assert [f for f, _ in ob.ObLambState._fields_] == list(step_module._STATE_FIELDS)
