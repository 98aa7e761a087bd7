"""Values at the ends of the number range in the kernels of the larger lists, against the oracle: NaN, Inf and zero variances,
gradients with NaN and Inf, tensors of zeros, in k_warmup_trail (with and without weight decay; with updates that wait in its
launch and in launches of their own) and in ob_lamb_ratios_apply_hist's forms, with the plain ratio pass in its launch and with the
table of the launch before, among empty and one-element tensors."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.refstep import HYPER, RefStep  # noqa: E402
from tests.test_gpu_parity import (LARGE, DeviceStep, _need_gpu, assert_close, finish, kernels_of, push_wire, start_pair,  # noqa: E402
                                   words_of)
from workloads import Streams, foreign_server_chunks, foreign_worker_chunks, gradient, init_state  # noqa: E402
from workloads.shapes import ParamList, padded_len  # noqa: E402

pytestmark = pytest.mark.gpu

T = 8192


def config(name, sizes, W, use_k=False):
    pl = ParamList(name, [(f"t{i}", s) for i, s in enumerate(sizes)])
    n_pad = padded_len(pl.N, W)
    return dict(name=name, plist=pl, W=W, n_pad=n_pad, n_c=n_pad // W, grad="student_t3", steps=4, server_chunk=W - 1,
                use_k=use_k)


LAMB = {   # sizes, workers, two_pass_warmup
    "waits": ([300, 64 * T + 5, 0, 65 * T - 1, 100_003, 3, 70 * T, 66 * T, 1], 3, False),
    "launches": ([70 * T + 9, 0, 66 * T, 1234, 64 * T, 1, 65 * T + 3], 3, True),
}


@pytest.mark.parametrize("wd", [0.0, 0.01])
@pytest.mark.parametrize("name", list(LAMB))
def test_lamb_steps(name, wd):
    _need_gpu()
    import paper_2104_06069_amd as ob
    sizes, W, two_pass = LAMB[name]
    cfg, st = config(name, sizes, W), Streams(31)
    off = cfg["plist"].offsets
    hyper = dict(HYPER, weight_decay=wd, c_min=1e-4)
    ref = RefStep(off, W, W - 1, **hyper)
    dev = DeviceStep(off, W, W - 1, two_pass=True, two_pass_warmup=two_pass, fused_max_tiles=8, **hyper)
    s = init_state(st, cfg)
    large = [l for l in range(len(sizes)) if sizes[l] >= 64 * T]
    at = lambda l: slice(int(off[l]), int(off[l + 1]))
    # the first large tensor: moments and variances of zero among others; the third: nothing but zeros (no gradient either: both
    # sums are 0); the fourth: NaN and Inf in the gradient (its sums and every element's update); the second as it comes
    for k in ("m", "v_fresh"):
        s[k][off[large[0]] + 5:off[large[0]] + 3 * T] = 0
        s[k][at(large[2])] = 0
    s["x"][at(large[2])] = 0
    ref.load_state(s)
    dev.load_state(ref.t)
    ob.ob_lamb_profile_enable(dev.ctx, True)
    for t in range(3):
        g = gradient(st, cfg, t)
        g[off[large[0]] + 5:off[large[0]] + 2 * T] = 0
        g[at(large[2])] = 0
        if t == 1:
            g[off[large[3]] + T] = np.inf
            g[off[large[3] + 1] - 1] = np.nan
        ref.warmup_step(g, 1e-3)
        dev.warmup_step(torch.from_numpy(g).to(dev.device), 1e-3)
        for k in ("m", "v_fresh", "x", "coeff_c", "c_avg"):
            assert_close(dev.get(k), ref.t[k], f"step {t}: {k}")
    assert "warmup_trail" in kernels_of(dev)
    for l in large[:3]:
        assert np.all(np.isfinite(dev.get("x")[at(l)]))
    finish(dev)


COMPRESS = {   # sizes, workers, the limit of the barrier kernel's layers, ratio pass in the same launch
    "same_launch": ([1, 0, 1, 700, 1, 1, 3000, 0, 400 * T + 5, 1023, 1, 5000, 12 * T, 0, 70 * T + 9, 1], 3, LARGE, True),
    "same_launch_large": ([40 * T + 3, 0, 1, 5 * T + 1, 70 * T, 9 * T, 64, 66 * T + 7], 3, 8, True),
    "table": ([1, 0, 12 * T, 0, 1] + [1001, 0, 1, 999] * 700 + [40 * T + 3, 1, 0, 0], 3, LARGE, False),
    "table_large": ([1, 0, 70 * T, 0, 1] + [1001, 0, 1, 999] * 700 + [6 * T + 3, 1, 0, 66 * T + 1, 0], 3, 8, False),
}


@pytest.mark.parametrize("use_k", [False, True])
@pytest.mark.parametrize("name", list(COMPRESS))
def test_compression_steps(name, use_k):
    _need_gpu()
    import paper_2104_06069_amd as ob
    sizes, W, cap, one = COMPRESS[name]
    cfg = config(name, sizes, W, use_k)
    st, ref, dev = start_pair(cfg, seed=32, two_pass=True, packed=True, fused=True, fused_max_tiles=cap, deferred=True,
                              deferred_variance=2)
    off = cfg["plist"].offsets
    hard = [("v_frozen", np.nan), ("v_frozen", np.inf), ("v_frozen", 0.0), ("v_fresh", 0.0), ("v_fresh", np.inf), ("v_fresh", np.nan)]
    n = 0
    for l in range(len(sizes)):      # one such value in most tensors, the last element, and one inside the longer ones
        if sizes[l] == 0 or l % 7 == 6:
            continue
        for o in ([sizes[l] - 1] if sizes[l] < T else [sizes[l] - 1, sizes[l] // 2, 3]):
            k, v = hard[n % len(hard)]
            ref.t[k][off[l] + o] = v
            n += 1
    dev.load_state(ref.t)
    ob.ob_lamb_profile_enable(dev.ctx, True)
    for t in range(5):
        g = gradient(st, cfg, t)
        if t == 3:                   # of the first chunk alone: its scale, and so the whole of it, is no number from here on
            g[cfg["n_c"] // 2] = np.inf
            g[7] = np.nan
        fw, fs = foreign_worker_chunks(st, cfg, t)
        fa, fss = foreign_server_chunks(st, cfg, t)
        ref.set_foreign_in(fw, fs)
        ref.set_foreign_all(fa, fss)
        dev.begin_step()
        push_wire(ref, dev)
        ref.step(g, 1e-3)
        dev.step(torch.from_numpy(g).to(dev.device), 1e-3)
        assert np.array_equal(words_of(dev.packed_local), ref.bits_local)
        assert np.array_equal(words_of(dev.packed_all), ref.bits_all)
        assert_close(dev.scales_local.cpu().numpy(), ref.scales_local, f"step {t}: scales")
        for k in ("x", "m", "v_fresh", "err_worker", "err_server", "r_prev", "coeff_c"):
            assert_close(dev.get(k), ref.t[k], f"step {t}: {k}")
        assert np.all(np.isfinite(dev.get("r_prev")))
    names = kernels_of(dev)
    assert names & {"ratios_apply_hist", "ratios_apply_hist_lds"}, names
    dev.begin_step()
    dev.ratios_apply(1e-3)
    assert ("ratios_pass" in kernels_of(dev)) == (not one)
    assert ("ratios_big_hist" in names) == (ob.ob_lamb_big_tile_params(dev.ctx) > 0) == (cap == 8)
    finish(dev)
