"""The worker's pass with a 16-bit gradient on both sides of the list length from which it sums the squares of its tiles and
forms their sign words through LDS (80 tiles of 1024 elements a CU), against binary32 arithmetic in numpy: error and sign words bit for bit, scales of the same sum."""
import numpy as np
import pytest

from tests.refstep import HYPER

pytestmark = pytest.mark.gpu

f32 = np.float32
SPAN = 1024


@pytest.mark.parametrize("tiles_of_chunk,cut,W", [(65536, 256, 1), (65535, 768, 1), (21846, 512, 3), (21845, 0, 3),
                                                  (20480, 256, 1), (20479, 768, 1), (6827, 512, 3), (6826, 0, 3)])
def test_pass(tiles_of_chunk, cut, W):
    import torch
    from paper_2104_06069_amd.step import DeviceStep
    n_c = tiles_of_chunk * SPAN - cut
    n = n_c * W - 100            # (the list ends before its padding does)
    ds = DeviceStep(np.array([0, 5 * SPAN + 3, n]), W, 0, packed_momentum=True, fused_apply=True, deferred_error=True, **HYPER)
    assert ds.n_c == n_c
    g = torch.Generator(device="cuda").manual_seed(7)
    words = lambda k: torch.randint(-2 ** 31, 2 ** 31, (k,), generator=g, device="cuda", dtype=torch.int32)
    z_old = torch.randn(ds.n_pad, generator=g, device="cuda").mul_(1e-4)
    grad = torch.randn(ds.n_pad, generator=g, device="cuda").mul_(1e-3).to(torch.bfloat16)
    ds.t["err_worker"].copy_(z_old)
    ds.m_is_packed, ds._cur = True, 1
    ds._pa[0].copy_(words(ds._pa[0].numel()))                 # the previous momentum
    ds.packed_local.copy_(words(ds.packed_local.numel()))     # C[z_old]
    s_m, s_e = (np.array([1e-4, 3e-4, 2e-4], f32)[:W] * k for k in (f32(1), f32(0.7)))
    ds._ss[0].copy_(torch.from_numpy(s_m))
    ds.scales_local.copy_(torch.from_numpy(s_e))
    bits_of = lambda t: np.unpackbits(t.cpu().numpy().view(np.uint8), bitorder="little").reshape(W, n_c) == 1
    m_bits, e_bits = bits_of(ds._pa[0]), bits_of(ds.packed_local)
    ds.compress_local(grad)
    got_z, got_bits, got_s = ds.t["err_worker"].cpu().numpy().reshape(W, n_c), bits_of(ds.packed_local), ds.scales_local.cpu().numpy()
    ds.close()
    z_old, grad = z_old.cpu().numpy().reshape(W, n_c), grad.float().cpu().numpy().reshape(W, n_c)
    b1, omb1 = f32(HYPER["beta1"]), f32(1) - f32(HYPER["beta1"])
    for c in range(W):
        m = np.where(m_bits[c], s_m[c], -s_m[c])
        m[max(0, n - c * n_c):] = 0      # (the padding has no momentum)
        z = (b1 * m + omb1 * grad[c]) + (z_old[c] - np.where(e_bits[c], s_e[c], -s_e[c]))
        assert z.dtype == f32 and np.array_equal(z.view(np.uint32), got_z[c].view(np.uint32)), c
        assert np.array_equal(z >= 0, got_bits[c]), c
        want = f32(np.sqrt(np.sum(z.astype(np.float64) ** 2) / n_c))
        assert abs(got_s[c] - want) <= np.spacing(want), (c, got_s[c], want)   # (another order of a binary64 sum)
