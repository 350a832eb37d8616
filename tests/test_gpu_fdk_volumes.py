"""Backprojections of volumes that are narrow in x and y or have few planes: blocks that go
from one plane of column pieces to the next, the last block part full, pieces of 1, 2, 4 and 8
voxels with a remainder, the angles split or not.  Reference and tolerance as for the other
volumes.  And that a narrow volume costs no more than three times a cubic one of as many
voxels (a block for every plane made it 60 times)."""
import numpy as np
import pytest

from oracle import recon
from paper_2201_13191_amd import mcx
from test_gpu_fdk_paths import U, _fdk, _geo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vol,n_ang,h", [
    ((1050001, 1, 1), 1, 2e-4), ((131100, 2, 4), 2, 1e-3), ((21000, 5, 10), 3, 0.01),
    ((300, 1, 1), 5, 0.5), ((77, 3, 5), 3, 1.25), ((1, 1030, 1021), 2, 0.3),
    ((2, 731, 720), 2, 0.4), ((3, 600, 601), 2, 0.5), ((4, 513, 512), 2, 0.5),
    ((5, 460, 461), 2, 0.6), ((9, 350, 350), 2, 0.7), ((1, 33, 31), 3, 4.0)])
def test_narrow_and_thin(vol, n_ang, h):
    print("fdk volume", vol, n_ang, flush=True)
    rng = np.random.default_rng(vol[0])
    nu, nv = 96, 80
    proj = rng.normal(0.0, 1.0, (n_ang, nv, nu)).astype(np.float32)
    geo = _geo(nu, nv, 4.0)
    q, v = _fdk(geo, proj, vol, h)
    ref = recon.fdk_backproject(q, geo, vol, float(np.float32(h)))   # as the call takes it
    atol = (n_ang + 4 * max(nu, nv)) * 2.0 ** -52 * np.pi * np.abs(q).max() * 2.0
    np.testing.assert_allclose(v, ref, rtol=2 * U, atol=atol)


def test_narrow_costs_no_more():
    import torch
    g = mcx.Projector(0)
    g.set_geometry(**_geo(128, 128, 2.0))
    proj = torch.rand((60, 128, 128), device="cuda")
    tmp = torch.empty_like(proj)

    def us(vol, h):
        v = torch.empty(vol, device="cuda")
        best = 1e9
        for _ in range(4):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            mcx.mc_fdk_async(g.ctx, proj, tmp, v, h, torch.cuda.current_stream())
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 1000)
        return best

    narrow, cube = us((1 << 20, 1, 1), 1e-4), us((64, 128, 128), 0.5)
    print("narrow", narrow, "cubic", cube, flush=True)
    assert narrow <= 3 * cube
    g.close()
