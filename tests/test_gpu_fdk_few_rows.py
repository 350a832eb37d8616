"""The filter's launch on both sides of each line of its rule for few rows: a block per row
(short rows, and rows in place), blocks of 32 x 64 sharing a row, and the wide blocks.
Reference and tolerance as for the other filter widths.  And that one angle of 130 x 66 pixels
takes no more than half again the time of one of 128 x 65 (wide blocks made it 2.4 times)."""
import numpy as np
import pytest

from oracle import recon
from paper_2201_13191_amd import mcx
from test_gpu_fdk_paths import U, _fdk, _geo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nu,nv,n_ang,in_place", [
    (5, 3, 1, False), (64, 128, 2, False), (64, 129, 2, True), (96, 64, 4, True),
    (96, 257, 1, False), (98, 51, 2, False), (40, 5440, 3, False), (40, 5472, 3, False),
    (130, 66, 1, False), (192, 512, 2, True), (192, 513, 2, True), (256, 200, 2, True),
    (256, 401, 1, True), (257, 33, 2, True), (130, 4096, 2, False), (514, 96, 3, False),
    (514, 3300, 1, False)])
def test_few_rows(nu, nv, n_ang, in_place):
    print("fdk rows", nu, nv, n_ang, in_place, flush=True)
    rng = np.random.default_rng(nu * 7 + nv)
    proj = rng.normal(1.0, 1.0, (n_ang, nv, nu)).astype(np.float32)
    geo = _geo(nu, nv)
    ref = recon.fdk_filter(proj, geo)
    got, _ = _fdk(geo, proj, (1, 1, 1), 1.0, in_place)
    np.testing.assert_allclose(got, ref, rtol=2 * U, atol=nu * 2.0 ** -52 * np.abs(ref).max())


def test_one_angle_costs_no_more():
    import torch

    def us(nu, nv):
        g = mcx.Projector(0)
        g.set_geometry(**_geo(nu, nv))
        proj = torch.rand((1, nv, nu), device="cuda")
        tmp, vol = torch.empty_like(proj), torch.empty((1, 1, 1), device="cuda")
        best = 1e9
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(20):
                mcx.mc_fdk_async(g.ctx, proj, tmp, vol, 1.0, torch.cuda.current_stream())
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 50)
        g.close()
        return best

    wide, narrow = us(130, 66), us(128, 65)
    print("130", wide, "128", narrow, flush=True)
    assert wide <= 1.5 * narrow
