"""The FDK's kernel variants at the sizes where they change: rows of every block
width of the filter (and one pixel past it), several column blocks, a filter in
place, and both forms of the backprojection with voxels off the panel.

Reference: oracle/recon.py (fp64).  Tolerance: both sides sum in fp64 and round
once to fp32, so two half-ulps of the result plus the sums' own rounding (at
most nu, or n_ang, terms of 2^-53) against the largest value."""
import numpy as np
import pytest

from oracle import recon
from paper_2201_13191_amd import mcx

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


def _geo(nu, nv, pitch=1.5):
    return dict(sod_mm=400.0, sdd_mm=800.0, nu=nu, nv=nv, pu_mm=pitch, pv_mm=2.0, snu=nu, snv=nv,
                step_mm=1.0, flags=0)


def _fdk(geo, proj, vol, voxel, in_place=False):
    import torch
    g = mcx.Projector(0)
    g.set_geometry(**geo)
    d_p = torch.from_numpy(proj).cuda()
    d_q = d_p if in_place else torch.empty_like(d_p)
    d_v = torch.full(vol, float("nan"), dtype=torch.float32, device="cuda")
    mcx.mc_fdk_async(g.ctx, d_p, d_q, d_v, voxel)
    torch.cuda.synchronize()
    out = d_q.cpu().numpy(), d_v.cpu().numpy()
    g.close()
    return out


@pytest.mark.parametrize("nu,nv,n_ang,in_place", [
    (1, 3, 2, False), (2, 5, 3, False), (33, 7, 3, True), (64, 33, 2, False), (65, 9, 5, False),
    (128, 31, 3, True), (129, 4, 3, False), (192, 13, 3, False), (193, 5, 2, True),
    (256, 11, 3, False), (257, 3, 3, False), (384, 7, 2, False), (385, 5, 2, False),
    (512, 5, 3, True), (513, 3, 2, False), (514, 3, 2, True), (1031, 5, 1, False)])
def test_filter_widths(nu, nv, n_ang, in_place):
    print("fdk filter", nu, nv, n_ang, in_place, flush=True)
    rng = np.random.default_rng(nu * 7 + nv)
    proj = rng.normal(1.0, 1.0, (n_ang, nv, nu)).astype(np.float32)
    geo = _geo(nu, nv)
    ref = recon.fdk_filter(proj, geo)
    got, _ = _fdk(geo, proj, (1, 1, 1), 1.0, in_place)
    np.testing.assert_allclose(got, ref, rtol=2 * U, atol=nu * 2.0 ** -52 * np.abs(ref).max())


@pytest.mark.parametrize("vol,n_ang,nu,nv,pitch", [
    ((3, 5, 7), 5, 40, 30, 6.0),           # angles split over waves, remainders in x, y and z
    ((9, 8, 8), 3, 12, 10, 4.0),           # most of the volume off the panel
    ((101, 102, 103), 3, 96, 80, 4.0),     # 8 voxels a thread, remainders, all on the panel
    ((104, 101, 100), 2, 64, 30, 2.0),     # the same, half of it off the panel
    ((128, 128, 64), 1, 90, 90, 4.0)])
def test_backprojection_paths(vol, n_ang, nu, nv, pitch):
    print("fdk backprojection", vol, n_ang, nu, nv, flush=True)
    rng = np.random.default_rng(nu)
    proj = rng.normal(0.0, 1.0, (n_ang, nv, nu)).astype(np.float32)
    geo = _geo(nu, nv, pitch)
    h = 1.25
    q, v = _fdk(geo, proj, vol, h)
    ref = recon.fdk_backproject(q, geo, vol, h)
    # coordinates of up to max(nu, nv) pixels carry that many ulps into the weights
    atol = (n_ang + 4 * max(nu, nv)) * 2.0 ** -52 * np.pi * np.abs(q).max() * 2.0
    np.testing.assert_allclose(v, ref, rtol=2 * U, atol=atol)
