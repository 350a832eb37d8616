"""Eq. (7) on panels that take a wave per block: rounds of 64 rays that begin and end inside a
pixel, last blocks that are part full, one and many bins, more materials than the usual set,
both voxel storages, and the panels next to each line of the rule (2048 and 4096 waves).

Reference and tolerance as for the four waves: the oracle's fp64 sum, half an ulp each side."""
import numpy as np
import pytest

import oracle
from paper_2201_13191_amd import inputs, mcx

pytestmark = pytest.mark.gpu
MATS = inputs.DEFAULT_MATERIALS


@pytest.mark.parametrize("sub,nu,nv,bins,n_mat,generic", [
    (1, 511, 513, 2, 5, False), (1, 363, 362, 1, 5, True), (1, 362, 362, 1, 5, False),
    (2, 257, 256, 70, 5, True), (3, 172, 171, 3, 16, False), (5, 103, 103, 2, 5, False),
    (6, 86, 87, 60, 5, False), (8, 65, 64, 5, 5, False), (9, 58, 57, 1, 6, True),
    (14, 37, 37, 2, 5, False)])
def test_primary_waves(sub, nu, nv, bins, n_mat, generic):
    import torch
    print("primary waves", sub, nu, nv, bins, n_mat, generic, flush=True)
    rng = np.random.default_rng(sub * 100 + nu)
    shape = (11, 9, 13)
    ids = rng.integers(0, n_mat, shape).astype(np.uint8)
    rho = rng.uniform(0.0, 3.0, shape).astype(np.float32)
    if not generic:
        rho = np.round(rho * 2).astype(np.float32) / 2
    mats = [dict(MATS[i % 5], z_eff=MATS[i % 5]["z_eff"] + 0.25 * (i // 5)) for i in range(n_mat)]
    geo = dict(sod_mm=120.0, sdd_mm=240.0, nu=nu, nv=nv, pu_mm=60.0 / nu, pv_mm=50.0 / nv, snu=nu,
               snv=nv, step_mm=0.8, flags=0)
    e = np.linspace(20.0, 140.0, bins).astype(np.float32)
    w = rng.uniform(0.1, 1.0, bins).astype(np.float32)
    g, o = mcx.Projector(0), oracle.Oracle()
    for side in (g, o):
        side.set_materials(mats)
        if generic and side is g:
            side.set_layout(mcx.MC_LAYOUT_GENERIC)
        side.load_phantom(ids, rho, 2.0)
        side.set_geometry(**geo)
        side.set_spectrum(e, w)
    out = torch.full((nv, nu), float("nan"), device="cuda")
    mcx.mc_primary_expected_async(g.ctx, 0.7, sub, out)
    torch.cuda.synchronize()
    np.testing.assert_allclose(out.cpu().numpy(), o.primary_expected(0.7, sub), rtol=2.0 ** -23)
    g.close()
