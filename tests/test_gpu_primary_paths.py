"""Eq. (7)'s kernel at the sizes where its split of rays, steps and bins changes:
sub-pixel counts whose rays fill, straddle and exceed the 64 of a block, pixel
counts that leave a block part full, few and many bins, more materials than the
usual set, both voxel storages.

Reference: the oracle's fp64 sum, rounded to fp32 once on both sides: half an ulp
each, and the sums' order (some hundred terms of 2^-53) far below it."""
import numpy as np
import pytest

import oracle
from paper_2201_13191_amd import inputs, mcx

pytestmark = pytest.mark.gpu
MATS = inputs.DEFAULT_MATERIALS


@pytest.mark.parametrize("sub,nu,nv,bins,n_mat,generic", [
    (1, 9, 7, 1, 5, False), (1, 64, 3, 3, 5, True), (2, 17, 5, 4, 5, False),
    (3, 8, 8, 29, 1, False), (5, 6, 5, 30, 5, True), (7, 5, 4, 31, 16, False),
    (8, 3, 3, 60, 6, False), (9, 3, 2, 119, 5, False), (12, 2, 2, 7, 16, True)])
def test_primary_splits(sub, nu, nv, bins, n_mat, generic):
    import torch
    print("primary", sub, nu, nv, bins, n_mat, generic, flush=True)
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
    ref = o.primary_expected(0.7, sub)
    np.testing.assert_allclose(out.cpu().numpy(), ref, rtol=2.0 ** -23)
    g.close()
