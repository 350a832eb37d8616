"""Objects above 64 MiB of voxels march in groups of 4 steps: images of all three
storages, with and without binding effects, with steps of at most and of more
than a voxel, bit for bit the oracle's (the 512^3 benchmark object is covered by
the full-size tests)."""
import numpy as np
import pytest

from paper_2201_13191_amd import inputs, mcx
from test_gpu_parity import pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,physics,step", [
    ("generic", 0, 0.5), ("generic", 3, 1.3), ("shared", 0, 0.4), ("lane", 3, 0.4)])
def test_big_objects(storage, physics, step):
    if storage == "generic":
        shape, h = (240, 239, 242), 0.5
    else:
        shape, h = (262, 512, 508), 0.25
    ids, rho = inputs.ellipsoid_phantom(0, h, seed=11, shape=shape)
    if storage == "generic":
        rng = np.random.default_rng(2)
        obj = ids > 0
        rho[obj] *= rng.uniform(0.9, 1.1, int(obj.sum())).astype(np.float32)
    elif storage == "shared":       # 10 densities along z for each of the 21 pairs
        k = (np.arange(shape[0]) * 10 // shape[0]).astype(np.float32)
        rho *= 1.0 + 0.01 * k[:, None, None]
    assert ids.size * (5 if storage == "generic" else 1) > 64 << 20
    geo = dict(sod_mm=300.0, sdd_mm=600.0, nu=60, nv=44, pu_mm=4.0, pv_mm=4.0, snu=30, snv=22,
               step_mm=step, flags=0)
    o, g = pair(ids, rho, h, geo, inputs.kramers_spectrum(120, 1.0))
    assert g.layout()[0] == dict(generic=mcx.MC_LAYOUT_GENERIC, shared=mcx.MC_LAYOUT_PALETTE_SHARED,
                                 lane=mcx.MC_LAYOUT_PALETTE_LANE)[storage]
    for side in (o, g):
        side.set_physics(physics)
    print("big object", storage, physics, step, flush=True)
    po, so = o.project(0.9, 200_000, 6, threads=8)
    for shape_ in [(0, 0, 0), (128, 1, 5)]:
        g.set_launch(*shape_)
        p, s = g.project(0.9, 200_000, 6)
        assert po.sum() > 0 and so.sum() > 0
        assert np.array_equal(p, po) and np.array_equal(s, so), shape_
    g.close()
