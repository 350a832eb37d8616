"""The march probe on an object above 64 MiB of voxels, where it marches in groups of 4 steps
as the transport does: the step counts of the oracle's photons, which do not interact without
density, and the code sum of an object of one code."""
import numpy as np
import pytest

import oracle
from paper_2201_13191_amd import inputs, mcx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,generic", [((262, 512, 510), False), ((240, 239, 242), True)])
def test_probe_big_object(shape, generic):
    import torch
    print("probe", shape, generic, flush=True)
    ids = np.ones(shape, np.uint8)
    rho = np.zeros(shape, np.float32)
    geo = dict(sod_mm=300.0, sdd_mm=700.0, nu=40, nv=24, pu_mm=6.0, pv_mm=8.0, snu=20, snv=12,
               step_mm=0.31, flags=0)
    spec = inputs.kramers_spectrum(90, 1.0)
    n, seed, angle = 30_000, 5, 0.9
    o, g = oracle.Oracle(), mcx.Projector(0)
    if generic:
        g.set_layout(mcx.MC_LAYOUT_GENERIC)
    for side in (o, g):
        side.load_phantom(ids, rho, 0.4)
        side.set_geometry(**geo)
        side.set_spectrum(*spec)
    o.project(angle, n, seed, threads=8)
    steps = o.stats()["steps"]
    d = torch.zeros(2, dtype=torch.int64, device="cuda")
    mcx.mc_march_probe_async(g.ctx, angle, n, seed, 20, d)
    torch.cuda.synchronize()
    assert steps > 0 and d.tolist() == [steps if generic else 0, steps]
    g.close()
