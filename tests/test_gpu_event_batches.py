"""Event batches on both sides of the number of interactions a pass waits for, for
every kernel that waits, with photon counts from less than a wave to many:
images do not depend on it (bit for bit the oracle's)."""
import numpy as np
import pytest

from paper_2201_13191_amd import inputs, mcx
from test_gpu_parity import pair

pytestmark = pytest.mark.gpu
BATCHES = (1, 2, 11, 12, 13, 15, 16, 17, 63, 64)


@pytest.mark.parametrize("physics", [0, mcx.MC_PHYS_INCOH_SF | mcx.MC_PHYS_DOPPLER])
@pytest.mark.parametrize("layout", [mcx.MC_LAYOUT_PALETTE_LANE, mcx.MC_LAYOUT_GENERIC])
@pytest.mark.parametrize("n", [1, 50, 60_000])
def test_event_batches(physics, layout, n):
    import torch
    ids, rho = inputs.ellipsoid_phantom(20, 4.0, seed=3)
    geo = dict(sod_mm=200.0, sdd_mm=400.0, nu=30, nv=26, pu_mm=6.0, pv_mm=6.0, snu=15, snv=13,
               step_mm=2.5, flags=0)
    o, g = pair(ids, rho, 4.0, geo, inputs.kramers_spectrum(100, 1.0))
    g.set_layout(layout)
    g.load_phantom(ids, rho, 4.0)
    for side in (o, g):
        side.set_physics(physics)
    po, so = o.project(1.1, n, 4, threads=4)
    per = 30 * 26 + 15 * 13
    out = torch.empty(2 * per, dtype=torch.int64, device="cuda")
    jobs = [dict(phantom=0, angle_rad=1.1, n_photons=n, seed=4, primary_offset=i * per,
                 scatter_offset=i * per + 30 * 26) for i in range(2)]
    for eb in BATCHES:
        print("event batch", eb, "physics", physics, "layout", layout, "n", n, flush=True)
        g.set_launch(128 if eb % 2 else 256, 1, eb)
        p, s = g.project(1.1, n, 4)
        assert np.array_equal(p, po) and np.array_equal(s, so), eb
        mcx.mc_set_batch_launch(g.ctx, 64, 2, eb)
        mcx.mc_project_batch(g.ctx, jobs, out, out.numel(), flags=0,
                             stream=torch.cuda.current_stream())
        h = out.cpu().numpy().reshape(2, per)
        for k in range(2):
            assert np.array_equal(h[k, :30 * 26], po.ravel()), eb
            assert np.array_equal(h[k, 30 * 26:], so.ravel()), eb
    g.close()
