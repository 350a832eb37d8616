"""Hand-out of pseudo-particles to a wave's lanes: splits from one to more than a
wave, photon counts that leave lanes without a photon, event batches on both
sides of the number of free lanes that starts a round, both point-detector
modes.  Every image must be the default shape's, bit for bit, and the oracle's
within the 1e-9 of the point-detector parity tests (a score may differ by a
least significant bit)."""
import numpy as np
import pytest

import oracle
from paper_2201_13191_amd import inputs, mcx
from test_gpu_parity import pair, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,split,rr,n", [
    ("mixed", 1, 0.0, 3000), ("mixed", 2, 0.4, 1), ("mixed", 20, 1.0, 37), ("mixed", 20, 1.0, 4000),
    ("mixed", 63, 0.2, 700), ("mixed", 64, 0.0, 130), ("mixed", 65, 0.5, 129),
    ("mixed", 1024, 0.05, 40), ("point", 7, 0.1, 2000), ("point", 70, 0.01, 300)])
def test_pairs(mode, split, rr, n):
    ids, rho = inputs.ellipsoid_phantom(24, 3.0, seed=9)
    geo = dict(sod_mm=200.0, sdd_mm=400.0, nu=48, nv=40, pu_mm=4.0, pv_mm=4.0, snu=24, snv=10,
               step_mm=2.0, flags=0)
    o, g = pair(ids, rho, 3.0, geo, inputs.kramers_spectrum(120, 1.0))
    g.set_estimator(dict(mixed=mcx.MC_SCORE_POINT_MIXED, point=mcx.MC_SCORE_POINT)[mode], split, rr)
    o.set_estimator(dict(mixed=oracle.SCORE_POINT_MIXED, point=oracle.SCORE_POINT)[mode], split, rr)
    print("pairs", mode, split, rr, n, flush=True)
    ref = g.project(0.4, n, 5)
    po, so = o.project(0.4, n, 5, threads=4)
    assert np.array_equal(ref[0], po)
    assert rel_l2(ref[1], so) <= 1e-9 if so.any() else not ref[1].any()
    for shape in [(64, 1, 1), (64, 2, 7), (128, 1, 23), (192, 0, 24), (256, 1, 25), (256, 0, 64)]:
        print("  shape", shape, flush=True)
        g.set_launch(*shape)
        got = g.project(0.4, n, 5)
        assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1]), shape
    g.close()
