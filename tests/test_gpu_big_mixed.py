"""Objects above 64 MiB of voxels on both sides of the share of non-uniform cells up to which
they march in groups of 4 steps: images bit for bit the oracle's, in the storages of ids with
densities and of codes."""
import numpy as np
import pytest

from paper_2201_13191_amd import inputs, mcx
from test_gpu_parity import pair

pytestmark = pytest.mark.gpu


def _noise(shape, share, generic, seed):
    """A block of noise over about `share` of the object in its middle, air around it."""
    rng = np.random.default_rng(seed)
    ids = np.zeros(shape, np.uint8)
    rho = np.full(shape, 0.001205, np.float32)
    side = [max(4, int(n * share ** (1 / 3))) for n in shape]
    box = tuple(slice((n - s) // 2, (n - s) // 2 + s) for n, s in zip(shape, side))
    ids[box] = 1
    f = rng.random(side, dtype=np.float32)
    rho[box] = 0.8 + (0.4 * f if generic else np.floor(f * 16) * np.float32(0.025))
    return ids, rho


@pytest.mark.parametrize("generic,share", [(True, 0.15), (True, 0.4), (False, 0.02),
                                           (False, 0.2)])
def test_mixed_shares(generic, share):
    shape, h = ((241, 240, 239), 0.5) if generic else ((262, 512, 508), 0.25)
    ids, rho = _noise(shape, share, generic, 3)
    geo = dict(sod_mm=300.0, sdd_mm=600.0, nu=60, nv=44, pu_mm=4.0, pv_mm=4.0, snu=30, snv=22,
               step_mm=0.6, flags=0)
    o, g = pair(ids, rho, h, geo, inputs.kramers_spectrum(120, 1.0))
    print("big mixed object", generic, share, flush=True)
    po, so = o.project(0.4, 200_000, 8, threads=8)
    p, s = g.project(0.4, 200_000, 8)
    assert po.sum() > 0 and so.sum() > 0
    assert np.array_equal(p, po) and np.array_equal(s, so)
    g.close()
