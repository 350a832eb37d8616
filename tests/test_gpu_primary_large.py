"""Eq. (7) on a panel of more blocks than a launch has along x: more than 2^24 pixels of 36 rays.

Reference: without attenuation a pixel's value is the sum of its rays' solid angles, in
fp64 from the geometry as the kernel has it; rounded to fp32 on one side only, with the sums
(36 terms of 2^-53) far below that."""
import math

import numpy as np
import pytest

from paper_2201_13191_amd import mcx

pytestmark = pytest.mark.gpu


def test_large_panel():
    import torch
    n, sub, sdd, pitch = 4104, 6, 1000.0, 0.25
    print("primary", n, sub, flush=True)
    g = mcx.Projector(0)
    g.load_phantom(np.zeros((4, 4, 4), np.uint8), np.zeros((4, 4, 4), np.float32), 1.0)
    g.set_geometry(sod_mm=500.0, sdd_mm=sdd, nu=n, nv=n, pu_mm=pitch, pv_mm=pitch, snu=n, snv=n,
                   step_mm=1.0, flags=0)
    g.set_spectrum(np.array([60.0], np.float32), np.array([1.0], np.float32))
    out = torch.full((n, n), float("nan"), device="cuda")
    mcx.mc_primary_expected_async(g.ctx, 0.0, sub, out, torch.cuda.current_stream())
    hu = 0.5 * n * pitch
    omc = float(np.float32(1.0 - sdd / math.sqrt(sdd * sdd + 2 * hu * hu)))
    ref = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    px = torch.arange(n, dtype=torch.float64, device="cuda")
    for b in range(sub):
        for a in range(sub):
            u = (-hu + (px + (a + 0.5) / sub) * pitch).view(1, n)
            v = (-hu + (px + (b + 0.5) / sub) * pitch).view(n, 1)
            r2 = sdd * sdd + u * u + v * v
            ref += sdd / (r2 * r2.sqrt())
    ref *= 60.0 * pitch * pitch / (sub * sub) / (2 * math.pi * omc)
    rel = ((out.double() - ref) / ref).abs().max().item()
    assert rel <= 2.0 ** -24 * 1.01, rel
    g.close()
