"""The weight gradient of inputs with infinities: each tap takes the pixels that it meets
and no others, in every row of a strip.

Reference: the products that a tap has, in fp64 (padded inputs are zeros, as they are for
the kernel): finite taps within the half-ulps of their terms, the others the same infinity
or NaN."""
import numpy as np
import pytest

from paper_2201_13191_amd import mcx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w,splits,at", [
    (1, 6, 16, 1, [(0, 0, 3)]), (1, 6, 16, 1, [(0, 5, 0)]), (2, 5, 32, 2, [(1, 0, 31)]),
    (2, 40, 32, 4, [(0, 39, 7), (1, 0, 20)]), (1, 1, 16, 1, [(0, 0, 15)]),
    (1, 33, 48, 3, [(0, 16, 16)])])
def test_infinite_inputs(n, h, w, splits, at):
    import torch
    print("wgrad infinities", n, h, w, splits, at, flush=True)
    cin, cout = 32, 16
    g = mcx.Projector(0)
    gen = torch.Generator(device="cuda").manual_seed(h)
    x = (torch.rand((n, h, w, cin), generator=gen, device="cuda") + 0.5).bfloat16()
    dy = (torch.rand((n, h, w, cout), generator=gen, device="cuda") + 0.5).bfloat16()
    for c, (i, r, col) in enumerate(at):
        x[i, r, col, c] = float("inf")
    ws = torch.empty((splits + 1) * 9 * cout * cin, device="cuda")
    dw = torch.empty((cout, 9, cin), device="cuda")
    mcx.mc_nn_conv3x3_wgrad_async(g.ctx, x, cin, 0, dy, cout, 0, n, h, w, cin, cout, splits, ws,
                                  dw, torch.cuda.current_stream())
    torch.cuda.synchronize()
    xp = np.pad(x.cpu().double().numpy(), ((0, 0), (1, 1), (1, 1), (0, 0)))
    y = dy.cpu().double().numpy().reshape(-1, cout)
    ref = np.zeros((cout, 9, cin))
    for t in range(9):
        ref[:, t] = y.T @ xp[:, t // 3:t // 3 + h, t % 3:t % 3 + w].reshape(-1, cin)
    got = dw.cpu().double().numpy()
    fin = np.isfinite(ref)
    assert fin[:, :, len(at):].all() and (at[0][1] not in (0, h - 1) or fin[:, :, 0].any())
    np.testing.assert_array_equal(got[~fin], ref[~fin])
    tol = (n * h * w + splits) * 2.0 ** -24 * ref[fin]
    assert np.all(np.abs(got[fin] - ref[fin]) <= tol)
    g.close()
