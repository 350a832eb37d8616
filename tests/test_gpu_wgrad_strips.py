"""The weight gradient's strips of 16-pixel columns: images of one row and one
column, strips that end inside a column and go on in the next image, channel
counts that leave tiles part full, channel slices, one split and more splits than
slices, and a width that takes the other kernel.

Reference in fp64 on the same bf16 values; the GPU adds in fp32, at most
n h w + splits terms in a row: that many half-ulps of the terms' magnitudes."""
import numpy as np
import pytest

from paper_2201_13191_amd import mcx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w,cin,cout,splits,pad", [
    (1, 1, 16, 16, 16, 1, 0), (1, 1, 48, 32, 32, 5, 16), (3, 5, 16, 48, 80, 4, 0),
    (2, 7, 32, 64, 16, 64, 0), (5, 9, 48, 96, 64, 3, 32), (1, 130, 16, 16, 48, 2, 0),
    (2, 33, 64, 32, 128, 16, 16), (4, 64, 64, 80, 32, 86, 0), (2, 6, 24, 32, 32, 3, 0)])
def test_wgrad_strips(n, h, w, cin, cout, splits, pad):
    import torch
    print("wgrad", n, h, w, cin, cout, splits, pad, flush=True)
    g = mcx.Projector(0)
    gen = torch.Generator(device="cuda").manual_seed(n * 1000 + h)
    x = torch.randn((n, h, w, cin + pad), generator=gen, device="cuda").bfloat16()
    dy = torch.randn((n, h, w, cout + pad), generator=gen, device="cuda").bfloat16()
    ws = torch.full(((splits + 1) * 9 * cout * cin,), float("nan"), device="cuda")
    dw = torch.full((cout, 9, cin), float("nan"), device="cuda")
    mcx.mc_nn_conv3x3_wgrad_async(g.ctx, x, cin + pad, pad, dy, cout + pad, pad, n, h, w, cin,
                                  cout, splits, ws, dw, torch.cuda.current_stream())
    torch.cuda.synchronize()
    xs, ys = x[..., pad:].cpu().double().numpy(), dy[..., pad:].cpu().double().numpy()
    xp = np.pad(xs, ((0, 0), (1, 1), (1, 1), (0, 0)))
    ref, mag = np.zeros((cout, 9, cin)), np.zeros((cout, 9, cin))
    for t in range(9):
        v = xp[:, t // 3:t // 3 + h, t % 3:t % 3 + w].reshape(-1, cin)
        y = ys.reshape(-1, cout)
        ref[:, t], mag[:, t] = y.T @ v, np.abs(y).T @ np.abs(v)
    tol = (n * h * w + splits) * 2.0 ** -24 * mag + 1e-30
    assert np.all(np.abs(dw.cpu().numpy() - ref) <= tol)
    g.close()
