"""The tiles of the staged convolutions: the wide layers' blocks of four image rows
(heights that leave a part of a block, channel counts that leave a part of a tile) and
the split reductions of 32-channel tiles over two and four waves, in tiles of 64 and of
32 pixels, with images of one tile's rows and channel counts that are no multiple of 32.

Reference in fp64 on the same bf16 values; the GPU adds 9 cin products, the partial
sums and the bias in fp32: each addition is off by at most an ulp of the magnitudes."""
import numpy as np
import pytest

from paper_2201_13191_amd import mcx, unet

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w,cin,cout", [
    (1, 1030, 128, 16, 40), (1, 1025, 128, 32, 20), (1, 1027, 64, 16, 144), (3, 342, 128, 16, 64),
    (1, 6, 64, 48, 40), (3, 4, 16, 16, 70), (1, 1026, 64, 64, 40),
    (1, 5, 64, 80, 70), (2, 8, 32, 64, 40), (1, 4, 16, 256, 33), (1, 1, 64, 64, 96),
    (1, 3, 64, 272, 40), (1, 4, 32, 80, 20), (1, 520, 64, 64, 48), (2, 4, 16, 288, 100)])
def test_conv_tiles(n, h, w, cin, cout):
    check(n, h, w, cin, cout)


# the split reductions staged by the whole block: tiles of 32 pixels with one group of 64
# channels and with several (wide rows, 2 whole rows of 16, more blocks than 512), tiles of
# 64 (one group, rows of 32 and 16, the long reductions with more blocks)
@pytest.mark.parametrize("n,h,w,cin,cout", [
    (1, 100, 64, 64, 64), (3, 42, 32, 64, 96), (1, 260, 64, 128, 40), (17, 64, 16, 128, 33),
    (1, 257, 64, 64, 20), (9, 60, 32, 128, 17), (17, 64, 16, 192, 32), (1, 600, 64, 256, 20),
    (16, 16, 16, 320, 260)])
def test_conv_shared_tiles(n, h, w, cin, cout):
    check(n, h, w, cin, cout)


# the direct kernel's tiles by the number of blocks: one pixel, parts of tiles, 250 blocks of
# 32 x 32, 188 and 256 of 64 x 32, 258 (which take 64 x 64)
@pytest.mark.parametrize("n,h,w,cin,cout", [
    (1, 1, 1, 32, 1), (2, 5, 7, 48, 33), (3, 8, 8, 256, 256), (2, 50, 40, 32, 33),
    (3, 50, 40, 32, 64), (4, 51, 40, 32, 40), (5, 41, 40, 32, 64)])
def test_conv_direct_tiles(n, h, w, cin, cout):
    check(n, h, w, cin, cout)


def check(n, h, w, cin, cout):
    import torch
    print("conv tiles", n, h, w, cin, cout, flush=True)
    g = mcx.Projector(0)
    gen = torch.Generator(device="cuda").manual_seed(n * 10000 + h)
    x = torch.randn((n, h, w, cin), generator=gen, device="cuda").bfloat16()
    wt = torch.zeros((unet.cout_alloc(cout), 9, cin), device="cuda").bfloat16()
    wt[:cout] = torch.randn((cout, 9, cin), generator=gen, device="cuda").bfloat16()
    b = torch.randn((cout,), generator=gen, device="cuda")
    y = torch.zeros((n, h, w, cout + 16), dtype=torch.bfloat16, device="cuda")
    yf = torch.full((n, h, w, cout), float("nan"), device="cuda")
    mcx.mc_nn_conv3x3_async(g.ctx, x, cin, 0, wt, b, y, cout + 16, 16, n, h, w, cin, cout,
                            relu=0, yf=yf, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    xp = np.pad(x.cpu().double().numpy(), ((0, 0), (1, 1), (1, 1), (0, 0)))
    wd, bd = wt[:cout].cpu().double().numpy(), b.cpu().double().numpy()
    ref = np.zeros((n * h * w, cout)) + bd
    mag = np.zeros((n * h * w, cout)) + np.abs(bd)
    for t in range(9):
        v = np.ascontiguousarray(xp[:, t // 3:t // 3 + h, t % 3:t % 3 + w]).reshape(-1, cin)
        ref += v @ wd[:, t].T
        mag += np.abs(v) @ np.abs(wd[:, t]).T
    tol = (9 * cin + 4) * 2.0 ** -23 * mag
    got = yf.cpu().double().numpy().reshape(-1, cout)
    assert np.all(np.abs(got - ref) <= tol)
    gb = y[..., 16:].cpu().double().numpy().reshape(-1, cout)
    assert np.all(np.abs(gb - ref) <= 2.0 ** -8 * np.abs(ref) + 2 * tol)
    assert not y[..., :16].any()
    g.close()
