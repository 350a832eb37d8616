"""The wide layers' convolutions on images of few rows, whose four waves a block take tiles of
their own: heights 1, 2 and 5, tile counts that leave a part of the last block, images that
end inside a block.  Their results (reference and tolerance as for the other tiles), and that
images of one row take no more than half again the time of the same pixels in fours (the same
products; rows past an image's end cost 2.2 times)."""
import pytest

from paper_2201_13191_amd import mcx, unet
from test_gpu_conv_tiles import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w,cin,cout", [
    (2049, 1, 64, 16, 40), (683, 1, 192, 32, 20), (513, 2, 128, 16, 70), (411, 5, 64, 48, 32),
    (103, 5, 256, 16, 33), (1, 2, 65600, 16, 16)])
def test_low_images(n, h, w, cin, cout):
    check(n, h, w, cin, cout)


def test_one_row_costs_no_more():
    import torch
    g = mcx.Projector(0)
    cin, cout, pixels = 96, 32, 131072
    x = torch.randn((pixels, cin), device="cuda").bfloat16()
    w = torch.randn((unet.cout_alloc(cout), 9, cin), device="cuda").bfloat16()
    y = torch.empty((pixels, cout), device="cuda").bfloat16()

    def us(h):
        best = 1e9
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(20):
                mcx.mc_nn_conv3x3_async(g.ctx, x, cin, 0, w, None, y, cout, 0, pixels // (64 * h),
                                        h, 64, cin, cout, stream=torch.cuda.current_stream())
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 50)
        return best

    one, four = us(1), us(4)
    print("one row", one, "four rows", four, flush=True)
    assert one <= 1.5 * four
    g.close()
