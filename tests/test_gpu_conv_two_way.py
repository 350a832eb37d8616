"""The two-way split reductions in tiles of 64 channels: just past the shortest reduction that
takes them, rows of 64, 32 and 16 pixels, a last tile of 64 part empty, a part-filled last
round, and the neighbours that keep tiles of 32 (a shorter reduction, an odd number of
32-channel tiles, a last round half empty).  Reference and tolerance as for the other tiles."""
import pytest

from test_gpu_conv_tiles import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w,cin,cout", [
    (4, 64, 64, 144, 256), (4, 64, 64, 128, 256), (17, 32, 32, 176, 250), (4, 64, 64, 144, 192),
    (62, 16, 16, 144, 260), (1, 1007, 64, 272, 64), (17, 64, 64, 144, 64), (3, 120, 192, 144, 120)])
def test_conv_two_way_tiles(n, h, w, cin, cout):
    check(n, h, w, cin, cout)
