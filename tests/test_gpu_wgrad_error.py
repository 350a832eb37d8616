"""The weight gradient's rounding error where its sums are longest: few tiles with many
splits, and many tiles with the caller's few splits, whose waves take long rows of slices.

Reference: the same sum in fp64.  Bound: the error of fp32 sums in the order of the
per-tap kernel, made here: eight pixels' products exact (the matrix instruction rounds its
accumulator once for each eight), a wave's 16-pixel slices in a row (every fourth of its
split), a split's four waves, 32 splits in a row, the groups of 32.
All terms are positive, so that rounding errors pile up along a sum as they do in the sum
of a gradient with a mean."""
import pytest

from paper_2201_13191_amd import mcx

pytestmark = pytest.mark.gpu


def in_a_row(t, dim):
    """fp32 sum over `dim`, one term after the other (each exact or fp32, rounded once)."""
    s = None
    for v in t.unbind(dim):
        s = v.float() if s is None else (s.double() + v.double()).float()
    return s


@pytest.mark.parametrize("n,size,cin,cout,splits", [
    (8, 128, 32, 32, 512), (4, 256, 32, 16, 1024), (8, 64, 192, 64, 86), (8, 64, 384, 384, 8),
    (4, 64, 512, 512, 4), (4, 128, 512, 64, 32), (1, 16, 32, 32, 1), (1, 128, 32, 32, 64)])
def test_wgrad_error(n, size, cin, cout, splits):
    import torch
    print("wgrad error", n, size, cin, cout, splits, flush=True)
    g = mcx.Projector(0)
    gen = torch.Generator(device="cuda").manual_seed(size)
    x = torch.rand((n, size, size, cin), generator=gen, device="cuda").bfloat16()
    dy = torch.rand((n, size, size, cout), generator=gen, device="cuda").bfloat16()
    ws = torch.empty((splits + 1) * 9 * cout * cin, device="cuda")
    dw = torch.empty((cout, 9, cin), device="cuda")
    mcx.mc_nn_conv3x3_wgrad_async(g.ctx, x, cin, 0, dy, cout, 0, n, size, size, cin, cout, splits,
                                  ws, dw, torch.cuda.current_stream())
    # the centre tap of one tile of channels; slices (two halves each) padded with zeros to
    # whole splits
    co = min(32, cout)
    xs = x[..., :32].double().reshape(-1, 8, 32)
    ys = dy[..., :co].double().reshape(-1, 8, co).transpose(1, 2).contiguous()
    halves = torch.bmm(ys, xs)
    exact = halves.sum(0)
    per = -(-halves.shape[0] // (2 * splits))
    per += -per % 4
    pad = torch.zeros((2 * per * splits - halves.shape[0], co, 32), dtype=torch.float64,
                      device="cuda")
    parts = torch.cat([halves, pad]).view(splits, per // 4, 4, 2, co, 32).transpose(2, 3)
    parts = in_a_row(in_a_row(parts.reshape(splits, per // 2, 4, co, 32), 1), 1)
    groups = torch.stack([in_a_row(p, 0) for p in parts.split(32)])
    order = in_a_row(groups, 0)

    def rms(v):
        return float((v.double() - exact).square().mean().sqrt())

    got = rms(dw[:co, 4, :32])
    assert got <= rms(order), (got, rms(order))
    g.close()
