"""float32 pointwise convolutions and matmuls whose rows are no whole 16 bytes (planes and output widths around the edges of the tiles), against
float64: the last pieces of a row run into the next one and, in the last row, past the end of the operand.  What they meet there, a NaN among it,
reaches no result.  The bound: K products and the additions after them, each rounded once, of the sum of their sizes."""
import pytest
import torch

from test_gpu_parity import nf  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


def close(got, ref, size, K):
    assert ((got.cpu().double() - ref).abs() <= (K + 4) * 2.0 ** -24 * size).all()


@pytest.mark.parametrize("hw", [1, 3, 5, 7, 9, 13, 25])
@pytest.mark.parametrize("cin,cout,B", [(20, 16, 1), (33, 70, 2), (64, 17, 3), (256, 40, 1), (1540, 20, 1)])
def test_pointwise(nf, hw, cin, cout, B):
    M = 3
    g = torch.Generator().manual_seed(100 * hw + cin)
    x, w = torch.randn(B, M * cin, hw, hw, generator=g), torch.randn(M * cout, cin, 1, 1, generator=g)
    r = torch.randn(B, M * cout, hw, hw, generator=g)
    got = nf.conv2d(x.cuda(), w.cuda(), M, residual=r.cuda())
    xd, wd = x.double().view(B, M, cin, hw * hw), w.double().view(1, M, cout, cin)
    ref = (wd @ xd).view(r.shape) + r
    close(got, ref, (wd.abs() @ xd.abs()).view(r.shape) + r.abs(), cin)


@pytest.mark.parametrize("K,N,Nout", [(33, 5, 1), (50, 65, 99), (32, 130, 63), (9, 64, 257), (62, 1500, 99), (63, 20, 1001)])
def test_matmul(nf, K, N, Nout):
    M = 4
    g = torch.Generator().manual_seed(K + Nout)
    x, w = torch.randn(M, N, K, generator=g), torch.randn(M, K, Nout, generator=g)
    b, r = torch.randn(M, Nout, generator=g), torch.randn(M, N, Nout, generator=g)
    got = nf.linear(x.cuda(), w.cuda(), bias=b.cuda(), residual=r.cuda())
    xd, wd = x.double(), w.double()
    close(got, xd @ wd + b[:, None] + r, xd.abs() @ wd.abs() + b[:, None].abs() + r.abs(), K)


def test_a_column_keeps_its_nan(nf):
    x, w = torch.randn(2, 70, 50), torch.randn(2, 50, 67)
    w[0, :, 0] = float("nan")                                 # read behind column 66 of the row before
    w[1, 0, 0] = float("inf")                                 # behind the last row of the model before
    got = nf.linear(x.cuda(), w.cuda()).cpu()
    assert got[0, :, 0].isnan().all() and got[0, :, 1:].isfinite().all()
    assert not got[1, :, 0].isfinite().any() and got[1, :, 1:].isfinite().all()


@pytest.mark.parametrize("hw", [1, 5, 7, 15])
@pytest.mark.parametrize("cig,cog,g", [(4, 16, 1), (16, 4, 3), (17, 3, 2), (17, 4, 64), (7, 32, 5), (7, 33, 3), (8, 8, 5), (8, 9, 5), (16, 13, 4), (64, 1, 2),
                                          (65, 1, 64), (8, 28, 64), (1, 230, 1), (1, 231, 1)])
def test_pointwise_of_narrow_groups(nf, hw, cig, cog, g):
    """Either side of the line between the kernel of one thread per output and the matrix kernel."""
    M, B = 2, 2
    gen = torch.Generator().manual_seed(100 * hw + cig)
    x, w = torch.randn(B, M * g * cig, hw, hw, generator=gen), torch.randn(M * g * cog, cig, 1, 1, generator=gen)
    got = nf.conv2d(x.cuda(), w.cuda(), M, g)
    xd, wd = x.double().view(B, M * g, cig, hw * hw), w.double().view(1, M * g, cog, cig)
    close(got, (wd @ xd).view(got.shape), (wd.abs() @ xd.abs()).view(got.shape), cig)


def test_an_odd_plane_is_no_slower_than_a_larger_even_one(nf):
    """8 -> 28 and 16 -> 13 channels per group over 15 x 15 against 16 x 16 positions: the same kernel for both."""
    def us(cig, cog, g, hw):
        x, w = torch.randn(1, 32 * g * cig, hw, hw, device="cuda"), torch.randn(32 * g * cog, cig, 1, 1, device="cuda")
        out, best = nf.conv2d(x, w, 32, g), 1e9
        for _ in range(6):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(10):
                nf.conv2d(x, w, 32, g, out=out)
            end.record()
            end.synchronize()
            best = min(best, start.elapsed_time(end) * 100)
        return best
    for cig, cog in ((8, 28), (16, 13)):
        assert us(cig, cog, 64, 15) < 1.5 * us(cig, cog, 64, 16)
