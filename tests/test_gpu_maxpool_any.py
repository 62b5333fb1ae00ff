"""The 3 x 3 stride-2 max-pool over rows of any width in bf16 and float32: widths about the 8 columns and 4 outputs of a thread, one row, odd
and even numbers of rows, bases off every alignment, NaN, infinities and the lowest finite values.  The maximum is exact."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


# the kernel for any window: below 8 columns, 2^14 outputs, two rows, and at the line
GENERIC = [(3, 5, 7, 7), (2, 9, 40, 40), (1, 4, 1, 9000), (1, 2048, 3, 8)]
ROWS = [(1, 2049, 4, 8), (2, 1700, 3, 9), (1, 2050, 5, 10), (2, 700, 6, 15), (1, 911, 3, 17), (3, 23, 9, 100), (1, 7, 113, 113), (1, 12, 6, 1030)]


@pytest.mark.parametrize("B,C,H,W", GENERIC + ROWS)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shift", [0, 1])
def test_values(oracle, B, C, H, W, dtype, shift):
    import paper_2009_13062_amd as nf
    x = torch.randn(B, C, H, W, generator=torch.Generator().manual_seed(H * W)).to(dtype).float().numpy()
    f = x.reshape(-1)
    f[::5], f[1::7], f[2::11] = np.nan, -np.inf, np.inf
    x[:, 0] = torch.finfo(dtype).min
    Ho, Wo = (H - 1) // 2 + 1, (W - 1) // 2 + 1
    assert (W >= 8 and Ho > 1 and B * C * Ho * Wo > 2 ** 14) == ((B, C, H, W) in ROWS)
    xs = torch.empty(x.size + 9, dtype=dtype, device="cuda")
    ys = torch.full((B * C * Ho * Wo + 9,), 77.0, dtype=dtype, device="cuda")
    xin = xs[shift:shift + x.size].view(B, C, H, W)
    xin.copy_(torch.from_numpy(x))
    out = ys[shift:shift + B * C * Ho * Wo].view(B, C, Ho, Wo)
    nf.maxpool2d(xin, 3, 2, 1, out=out)
    assert np.array_equal(out.float().cpu().numpy(), oracle.maxpool2d(x, 3, 2, 1))
    assert (ys[:shift] == 77).all() and (ys[shift + out.numel():] == 77).all()
