"""Layer norm of rows in whole 4-feature pieces around the multiples of 256 that set how many a lane takes, up to and past the
register limit of 1024, in both merge layouts, with and without a residual and at odd and even row counts."""
import numpy as np
import pytest
import torch

import netfuse_inputs as NI
from test_gpu_parity import check, dev, host, nf, rnd  # noqa: F401  (nf is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("M,rows,H", [(3, 7, H) for H in (4, 252, 256, 260, 508, 512, 516, 768, 1020, 1024, 1028)] +
                         [(2, 8200, H) for H in (4, 260, 512, 516, 768)])    # two rows per wavefront up to 512 features
def test_layernorm_widths(nf, oracle, M, rows, H, dtype):
    bf = dtype == torch.bfloat16
    grid = NI.on_bf16_grid if bf else (lambda a: a)
    x, res = grid(rnd(M, rows, H)), grid(rnd(M, rows, H))
    g, b = rnd(M * H, std=0.2) + 1, rnd(M * H, std=0.2)
    for r in (None, res):
        got = nf.layernorm(dev(x, dtype), dev(g), dev(b), M, residual=None if r is None else dev(r, dtype))
        ref = oracle.layernorm(x, g, b, M, residual=r, out_bf16=bf)
        check(host(got), ref, dtype, "H %d" % H)
    flat = lambda a: np.ascontiguousarray(a.transpose(1, 0, 2).reshape(rows, M * H))
    chan = nf.layernorm(dev(flat(x), dtype), dev(g), dev(b), M, residual=dev(flat(res), dtype), layout=nf.MERGE_CHANNEL)
    assert torch.equal(chan.view(rows, M, H).transpose(0, 1), got)
