"""Masked attention around the edges of its 64-key blocks (the mask of a block passes through LDS): against the oracle, and
a mask of zeros against no mask at a scale that is a power of two (the same bits: scaling is then exact)."""
import pytest
import torch

import netfuse_inputs as NI
from test_gpu_parity import check, dev, host, nf, rnd  # noqa: F401  (nf is a fixture)

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


@pytest.mark.parametrize("S", [1, 63, 64, 65, 127, 128, 129, 200])
def test_mask_edges(nf, oracle, S):
    M, B, heads = 2, 2, 2
    qkv = NI.on_bf16_grid(rnd(M, B * S, 3 * heads * 64))
    mask = rnd(M, B, S, std=2.0)
    mask[:, :, S // 2 + 1:] = -10000.0
    got = nf.attention_packed(dev(qkv, BF), B, S, heads, mask=dev(mask))
    check(host(got), oracle.attention_packed(qkv, B, S, heads, mask=mask, out_bf16=True), BF, "S %d" % S)
    mask[0, 0] = -3.0e38                                      # a whole row at the lowest value: even weights
    mask[1, 1, 0] = float("nan")                              # stays in its own sequence
    bad = host(nf.attention_packed(dev(qkv, BF), B, S, heads, mask=dev(mask))).reshape(M, B, S, -1)
    ok = host(got).reshape(M, B, S, -1)
    assert (bad[0, 1] == ok[0, 1]).all() and (bad[1, 0] == ok[1, 0]).all()
