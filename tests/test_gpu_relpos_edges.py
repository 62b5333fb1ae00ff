"""Relative-position attention around the edges of its tiles (32-key sub-blocks, 64-key blocks, 128-query blocks), where the
skewed band changes which of its two accumulators a score comes from; with and without mask and biases, and with a
negative scale.  Same bound as the other attention parity tests."""
import numpy as np
import pytest
import torch

import netfuse_inputs as NI
from test_gpu_parity import check, dev, host, nf, rnd  # noqa: F401  (nf is a fixture)

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


@pytest.mark.parametrize("scale", [None, -0.1])
@pytest.mark.parametrize("S", [1, 2, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 193, 257])
def test_relpos_edges(nf, oracle, S, scale):
    M, B, heads = 2, 1, 2
    qkv = NI.on_bf16_grid(rnd(M, B * S, 3 * heads * 64))
    Kr = NI.on_bf16_grid(rnd(M, 2 * S, heads * 64))
    bw, br, mask = rnd(M, heads * 64, std=0.5), rnd(M, heads * 64, std=0.5), rnd(M, B, S, std=2.0)
    for kw in (dict(bias_w=bw, bias_r=br, mask=mask), dict(bias_r=br), dict()):
        ref = oracle.attention_relpos_packed(qkv, Kr, B, S, heads, scale=scale, out_bf16=True, **kw)
        got = nf.attention_relpos_packed(dev(qkv, BF), dev(Kr, BF), B, S, heads, scale=scale, **{k: dev(v) for k, v in kw.items()})
        check(host(got), ref, BF, "S %d %s" % (S, sorted(kw)))
