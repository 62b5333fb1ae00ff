"""Masked attention around the edges of its 64-key blocks (the mask of a block passes through LDS): against the oracle; a
mask of zeros against no mask at a scale that is a power of two in log2 units (the same bits: scaling is then exact);
rows whose keys are all masked with the lowest values of the type."""
import numpy as np
import pytest
import torch

import netfuse_inputs as NI
from test_gpu_parity import check, dev, host, nf, rnd  # noqa: F401  (nf is a fixture)

pytestmark = pytest.mark.gpu
BF, F32 = torch.bfloat16, torch.float32
LOWEST = float(np.finfo(np.float32).min)


@pytest.mark.parametrize("S", [1, 63, 64, 65, 127, 128, 129, 200])
def test_mask_edges(nf, oracle, S):
    M, B, heads = 2, 2, 2
    qkv = NI.on_bf16_grid(rnd(M, B * S, 3 * heads * 64))
    mask = rnd(M, B, S, std=2.0)
    mask[:, :, S // 2 + 1:] = -10000.0
    got = nf.attention_packed(dev(qkv, BF), B, S, heads, mask=dev(mask))
    check(host(got), oracle.attention_packed(qkv, B, S, heads, mask=mask, out_bf16=True), BF, "S %d" % S)
    mask[0, 0] = -3.0e38
    mask[1, 1, 0] = float("nan")                              # stays in its own sequence
    bad = host(nf.attention_packed(dev(qkv, BF), B, S, heads, mask=dev(mask))).reshape(M, B, S, -1)
    ok = host(got).reshape(M, B, S, -1)
    assert (bad[0, 1] == ok[0, 1]).all() and (bad[1, 0] == ok[1, 0]).all()
    assert np.isnan(bad[1, 1]).all() and np.isfinite(bad[0, 0]).all()


@pytest.mark.parametrize("S", [1, 63, 64, 65, 200])
def test_mask_of_zeros_changes_no_bit(nf, S):
    qkv, kr = dev(rnd(2, S, 3 * 128), BF), dev(rnd(2, 2 * S, 128), BF)
    zero = torch.zeros(2, 1, S, device="cuda")
    scale = 0.125 * float(np.log(2.0))                        # x log2 e = 1 / 8 in float32
    assert torch.equal(nf.attention_packed(qkv, 1, S, 2, scale=scale, mask=zero), nf.attention_packed(qkv, 1, S, 2, scale=scale))
    assert torch.equal(nf.attention_relpos_packed(qkv, kr, 1, S, 2, scale=scale, mask=zero),
                       nf.attention_relpos_packed(qkv, kr, 1, S, 2, scale=scale))


@pytest.mark.parametrize("low", [-2.0e38, -3.0e38, LOWEST], ids=["-2e38", "-3e38", "lowest"])
@pytest.mark.parametrize("dtype,S,d", [(BF, 3, 64), (BF, 65, 64), (BF, 200, 64), (BF, 70, 32), (F32, 5, 64), (F32, 65, 64), (F32, 130, 20)],
                         ids=lambda v: str(v))
def test_lowest_mask_gives_even_weights(nf, dtype, S, d, low):
    """Every score is absorbed by such a mask, so the row is the mean of the values; weights of 1 are exact in bfloat16, the
    sum has S float32 roundings and the result one of its type.  One key left unmasked takes all the weight."""
    M, heads = 2, 2
    H = heads * d
    qkv = NI.on_bf16_grid(rnd(M, S, 3 * H))
    kr = dev(rnd(M, 2 * S, H), dtype)
    mask = np.zeros((M, 1, S), np.float32)
    mask[0] = low
    mask[1, 0, 1:] = low
    v = qkv[:, :, 2 * H:].astype(np.float64)
    tol = 2.0 ** -8 if dtype == BF else 2.0 ** -22
    for got in (nf.attention_packed(dev(qkv, dtype), 1, S, heads, mask=dev(mask)),
                nf.attention_relpos_packed(dev(qkv, dtype), kr, 1, S, heads, mask=dev(mask))):
        got = host(got)
        mean = v[0].mean(axis=0)
        assert (np.abs(got[0] - mean) <= tol * np.abs(mean) + S * 2.0 ** -23 * np.abs(v[0]).max()).all()
        assert (np.abs(got[1] - v[1, 0]) <= tol * np.abs(v[1, 0])).all()


@pytest.mark.parametrize("S", [3, 65])
def test_keys_past_the_end_have_no_weight_at_any_scale(nf, S):
    """Also at a scale that makes every score vanish: the mean over the S keys, not over the padded block."""
    qkv, kr = NI.on_bf16_grid(rnd(1, S, 3 * 128)), dev(rnd(1, 2 * S, 128), BF)
    mean = qkv[0, :, 256:].astype(np.float64).mean(axis=0)
    for got in (nf.attention_packed(dev(qkv, BF), 1, S, 2, scale=1.2e-38),
                nf.attention_relpos_packed(dev(qkv, BF), kr, 1, S, 2, scale=1.2e-38)):
        assert (np.abs(host(got)[0] - mean) <= 2.0 ** -8 * np.abs(mean) + S * 2.0 ** -23 * np.abs(qkv).max()).all()
