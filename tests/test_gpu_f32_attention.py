"""float32 attention around the edges of its 16-query groups, 64-key (32-key above 64 features) stages and feature blocks, where the number of key
shares changes, against float64.  The bound: a score is a sum of d products (d + 2 roundings of the sum of their sizes), a weight's
relative error is that of its score and of the row's maximum plus the exponential's, and S weighted values are added."""
import pytest
import torch

from test_gpu_parity import nf  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


def problem(M, B, S, heads, d, masked):
    g = torch.Generator().manual_seed(100 * S + d)
    qkv = torch.randn(M, B * S, 3 * heads * d, generator=g)
    mask = None
    if masked:
        mask = torch.randn(M, B, S, generator=g)
        mask[:, :, S // 2 + 1:] = -10000.0
    return qkv, mask


def reference(qkv, mask, M, B, S, heads, d, scale):
    q, k, v = [t.reshape(M, B, S, heads, d).permute(0, 1, 3, 2, 4).double() for t in qkv.split(heads * d, -1)]
    kt = k.transpose(-1, -2).contiguous()
    s, size = q @ kt * scale, (q.abs() @ kt.abs()) * abs(scale)
    if mask is not None:
        s, size = s + mask[:, :, None, None, :], size + mask[:, :, None, None, :].abs() * (mask[:, :, None, None, :] > -1000)
    p = s.softmax(-1)
    rel = 2 * (d + 4) * 2.0 ** -24 * size.amax(-1, keepdim=True) + (S + 16) * 2.0 ** -23
    back = lambda t: t.permute(0, 1, 3, 2, 4).reshape(M, B * S, heads * d)
    return back(p @ v.contiguous()), back(rel * (p @ v.abs().contiguous()))


@pytest.mark.parametrize("masked", [False, True], ids=["", "mask"])
@pytest.mark.parametrize("S", [9, 16, 17, 32, 33, 64, 65, 130])
@pytest.mark.parametrize("d", [4, 20, 32, 36, 64, 68, 128])
def test_edges(nf, d, S, masked):
    M, B, heads, scale = 2, 2, 3, d ** -0.5
    qkv, mask = problem(M, B, S, heads, d, masked)
    got = nf.attention_packed(qkv.cuda(), B, S, heads, mask=None if mask is None else mask.cuda()).cpu().double()
    ref, bound = reference(qkv, mask, M, B, S, heads, d, scale)
    assert ((got - ref).abs() <= bound).all()


@pytest.mark.parametrize("S", [12, 20, 70])
@pytest.mark.parametrize("scale", [-0.3, 0.0])
def test_scales_that_turn_the_order(nf, S, scale):
    qkv, _ = problem(1, 1, S, 2, 64, False)
    got = nf.attention_packed(qkv.cuda(), 1, S, 2, scale=scale).cpu().double()
    ref, bound = reference(qkv, None, 1, 1, S, 2, 64, scale)
    assert ((got - ref).abs() <= bound).all()


@pytest.mark.parametrize("S", [12, 20, 70])
def test_a_model_has_the_same_bits_alone(nf, S):
    qkv, mask = problem(3, 2, S, 2, 64, True)
    qkv, mask = qkv.cuda(), mask.cuda()
    all_of = nf.attention_packed(qkv, 2, S, 2, mask=mask)
    for m in range(3):
        assert torch.equal(all_of[m:m + 1], nf.attention_packed(qkv[m:m + 1].contiguous(), 2, S, 2, mask=mask[m:m + 1].contiguous()))
