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


def scores_as_given(nf, scores, v, mask=None):
    """One sequence and head of 64 features: query 0 against keys whose scores are exactly `scores` (feature 0 of the keys, 1 in the query)."""
    S = len(scores)
    qkv = torch.zeros(1, S, 3 * 64)
    qkv[0, :, 0] = 1
    qkv[0, :, 64] = scores
    qkv[0, :, 128:] = v
    return nf.attention_packed(qkv.cuda(), 1, S, 1, scale=1.0, mask=None if mask is None else mask.cuda()).cpu().double()[0]


@pytest.mark.parametrize("masked", [False, True], ids=["", "mask"])
@pytest.mark.parametrize("S", [12, 20, 70])
@pytest.mark.parametrize("top", [2.0 ** 31, -2.0 ** 33, 1.2345 * 2.0 ** 40, 1e20, -1e30, 2.9e38])
def test_scores_of_any_size(nf, S, masked, top):
    """Scores of neighbouring float32 numbers about `top` are 2^8 and more apart: all weight is on the largest, which a softmax gives weight 1 however
    large it is."""
    steps = torch.randperm(S, generator=torch.Generator().manual_seed(S)).float()
    scores = torch.tensor(top) * (1 - steps * 2.0 ** -20)
    best = int(scores.argmax())
    v = torch.randn(S, 64, generator=torch.Generator().manual_seed(1))
    got = scores_as_given(nf, scores, v, torch.zeros(1, 1, S) if masked else None)
    assert torch.equal(got, v[best].double().expand(S, 64))


@pytest.mark.parametrize("masked", [False, True], ids=["", "mask"])
@pytest.mark.parametrize("S", [12, 20, 70])
def test_exponents_of_exact_scores(nf, S, masked):
    """Scores that float32 holds exactly, about 1000: no rounding but the exponential's own (2 units), the sums' and the division's is left."""
    g = torch.Generator().manual_seed(S)
    scores = 1000 + torch.randint(-4096, 4096, (S,), generator=g).float() * 2.0 ** -10
    mask = torch.randint(-3, 3, (1, 1, S), generator=g).float() if masked else None
    v = torch.randn(S, 64, generator=g)
    got = scores_as_given(nf, scores, v, mask)
    p = (scores.double() + (mask[0, 0].double() if masked else 0)).softmax(0)
    assert ((got[0] - p @ v.double()).abs() <= (S + 16) * 2.0 ** -24 * (p @ v.double().abs())).all()


@pytest.mark.parametrize("S", [12, 20, 70])
def test_a_weight_below_the_normal_numbers(nf, S):
    """exp(-95) = 2^-137.05 times a value of 2^127, beside values of 0: held as a subnormal number, to 2^-13."""
    scores, v = torch.full((S,), -200.0), torch.zeros(S, 64)
    scores[0], scores[5], v[5] = 0.0, -95.0, 2.0 ** 127
    got = scores_as_given(nf, scores, v)
    ref = 2.0 ** 127 * torch.tensor(-95.0).double().exp()
    assert ((got - ref).abs() <= 2.0 ** -12 * ref).all()
