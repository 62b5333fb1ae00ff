"""Every tile of the ragged matmul kernel at shapes that route to it, and those of the whole-tile kernels, which are left
with k below 256 or not a multiple of 64: rows and columns past the last whole tile, several rounds of workgroups, with packed weights k-groups with unequal numbers of steps and with none.  Integer-coded: every sum is exact in
float32 in any order, so bias, residual and ReLU included the result must match the oracle bit for bit; GELU within the
rounding of a bf16 result (2^-8) and the 6.3e-7 of its polynomial."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [
    (12, 33, 256, 40), (48, 76, 256, 40), (2, 128, 768, 768), (3, 100, 1024, 264),    # 32 x 32, 64 x 64 (three)
    (48, 72, 256, 136), (48, 344, 448, 32), (48, 149, 256, 328),                      # 64 x 128, 96 x 128, 96 x 256
    (48, 208, 256, 144), (48, 199, 320, 272), (48, 142, 256, 656),                    # 128 x 128, 128 x 256, 128 x 384
    (48, 415, 256, 392), (12, 279, 768, 768), (16, 384, 320, 128),                    # 256 x 256, 96 x 128, 64 x 64
]
PACKED = [(1, 128, 256, 96), (24, 128, 256, 96), (48, 256, 256, 128), (48, 128, 384, 384), (48, 384, 256, 192),
          (48, 256, 256, 672)]                                                    # the six packed tiles, 32 x 32 first

WHOLE = [(2, 128, 160, 128), (2, 128, 192, 384), (2, 128, 160, 288), (2, 128, 192, 96), (32, 512, 160, 1024),
         (100, 256, 160, 384),                     # 128 x 128 (32- and 64-k steps), 128 x 288, 128 x 96, 256 x 256, 128 x 384
         (32, 512, 160, 3072), (32, 512, 160, 2304)]    # three tiles per workgroup: 256 x 256 with GELU; 128 x 384 without


def run(oracle, shape, packed, act):
    import paper_2009_13062_amd as nf
    M, N, K, Nout = shape
    rng = np.random.default_rng(N * K + Nout)
    sample = sorted({0, M // 2, M - 1})
    X = rng.integers(-2, 3, (M, N, K)).astype(np.float32)
    W = rng.integers(-1, 2, (M, K, Nout)).astype(np.float32)
    b = rng.integers(-4, 5, (M, Nout)).astype(np.float32)
    R = rng.integers(-8, 9, (M, N, Nout)).astype(np.float32)
    if act == 2:
        W, b = W / 16, b / 16                                # GELU's interesting range
    ref = oracle.linear(X[sample], W[sample], bias=b[sample], residual=R[sample], act=act, out_bf16=True)
    d = lambda a, dt=torch.bfloat16: torch.from_numpy(a).to("cuda", dt)
    Wd = d(W)
    f, Wd = (nf.linear_packed, nf.linear_pack_weight(Wd)) if packed else (nf.linear, Wd)
    got = f(d(X), Wd, bias=d(b, torch.float32), residual=d(R), act=act)
    return got[sample].float().cpu().numpy(), ref


@pytest.mark.parametrize("act", [0, 1])
@pytest.mark.parametrize("shape,packed", [(s, False) for s in CASES] + [(s, True) for s in PACKED] + [(s, False) for s in WHOLE])
def test_exact(oracle, shape, packed, act):
    got, ref = run(oracle, shape, packed, act)
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("shape,packed", [(CASES[0], False), (CASES[4], False), (PACKED[0], True), (PACKED[5], True)] +
                         [(s, False) for s in WHOLE])
def test_gelu(oracle, shape, packed):
    got, ref = run(oracle, shape, packed, 2)
    assert np.all(np.abs(got - ref) <= 2.0 ** -7 * np.abs(ref) + 2e-6)


def test_merged_equals_single(oracle):
    """k is summed in one ascending chain whatever tile the number of models leads to: the same bits per model."""
    import paper_2009_13062_amd as nf
    g = torch.Generator(device="cuda").manual_seed(5)
    for N, K, Nout in ((93, 768, 768), (128, 3072, 768), (279, 768, 2304)):
        X = torch.empty(32, N, K, device="cuda").normal_(generator=g).bfloat16()
        W = torch.empty(32, K, Nout, device="cuda").normal_(0, 0.03, generator=g).bfloat16()
        one = nf.linear(X[31:], W[31:])
        for M in (2, 5, 12, 32):
            assert torch.equal(nf.linear(X[32 - M:], W[32 - M:])[M - 1], one[0]), (M, N, K, Nout)


# more than 128 rows: 64 x 256, 160 x 256, 192 x 192, 288 x 128 (five and seven steps of 64 as well as four), then the others
TALL = [(24, 129, 256, 656), (24, 129, 448, 656), (48, 300, 256, 392), (48, 300, 320, 392), (48, 300, 256, 264), (48, 300, 448, 264),
        (48, 199, 256, 328), (48, 577, 320, 120), (32, 129, 320, 136), (16, 129, 256, 656), (48, 129, 256, 328), (48, 199, 256, 136),
        (48, 415, 256, 264), (48, 344, 256, 392)]


@pytest.mark.parametrize("act", [0, 1])
@pytest.mark.parametrize("shape", TALL)
def test_tall_exact(oracle, shape, act):
    got, ref = run(oracle, shape, False, act)
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("shape", [(48, 300, 256, 392), (48, 300, 320, 264), (48, 199, 256, 328), (24, 129, 256, 656)])
def test_tall_one_model(shape):
    """Random values: a model's bits are those it has alone, in whatever tile."""
    import paper_2009_13062_amd as nf
    M, N, K, Nout = shape
    torch.manual_seed(N + K)
    X, W = torch.randn(M, N, K, device="cuda").bfloat16(), torch.randn(M, K, Nout, device="cuda").bfloat16()
    b = torch.randn(M, Nout, device="cuda")
    Y = nf.linear(X, W, bias=b, act=2)
    for m in (0, M - 1):
        assert torch.equal(Y[m:m + 1], nf.linear(X[m:m + 1].clone(), W[m:m + 1].clone(), bias=b[m:m + 1].clone(), act=2))
