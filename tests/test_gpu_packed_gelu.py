"""Packed weights, GELU, three 256 x 256 tiles per compute unit and more (kernels chosen by k): the shortest k of the ring tile and the shorter
ones of the streaming one, a k that the 128-row tiles do not take, an odd number of 64-k steps, a last round that is not full, one row
tile per model and many, outputs a multiple of 4 KB apart."""
import numpy as np
import pytest
import torch

import netfuse_inputs as NI
from test_gpu_parity import check, dev, host, nf, rnd  # noqa: F401  (nf is a fixture)
from test_gpu_linear_packed import BF

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,Nout,res", [
    (768, 256, 256, 256, False), (97, 512, 320, 1024, True), (20, 1024, 576, 2560, False), (32, 512, 768, 3072, True),
    (1, 16384, 1024, 3072, False), (400, 256, 128, 512, False), (256, 256, 512, 768, False), (12, 2048, 1536, 2048, True), (12, 2048, 768, 2048, False),
])
def test_gelu_tiles(nf, oracle, M, N, K, Nout, res):
    sample = sorted({0, M - 1})
    gen = torch.Generator(device="cuda").manual_seed(K + M)
    mk = lambda *s, std=1.0: torch.empty(*s, device="cuda", dtype=BF).normal_(0, std, generator=gen)
    X, W, b = mk(M, N, K), mk(M, K, Nout, std=K ** -0.5), torch.randn(M, Nout, device="cuda", generator=gen) * 0.5
    R = mk(M, N, Nout) if res else None
    got = nf.linear_packed(X, nf.linear_pack_weight(W), bias=b, residual=R, act=2)
    rows = np.r_[0:64, N // 2 - 32:N // 2 + 32, N - 64:N]      # rows the oracle evaluates, of every row tile's kind
    f = lambda t: t[sample].float().cpu().numpy()
    ref = oracle.linear(f(X)[:, rows], f(W), bias=f(b), residual=None if R is None else f(R)[:, rows], act=2, out_bf16=True)
    check(host(got[sample])[:, rows], ref, BF, "packed gelu")
    if M * N * Nout < 2 ** 28:                                # every model against the row-major kernels
        want = nf.linear(X, W, bias=b, residual=R, act=2).float()
        assert float((got.float() - want).norm() / want.norm()) < 4e-3     # both round to 8 bits: 2^-8 per element at most
