"""Packed weights with few models: where netfuse_linear_packed_supported offers them (one round of 32 x 32 tiles, or long k over few rows), where it
does not, and the tiles that share k between wavefronts against the oracle: one round exactly (256 tiles), K of fewer steps than
wavefronts, K no multiple of the wavefronts' steps."""
import numpy as np
import pytest

import netfuse_inputs as NI
from test_gpu_parity import check, dev, host, nf, rnd  # noqa: F401  (nf is a fixture)
from test_gpu_linear_packed import BF

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,Nout", [(1, 128, 768, 768), (2, 128, 3072, 768), (2, 128, 1024, 1024), (8, 128, 256, 256), (1, 256, 512, 768),
                                        (3, 128, 3072, 768), (6, 128, 3072, 768), (1, 384, 4096, 1024), (2, 128, 1792, 768)])
def test_offered_and_right(nf, oracle, M, N, K, Nout):
    assert nf.linear_packed_supported(M, N, K, Nout)
    X, W = NI.on_bf16_grid(rnd(M, N, K)), NI.on_bf16_grid(rnd(M, K, Nout, std=K ** -0.5))
    b, R = rnd(M, Nout, std=0.5), NI.on_bf16_grid(rnd(M, N, Nout))
    got = nf.linear_packed(dev(X, BF), nf.linear_pack_weight(dev(W, BF)), bias=dev(b), residual=dev(R, BF), act=2)
    sample = sorted({0, M - 1})
    check(host(got[sample]), oracle.linear(X[sample], W[sample], bias=b[sample], residual=R[sample], act=2, out_bf16=True), BF, "packed")


@pytest.mark.parametrize("M,N,K,Nout", [(3, 128, 768, 768), (8, 128, 3072, 768), (1, 128, 768, 2304), (12, 128, 256, 256), (1, 100, 3072, 768), (1, 128, 128, 768)])
def test_not_offered(nf, M, N, K, Nout):
    assert not nf.linear_packed_supported(M, N, K, Nout)
