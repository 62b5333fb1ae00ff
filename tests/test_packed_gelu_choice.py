"""Which of the two 256 x 256 kernels takes large packed matmuls with a GELU, asked of the library on the CPU."""
import pytest


# Left to the streaming kernel: shapes that took up to 1.3 times as long on the ring tile.
@pytest.mark.parametrize("N,K,Nout,ring", [
    (512, 768, 3072, True), (512, 512, 3072, True), (512, 448, 3072, False), (512, 256, 3072, False), (4096, 320, 2048, False), (4096, 768, 2048, False),
    (2048, 1024, 4096, False), (2048, 1536, 4096, True), (1024, 768, 2048, True), (4096, 768, 3072, True), (8192, 3072, 2048, True), (512, 544, 3072, False),
])
def test_gelu_tile(N, K, Nout, ring):
    import paper_2009_13062_amd as nf
    assert bool(nf.lib.netfuse_packed_gelu_ring(N, K, Nout)) == ring
