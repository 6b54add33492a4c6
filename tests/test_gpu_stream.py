"""The one-wave FP32 tiles form every sum in the order of the workgroup tiles:
the same bits, at the edges of tiles, slabs of 32 K and slabs in flight."""
import math

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def spca():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1212_4137_amd as m

    m.load()
    m.tune_table_clear()
    yield m
    m.tune_table_clear()


# K below 192: such products stay on FP32 tiles
@pytest.mark.parametrize("M,N,K", [(1, 1, 5), (1, 500, 100), (15, 17, 31), (16, 300, 32),
                                   (17, 33, 65), (33, 1501, 191), (64, 2000, 160), (65, 90, 127)])
def test_same_bits_as_workgroup_tiles(spca, M, N, K):
    g = torch.Generator(device="cuda").manual_seed(M * N + K)
    ld = (K + 3) // 4 * 4
    P = torch.full((M, ld), float("nan"), device="cuda")  # past K must not enter
    Q = torch.full((N, ld), float("nan"), device="cuda")
    P[:, :K] = torch.randn(M, K, generator=g, device="cuda")
    Q[:, :K] = torch.randn(N, K, generator=g, device="cuda")
    got = spca.gemm_nt(P[:, :K], Q[:, :K])
    b = [int(round(2.0 * math.log2(x))) for x in (M, N, K)]
    spca.tune_table_import(f"4 1 {b[0]} {b[1]} {b[2]} 0 1\n")
    try:
        ref = spca.gemm_nt(P[:, :K], Q[:, :K])
        torch.cuda.synchronize()
    finally:
        spca.tune_table_clear()
    assert torch.equal(got, ref)
