"""BF16 products with K shared by the waves of small tiles, at the edges of
tiles, slabs and waves, against FP64 on the same BF16 values; odd leading
dimensions of C."""
import numpy as np
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
    return m


@pytest.mark.parametrize("M,N,K", [
    (1, 1, 64), (16, 16, 4096), (15, 17, 65), (17, 33, 511), (16, 583, 4000), (23, 583, 20001),
    (33, 1501, 777), (64, 65, 513), (65, 3001, 2047), (100, 3011, 7620), (129, 2047, 1663),
    (128, 5984, 1687), (350, 1925, 9999), (485, 1000, 6001), (700, 2654, 2781)])
def test_bf16_products_match_fp64(spca, M, N, K):
    print(f"bf16 M={M} N={N} K={K}", flush=True)
    ld = (K + 7) // 8 * 8
    g = torch.Generator().manual_seed(M + N + K)
    P = torch.full((M, ld), float("nan"), dtype=torch.bfloat16)  # past K must not enter
    Q = torch.full((N, ld), float("nan"), dtype=torch.bfloat16)
    P[:, :K] = torch.randn(M, K, generator=g).bfloat16()
    Q[:, :K] = torch.randn(N, K, generator=g).bfloat16()
    C = spca.gemm_nt_bf16(P.cuda()[:, :K], Q.cuda()[:, :K]).cpu().numpy().astype(np.float64)
    P64 = P[:, :K].double().numpy()
    Q64 = Q[:, :K].double().numpy()
    # FP32 accumulation: one rounding a term at most
    bound = (np.abs(P64) @ np.abs(Q64).T) * (K * 2.0 ** -24) * 1.01 + 1e-30
    assert np.all(np.abs(C - P64 @ Q64.T) <= bound)


@pytest.mark.parametrize("M,N,K", [(255, 50001, 3001), (511, 25003, 3007), (250, 52000, 2111),
                                   (129, 50001, 3001), (256, 57344, 3072)])
def test_large_bf16_tiles_match_fp64(spca, M, N, K):
    print(f"bf16 M={M} N={N} K={K}", flush=True)
    ld = (K + 7) // 8 * 8
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    P = torch.full((M, ld), float("nan"), dtype=torch.bfloat16, device="cuda")
    Q = torch.full((N, ld), float("nan"), dtype=torch.bfloat16, device="cuda")
    P[:, :K] = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    Q[:, :K] = torch.randn(N, K, generator=g, device="cuda").bfloat16()
    C = spca.gemm_nt_bf16(P[:, :K], Q[:, :K]).double()
    P64, Q64 = P[:, :K].double(), Q[:, :K].double()
    bound = (P64.abs() @ Q64.abs().t()) * (K * 2.0 ** -24) * 1.01 + 1e-30
    assert bool(torch.all((C - P64 @ Q64.t()).abs() <= bound))
