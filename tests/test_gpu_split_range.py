"""Operands that products on BF16 parts leave to the FP32 tiles: their results
are the FP32 tiles', and no slower by more than the first look costs."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = range(64, 72)  # 256x160, 256x128, 64x80, 64x64, 64x32, 32x32, 64x16, 16x16


@pytest.fixture(scope="module")
def spca():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1212_4137_amd as m

    m.load()
    m.tune_table_clear()
    yield m
    m.tune_table_clear()


def _dense(rows, K, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    X = torch.full((rows, (K + 3) // 4 * 4), float("nan"), device="cuda")  # past K must not enter
    X[:, :K] = torch.randn(rows, K, generator=g, device="cuda")
    return X[:, :K]


def _ld(X):
    """X with a leading dimension that is a multiple of 4; past K NaN."""
    K = X.shape[1]
    return torch.nn.functional.pad(X, (0, -K % 4), value=float("nan"))[:, :K]


def _bits(C):
    return torch.where(torch.isnan(C), torch.full_like(C, 7.0), C).view(torch.int32)


def _time(f, n=10):
    f()
    best = float("inf")
    for _ in range(5):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(n):
            f()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) / n)
    return best


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("M,N,K", [(1, 1, 192), (300, 333, 225), (65, 1000, 1001)])
def test_special_values_give_the_fp32_bits(spca, shape, M, N, K):
    """Infinities, NaN, sums that overflow, all of C tiny."""
    print(f"special values shape={shape} M={M} N={N} K={K}", flush=True)
    P, Q = _dense(M, K, 1), _dense(N, K, 2)
    row, col = M // 2, N // 3
    P1, Q1 = P.clone(), Q.clone()
    P1[row, K - 1] = float("inf")
    Q1[col, 0] = float("nan")
    for A, B in ((P1, Q), (P, Q1), (P1, Q1)):
        got, ref = (spca.gemm_nt_shape(_ld(A), _ld(B), s)[0] for s in (shape, 0))
        bad = ~torch.isfinite(ref)
        assert torch.equal(bad, ~torch.isfinite(got))
        assert torch.equal(_bits(got)[bad], _bits(ref)[bad])
    for a, b in ((1e20, 1e20), (1e-15, 1e-15), (1e-40, 1.0), (1.0, 1e-38), (0.0, 1e30)):
        got, ref = (spca.gemm_nt_shape(_ld(P * a), _ld(Q * b), s)[0] for s in (shape, 0))
        assert torch.equal(_bits(got), _bits(ref)), (a, b)


@pytest.mark.parametrize("M,N,K", [(1024, 10000, 1000), (1024, 1000, 10000), (300, 5000, 1200)])
def test_special_values_are_not_slow(spca, M, N, K):
    """At most the time of the parts on top of the FP32 tiles' (an infinity, a
    NaN for every sum, tiny operands)."""
    P, Q = _dense(M, K, 3), _dense(N, K, 4)
    ref = P.clone()
    f32 = _time(lambda: spca.gemm_nt_shape(P, Q, 0))
    parts = _time(lambda: spca.gemm_nt(P, Q))
    ref[M // 2, K // 2] = float("inf")
    Q1 = Q.clone()
    Q1[:, K // 2] = float("nan")
    for A, B in ((ref, Q), (P, Q1), (P * 1e-15, Q * 1e-15)):
        assert _time(lambda: spca.gemm_nt(A, B)) <= 1.3 * (f32 + parts)
