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


def _error(C, P, Q):
    ref = P.double() @ Q.double().t().contiguous()
    return float((C.double() - ref).norm() / ref.norm())


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("M,N,K", [(1, 1, 192), (300, 333, 225), (65, 1000, 1001)])
def test_tiny_rows_among_others(spca, shape, M, N, K):
    """A row whose parts all vanish, in a tile of ordinary rows, against an
    operand that is large enough for it."""
    print(f"tiny rows shape={shape} M={M} N={N} K={K}", flush=True)
    P, Q = _dense(M, K, 5), _dense(N, K, 6)
    for tiny in (1e-42, 1e-39, 1e-30):
        A = P.clone()
        A[M // 2] *= tiny
        for X, Y in ((A, Q * 1e30), (Q * 1e30, A)):
            got, ref = (spca.gemm_nt_shape(_ld(X), _ld(Y), s)[0] for s in (shape, 0))
            if X is not A:
                got, ref = got.t(), ref.t()
            assert float(ref[M // 2].abs().max()) > 0.0
            assert torch.equal(_bits(got[M // 2].contiguous()), _bits(ref[M // 2].contiguous()))


@pytest.mark.parametrize("shape", SHAPES)
def test_sparse_rows_give_the_fp32_bits(spca, shape):
    """Few nonzeros a row (in P, in Q, in both), where six roundings a slab
    would be more than the FP32 instructions' one a term."""
    M, N, K = 130, 200, 1501
    g = torch.Generator(device="cuda").manual_seed(7)
    P, Q = _dense(M, K, 8), _dense(N, K, 9)

    def sparse(X, nnz):
        at = torch.rand(X.shape, generator=g, device="cuda").topk(nnz, 1).indices
        return _ld(torch.zeros_like(X).scatter_(1, at, X.gather(1, at)))

    for nnz in (1, 5, 20, K // 3):
        for A, B in ((sparse(P, nnz), Q), (P, sparse(Q, nnz)), (sparse(P, nnz), sparse(Q, nnz))):
            got, ref = (spca.gemm_nt_shape(A, B, s)[0] for s in (shape, 0))
            assert torch.equal(got, ref), nnz


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("K", [192, 333, 1000, 4100])
def test_error_no_larger_than_on_fp32_tiles(spca, shape, K):
    """Rows that are just full enough, with as few common terms as two such
    rows can have; with a few zeros; with rows of zeros; and dense ones."""
    M, N = 130, 300
    P, Q = _dense(M, K, 10), _dense(N, K, 11)
    quad = (torch.arange(K, device="cuda") // 4) % 8
    few_p, few_q = _ld(P * (quad < 5)), _ld(Q * (quad > 2))
    g = torch.Generator(device="cuda").manual_seed(12)
    some = _ld(P * (torch.rand(M, K, generator=g, device="cuda") < 0.95))
    gone = _ld(P.clone())
    gone[::3] = 0.0
    for A, B in ((P, Q), (few_p, Q), (few_p, few_q), (some, Q), (some, few_q), (gone, Q)):
        got, ref = (spca.gemm_nt_shape(A, B, s)[0] for s in (shape, 0))
        assert _error(got, A, B) <= _error(ref, A, B)
    assert float(got[::3].abs().max()) == 0.0


@pytest.mark.parametrize("M,N,K", [(1024, 10000, 1000), (64, 2000, 20000)])
def test_sparse_rows_are_not_slow(spca, M, N, K):
    P, Q = _dense(M, K, 13), _dense(N, K, 14)
    f32 = _time(lambda: spca.gemm_nt_shape(P, Q, spca.gemm_plan(M, N, K, 2)[0]))
    P[:] = 0.0
    P[:, ::K // 5] = 1.0 / 3.0
    assert _time(lambda: spca.gemm_nt(P, Q)) <= 1.25 * f32
