"""FP32 products on BF16 parts (gemm_split.hip): every tile against an FP64
product at the edges of tiles and slabs, and the values that the
parts cannot hold (infinities, NaN, overflow, tiny operands) against the FP32
tiles."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPE0, NSHAPES = 64, 8  # 256x160, 256x128, 64x80, 64x64, 64x32, 32x32, 64x16, 16x16


@pytest.fixture(scope="module")
def spca():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1212_4137_amd as m

    m.load()
    m.tune_table_clear()
    yield m
    m.tune_table_clear()


def _bucket(x):
    return int(round(2.0 * math.log2(x)))


def _product(spca, P, Q, shape):
    """P Q^T with the tile forced through the tuning table."""
    M, K = P.shape
    spca.tune_table_import(f"4 1 {_bucket(M)} {_bucket(Q.shape[0])} {_bucket(K)} {shape} 1\n")
    try:
        C = spca.gemm_nt(P, Q)
        torch.cuda.synchronize()
    finally:
        spca.tune_table_clear()
    return C


def _operand(rng, rows, K):
    ld = (K + 3) // 4 * 4
    h = rng.standard_normal((rows, K)).astype(np.float32)
    buf = torch.full((rows, ld), float("nan"))  # what lies past K must not enter
    buf[:, :K] = torch.from_numpy(h)
    return buf.cuda()[:, :K], h.astype(np.float64)


@pytest.mark.parametrize("shape", range(SHAPE0, SHAPE0 + NSHAPES))
@pytest.mark.parametrize("M,N,K", [(1, 1, 192), (15, 17, 193), (64, 80, 256), (65, 81, 255),
                                   (256, 160, 224), (257, 161, 991), (130, 333, 1001),
                                   (300, 512, 4099)])
def test_split_product_matches_fp64(spca, shape, M, N, K):
    print(f"split shape={shape} M={M} N={N} K={K}", flush=True)
    rng = np.random.default_rng(shape * 31 + M + 3 * N + 7 * K)
    P, P64 = _operand(rng, M, K)
    Q, Q64 = _operand(rng, N, K)
    C = _product(spca, P, Q, shape).cpu().numpy().astype(np.float64)
    # the products left out are below 2^-23 of each term, and the sum is
    # rounded at most six times per 32 terms
    bound = (np.abs(P64) @ np.abs(Q64).T) * (2.0 ** -23 + (6 * (K // 32 + 2) + 16) * 2.0 ** -24)
    assert np.all(np.abs(C - P64 @ Q64.T) <= bound)


@pytest.mark.parametrize("shape", [64, 65, 67, 71])
def test_split_product_special_values(spca, shape):
    """Infinities, NaN and overflow come out as on the FP32 tiles; operands
    under the range of the parts keep their FP32 accuracy."""
    print(f"split special values shape={shape}", flush=True)
    M, N, K = 130, 200, 201
    rng = np.random.default_rng(shape)
    P0, _ = _operand(rng, M, K)
    Q0, _ = _operand(rng, N, K)

    def rows(X):  # leading dimension a multiple of 4
        return torch.nn.functional.pad(X, (0, -X.shape[1] % 4))[:, :X.shape[1]]

    def case(P, Q, tol):
        P, Q = rows(P), rows(Q)
        a, c = _product(spca, P, Q, 0), _product(spca, P, Q, shape)
        assert torch.equal(torch.isnan(a), torch.isnan(c))
        inf = torch.isinf(a)
        assert torch.equal(inf, torch.isinf(c)) and torch.equal(a[inf], c[inf])
        f = torch.isfinite(a)
        size = (P.abs().nan_to_num(0, 0, 0).double() @ Q.abs().nan_to_num(0, 0, 0).double().t())
        assert torch.all((a.double() - c.double()).abs()[f] <= tol * size[f] + 1e-44)

    tol = 2.0 * K * 2.0 ** -24
    Q = Q0.clone()
    Q[7, 3] = float("inf")
    case(P0, Q, tol)                      # inf of its sign
    Q[9, 5] = float("nan")
    P = P0.clone()
    P[11, 8] = -float("inf")
    case(P, Q, tol)
    P = P0.clone()
    P[:, 100:] = 0
    Q = Q0.clone()
    Q[7, 150] = float("inf")
    case(P, Q, tol)                       # inf times 0
    Q = Q0.clone()
    Q[3, 4] = 3.4e38                      # rounds to infinity in BF16
    case(P0 * 1e-3, Q, tol)
    for sp, sq in ((1.0, 1e-36), (1.0, 1e-40), (1e-20, 1e-20), (1e30, 1e-36), (1e18, 1e18),
                   (1e20, 1e20), (0.0, 1.0)):
        case(P0 * sp, Q0 * sq, tol)
