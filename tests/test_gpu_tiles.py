"""Every tile that a time model chooses among, forced: the one-wave FP32 tiles
give the bits of the workgroup tiles whatever the K split, a group's tiles
give the bits of a request alone, and the BF16 tiles loaded straight to LDS
match FP64."""
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


def _operand(g, rows, K, mult, dtype):
    ld = (K + mult - 1) // mult * mult
    X = torch.full((rows, ld), float("nan"), device="cuda", dtype=dtype)  # past K must not enter
    X[:, :K] = torch.randn(rows, K, generator=g, device="cuda").to(dtype)
    return X[:, :K]


# slabs of 32 K, up to eight in flight: K of a few to many times that, with and
# without a partial slab; rows and columns around the tiles' edges
@pytest.mark.parametrize("shape", range(32, 38))
@pytest.mark.parametrize("M,N,K,splits", [
    (1, 1, 32, 1), (65, 33, 800, 1), (64, 130, 785, 1), (33, 95, 1024, 3), (129, 66, 1601, 4),
    (16, 500, 4100, 16), (70, 40, 255, 2)])
def test_one_wave_tiles_same_bits(spca, shape, M, N, K, splits):
    print(f"one-wave tile {shape} M={M} N={N} K={K} splits={splits}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M * N + K)
    P, Q = (_operand(g, rows, K, 4, torch.float32) for rows in (M, N))
    got = spca.gemm_nt_shape(P, Q, shape, splits)
    for workgroup in (0, 5):
        ref = spca.gemm_nt_shape(P, Q, workgroup, splits)
        torch.cuda.synchronize()
        assert torch.equal(got, ref)


@pytest.mark.parametrize("shape", range(96, 102))
@pytest.mark.parametrize("M,N,K", [(1, 1, 64), (17, 33, 511), (129, 225, 1000), (257, 449, 641),
                                   (40, 70, 4097)])
def test_direct_bf16_tiles_match_fp64(spca, shape, M, N, K):
    print(f"bf16 tile {shape} M={M} N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    P, Q = (_operand(g, rows, K, 8, torch.bfloat16) for rows in (M, N))
    C = spca.gemm_nt_shape(P, Q, shape)[0].double()
    P64, Q64 = P.double(), Q.double()
    # FP32 accumulation: one rounding a term at most
    bound = (P64.abs() @ Q64.abs().t().contiguous()) * (K * 2.0 ** -24) * 1.01 + 1e-30
    assert bool(torch.all((C - P64 @ Q64.t().contiguous()).abs() <= bound))


def test_forced_tiles_refuse_what_they_cannot_take(spca):
    P = torch.zeros((4, 64), device="cuda")
    for shape, splits in ((12, 1), (38, 1), (64, 1), (72, 1), (64, 2)):
        with pytest.raises(spca.SpcaError):
            spca.gemm_nt_shape(P, P, shape, splits)  # 64: K below 192
    B = P.bfloat16()
    for shape, splits in ((12, 1), (96, 2), (102, 1)):
        with pytest.raises(spca.SpcaError):
            spca.gemm_nt_shape(B, B, shape, splits)
    with pytest.raises(spca.SpcaError):
        spca.gemm_nt_shape(B[:, :56], B[:, :56], 96, 1)  # K below 64


def test_group_of_many_tiles_same_bits_as_alone(spca):
    """Six requests take 32 x 32 tiles, one alone 16 x 16."""
    g = torch.Generator(device="cuda").manual_seed(3)
    reqs = []
    for q in range(6):
        A = torch.randn(6001 + q, 301 + 5 * q, generator=g, device="cuda").t()
        X0 = torch.randn(20, A.shape[1], generator=g, device="cuda")
        reqs.append(dict(A=A, X0=X0 / X0.norm(dim=1, keepdim=True), formulation=1 + q % 2,
                         s_or_gamma=15.0, tol=-1.0, maxit=12))
    both = spca.am_solve_group(reqs, return_X=True)
    for q, got in zip(reqs, both):
        alone = spca.am_solve_group([q], return_X=True)[0]
        assert torch.equal(got["X_final"], alone["X_final"])


def test_plan_is_what_runs(spca):
    """The reported tile of a solve's products of few starts is a one-wave tile
    where the solve takes one, and that of a single product runs as reported."""
    assert 32 <= spca.gemm_plan(64, 2000, 2500, 16)[0] < 38
    g = torch.Generator(device="cuda").manual_seed(4)
    for M, N, K in ((64, 2000, 160), (300, 1000, 1001)):
        P, Q = (_operand(g, rows, K, 4, torch.float32) for rows in (M, N))
        assert torch.equal(spca.gemm_nt(P, Q),
                           spca.gemm_nt_shape(P, Q, *spca.gemm_plan(M, N, K))[0])


def test_autotune_times_the_one_wave_tiles(spca):
    """Few starts: the one-wave tiles take a third to two thirds of the
    workgroup tiles' time on both products, and the table holds them."""
    g = torch.Generator(device="cuda").manual_seed(6)
    n, p, r = 1000, 8000, 12
    A = torch.randn(p, n, generator=g, device="cuda").t()
    X0 = torch.randn(r, p, generator=g, device="cuda")
    X0 /= X0.norm(dim=1, keepdim=True)
    spca.tune_table_clear()
    try:
        tuned = spca.am_solve(A, 1, 20.0, X0, tol=-1.0, maxit=3, flags=spca.FLAG_AUTOTUNE,
                              return_X=True)
        table = spca.tune_table_export()
        shapes = [int(line.split()[5]) for line in table.splitlines()]
        assert any(32 <= shape < 38 for shape in shapes), table
        assert spca.gemm_plan(r, n, p, 16)[0] in shapes
        again = spca.am_solve(A, 1, 20.0, X0, tol=-1.0, maxit=3, return_X=True)
        assert torch.equal(tuned["X_final"], again["X_final"])  # from the table
        spca.tune_table_clear()
        spca.tune_table_import(table)
        assert spca.tune_table_export() == table
    finally:
        spca.tune_table_clear()
