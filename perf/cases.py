"""The work that users of this framework have it do, as measurable cases.

The framework runs the alternating-maximization (AM) iteration of sparse PCA
from many starting points.  A user's program calls whole solves (dense,
grouped, sparse) or, when it builds its own loop, the blocks of one iteration:
the two matrix products and the x-update operators.  Sizes come from the
repository's own workloads (100 x 500, 1000 x 10000, 5000 x 50000,
20000 x 200000 and the serving stream's n in [200, 5000], p in [1000, 50000],
r in {16, 64, 256}); the ragged ones are generic.

Solves run a fixed number of iterations (stop test off, as the throughput
workload does) and return every start's final iterate, the whole of what a
solve computes.  They use formulations whose iterates settle within that
many iterations (F1, F2; F4 and F8 from few starts), so that rounding in an early iteration
does not decide which stationary point a start ends at; the operators of the
others are cases of their own.
"""
from __future__ import annotations

import math

import torch

import paper_1212_4137_amd as spca

DEV = "cuda:0"


def listed():
    return [
        # smallest call: one start e_i* on a 100 x 500 matrix, where launches
        # and latency are everything (an interactive user, a test suite)
        dict(name="solve 100x500 F1 r1", op="solve", n=100, p=500, r=1, fid=1, s=10, maxit=40,
             graph=False),
        # small requests solved together, as the request server does
        dict(name="group 8 requests", op="group", count=8, n=300, p=1500, r=16, s=20, maxit=40),
        # the throughput workload's shape, one formulation, graph replay
        dict(name="solve 1000x10000 F1 r1024", op="solve", n=1000, p=10000, r=1024, fid=1, s=50,
             maxit=200, graph=True),
        # a serving request too large to be grouped: rows beyond the
        # one-workgroup x-update, signs for y
        dict(name="solve 2000x20000 F2 r64", op="solve", n=2000, p=20000, r=64, fid=2, s=60,
             maxit=40, graph=False),
        # a word-count matrix: documents x words, few starts, s = 5
        dict(name="sparse 20000x6000 F1 r20", op="sparse", n=20000, p=6000, tokens=1500000, r=20,
             fid=1, s=5, maxit=20),
        # V = A^T Y of the throughput workload (unit columns Y)
        dict(name="gemm 1024x10000x1000", op="gemm", dtype="f32", M=1024, N=10000, K=1000),
        # U = A X of the same, while the iterates are dense
        dict(name="gemm 1024x1000x10000", op="gemm", dtype="f32", M=1024, N=1000, K=10000),
        # a serving-size product with ragged sizes
        dict(name="gemm 61x3001x777", op="gemm", dtype="f32", M=61, N=3001, K=777),
        # V = A^T Y of the BF16 storage workload
        dict(name="gemm bf16 256x50000x5000", op="gemm", dtype="bf16", M=256, N=50000, K=5000),
        # the operators of the throughput workload: top-s selection and the
        # L1-ball threshold
        dict(name="x_update T_s 1024x10000", op="x_update", fid=1, r=1024, p=10000, s=50),
        dict(name="x_update lambda_s 1024x10000", op="x_update", fid=3, r=1024, p=10000, s=50),
        # long rows (the 16 GB instance's 200000 columns): chunked kernels
        dict(name="x_update T_s 64x200000", op="x_update", fid=1, r=64, p=200000, s=200),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["solve", "group", "sparse", "gemm", "gemm", "gemm", "x_update", "x_update"])
    if op == "gemm":
        # r starts; n and p of the workloads; either product of an iteration
        M, n, p = _log(rng, 16, 1024), _log(rng, 200, 5000), _log(rng, 1000, 50000)
        if M * n * p > 64e9:
            M = max(16, int(64e9 / (n * p)))
        N, K = (p, n) if rng.random() < 0.6 else (n, p)
        return dict(op=op, dtype=rng.choice(["f32", "f32", "bf16"]), M=M, N=N, K=K)
    if op == "x_update":
        r, p = _log(rng, 16, 1024), _log(rng, 500, 200000)
        if r * p > 2e7:
            r = max(16, int(2e7 / p))
        return dict(op=op, fid=rng.choice([1, 3, 5, 7]), r=r, p=p,
                    s=_log(rng, 5, min(200, p // 20)))
    if op == "solve":
        n, p, r = _log(rng, 100, 2000), _log(rng, 500, 20000), _log(rng, 1, 512)
        return dict(op=op, n=n, p=p, r=r, fid=rng.choice([1, 2, 4, 8] if r <= 64 else [1, 2]),
                    s=_log(rng, 5, min(100, p // 20)), maxit=rng.choice([40, 60, 100]), graph=rng.random() < 0.5)
    if op == "group":
        return dict(op=op, count=rng.randint(2, 16), n=_log(rng, 100, 600), p=_log(rng, 500, 4000),
                    r=_log(rng, 4, 32), s=rng.randint(8, 25), maxit=rng.choice([30, 40, 50]))
    n, p = _log(rng, 4000, 40000), _log(rng, 2000, 10000)
    return dict(op=op, n=n, p=p, tokens=_log(rng, 20 * n, 60 * n), r=rng.randint(8, 32),
                fid=rng.choice([1, 2]), s=rng.randint(4, 10), maxit=20)


def _gen(seed, k=0):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + k) % (1 << 62))
    return g


def _unit_rows(g, r, p):
    X = torch.randn(r, p, generator=g, device=DEV)
    return X / X.norm(dim=1, keepdim=True)


def _spiked(g, n, p, nnz):
    """Spiked model G + sum_k theta_k u_k v_k^T, as a column-major (n, p)
    view (lda = n); theta scales with the noise level sqrt(n)."""
    At = torch.randn(p, n, generator=g, device=DEV)
    perm = torch.randperm(p, generator=g, device=DEV)
    for k, t in enumerate((1.9, 1.26, 0.79)):
        sup = perm[k * nnz:(k + 1) * nnz]
        u = torch.randn(n, generator=g, device=DEV)
        v = torch.randn(nnz, generator=g, device=DEV)
        At[sup] += t * math.sqrt(n) * torch.outer(v / v.norm(), u / u.norm())
    return At.t()


def _param(fid, s, A):
    return float(s) if fid <= 4 else 0.1 * float(A.double().norm(dim=0).max())


def _xu_param(case):
    """s, or a gamma that keeps the planted entries and some of the noise."""
    return {1: float(case["s"]), 3: float(case["s"]), 5: 9.0, 7: 3.0}[case["fid"]]


def _bag(g, n, p, tokens):
    """Word counts: Zipf word frequencies (exponent 1.07), log-normal
    document lengths; both compressed layouts on the GPU."""
    w = 1.0 / (torch.arange(p, device=DEV, dtype=torch.float64) + 2.7) ** 1.07
    cdf = torch.cumsum(w / w.sum(), 0)
    lens = torch.exp(0.8 * torch.randn(n, generator=g, device=DEV, dtype=torch.float64))
    dcdf = torch.cumsum(lens / lens.sum(), 0)
    words = torch.searchsorted(cdf, torch.rand(tokens, generator=g, device=DEV,
                                               dtype=torch.float64)).clamp_(max=p - 1)
    docs = torch.searchsorted(dcdf, torch.rand(tokens, generator=g, device=DEV,
                                               dtype=torch.float64)).clamp_(max=n - 1)
    key, cnt = torch.unique(words * n + docs, return_counts=True)
    col, row = key // n, key % n
    rkey, order = torch.sort(row * p + col)

    def ptr(idx, m):
        out = torch.zeros(m + 1, dtype=torch.int64, device=DEV)
        out[1:] = torch.cumsum(torch.bincount(idx, minlength=m), 0)
        return out

    val = cnt.float()
    return {"n": n, "p": p, "col_ptr": ptr(col, p), "row_idx": row.int(), "col_val": val,
            "row_ptr": ptr(row, n), "col_idx": (rkey % p).int(), "row_val": val[order]}


def prepare(case, seed):
    g = _gen(seed)
    op = case["op"]
    st = dict(case)
    if op == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        ld = (K + 7) // 8 * 8  # rows start 16-byte aligned in either type
        dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        P = torch.zeros(M, ld, dtype=dt, device=DEV)
        Q = torch.zeros(N, ld, dtype=dt, device=DEV)
        P[:, :K] = _unit_rows(g, M, K)
        Q[:, :K] = torch.randn(N, K, generator=g, device=DEV)
        st.update(P=P[:, :K], Q=Q[:, :K])
    elif op == "x_update":
        r, p, s = case["r"], case["p"], case["s"]
        # rows of A^T y near a stationary point: noise, and s planted entries
        V = torch.randn(r, p, generator=g, device=DEV)
        idx = torch.rand(r, p, generator=g, device=DEV).topk(s, dim=1).indices
        V.scatter_add_(1, idx, 6.0 * torch.randn(r, s, generator=g, device=DEV))
        st.update(V=V, par=_xu_param(case), out=(
            torch.empty(r, p, device=DEV), torch.empty(r, dtype=torch.float64, device=DEV),
            torch.empty(r, dtype=torch.int32, device=DEV)))
    elif op == "solve":
        A = _spiked(g, case["n"], case["p"], min(50, case["p"] // 20))
        X0 = None if case["r"] == 1 else _unit_rows(g, case["r"], case["p"])
        st.update(A=A, X0=X0, par=_param(case["fid"], case["s"], A), ctx=_ctx())
    elif op == "group":
        reqs = []
        for q in range(case["count"]):
            # requests of different sizes and formulations
            n, p = case["n"] + 7 * q, case["p"] + 13 * q
            A = _spiked(g, n, p, min(50, p // 20))
            fid = (1, 2)[q % 2]
            reqs.append(dict(A=A, X0=_unit_rows(g, case["r"], p), formulation=fid,
                             s_or_gamma=_param(fid, case["s"], A), tol=-1.0, maxit=case["maxit"]))
        st.update(reqs=reqs, ctx=_ctx())
    else:
        D = _bag(g, case["n"], case["p"], case["tokens"])
        st.update(D=D, X0=_unit_rows(g, case["r"], case["p"]), ctx=_ctx())
    return st


_shared = []


def _ctx():
    """The context that a program keeps: one for all its solves."""
    if not _shared:
        _shared.append(spca.Context(0))
    return _shared[0]


def run(st):
    op = st["op"]
    if op == "gemm":
        return spca.gemm_nt(st["P"], st["Q"]) if st["dtype"] == "f32" else \
            spca.gemm_nt_bf16(st["P"], st["Q"])
    if op == "x_update":
        return spca.x_update(st["fid"], st["V"], st["par"], out=st["out"])
    if op == "solve":
        res = spca.am_solve(st["A"], st["fid"], st["par"], st["X0"], tol=-1.0, maxit=st["maxit"],
                            flags=spca.FLAG_GRAPH if st["graph"] else 0, ctx=st["ctx"],
                            return_X=True)
        return res["X_final"]
    if op == "group":
        return [q["X_final"] for q in spca.am_solve_group(st["reqs"], ctx=st["ctx"],
                                                          return_X=True)]
    res = spca.am_solve_sparse(st["D"], st["fid"], float(st["s"]), st["X0"], tol=-1.0,
                               maxit=st["maxit"], ctx=st["ctx"], return_X=True)
    return res["X_final"]


def work(case):
    op = case["op"]
    if op == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        e = 4 if case["dtype"] == "f32" else 2
        return {"bytes": e * (M + N) * K + 4 * M * N, "flops": 2.0 * M * N * K}
    if op == "x_update":
        return {"bytes": 8 * case["r"] * case["p"] + 12 * case["r"], "flops": 0}
    if op == "sparse":
        # each iteration multiplies with every stored entry once (A^T Y)
        nnz = 0.6 * case["tokens"]
        return {"bytes": 16 * nnz + 8 * case["r"] * case["p"],
                "flops": 2.0 * nnz * case["r"] * case["maxit"]}
    # A^T Y is dense in every iteration; A X once (then over the supports)
    count = case.get("count", 1)
    n, p, r = case["n"] + 3.5 * (count - 1), case["p"] + 6.5 * (count - 1), case["r"]
    return {"bytes": count * 4 * (n * p + 2 * r * p),
            "flops": count * 2.0 * n * p * r * (case["maxit"] + 1)}


# ---------------------------------------------------------------------------
# The same results in 64 bits
# ---------------------------------------------------------------------------

def _lambda_s(W, s):
    """lambda_s of each row of W = |V| (FP64): the root of
    ||(w - l)_+||_1 = sqrt(s) ||(w - l)_+||_2 in closed form on its segment."""
    c, _ = torch.sort(W, dim=1, descending=True)
    k = torch.arange(1, c.shape[1] + 1, device=W.device, dtype=torch.float64)
    S1, S2 = torch.cumsum(c, 1), torch.cumsum(c * c, 1)
    lo = torch.cat([c[:, 1:], torch.zeros_like(c[:, :1])], 1)
    l1 = S1 - k * lo
    l2 = (S2 - 2 * lo * S1 + k * lo * lo).clamp(min=0)
    ok = (l1 >= math.sqrt(s) * l2.sqrt()) & (l2 > 0) & (k > s)
    has = ok.any(1)
    i = ok.double().argmax(1, keepdim=True)
    kk = (i + 1).double()
    a, b = S1.gather(1, i), S2.gather(1, i)
    lam = (a - torch.sqrt(s * (kk * b - a * a).clamp(min=0) / (kk - s).clamp(min=1e-300))) / kk
    lam = torch.minimum(torch.maximum(lam, lo.gather(1, i)), c.gather(1, i)).squeeze(1)
    slack = S1[:, -1] <= math.sqrt(s) * S2[:, -1].sqrt()
    return torch.where(has & ~slack, lam, torch.zeros_like(lam))


def _operator(fid, V, par):
    """(X, phi, nnz) of the x-update on the rows of V, in FP64."""
    fid -= 1 - fid % 2  # 2, 4, 6, 8 share the operators of 1, 3, 5, 7
    W = V.abs()
    if fid == 1:
        i = W.topk(int(par), dim=1).indices
        w = torch.zeros_like(V).scatter_(1, i, V.gather(1, i))
    elif fid in (3, 7):
        lam = _lambda_s(W, par)[:, None] if fid == 3 else par
        w = torch.sign(V) * (W - lam).clamp(min=0)
    else:
        w = torch.where(V * V > par, V, torch.zeros_like(V))
    nrm = w.norm(dim=1)
    phi = nrm
    if fid == 3:
        phi = lam[:, 0] * math.sqrt(par) + nrm
    elif fid == 5:
        phi = torch.where(w != 0, w * w - par, torch.zeros_like(w)).sum(1)
    X = w / torch.where(nrm > 0, nrm, torch.ones_like(nrm))[:, None]
    return X, phi, (w != 0).sum(1).int()


def _am(fid, par, X, iters, ax, aty):
    """`iters` AM iterations from the rows of X; y = u / ||u||_2 (odd
    formulations) or sgn(u) (even ones)."""
    for _ in range(iters):
        U = ax(X)
        Y = U / U.norm(dim=1, keepdim=True) if fid % 2 == 1 else torch.sign(U)
        X = _operator(fid, aty(Y), par)[0]
    return X


def _am_dense(fid, par, A, X0, iters):
    At = A.double().t().contiguous()  # p x n
    if X0 is None:
        X0 = torch.zeros(1, At.shape[0], device=DEV)
        X0[0, At.norm(dim=1).argmax()] = 1.0
    Ac = At.t().contiguous()
    return _am(fid, par, X0.double(), iters, lambda X: X @ At, lambda Y: Y @ Ac)


def exact(case, seed):
    st = prepare(case, seed)
    op = case["op"]
    if op == "gemm":
        return st["P"].double() @ st["Q"].double().t().contiguous()
    if op == "x_update":
        return _operator(case["fid"], st["V"].double(), st["par"])
    if op == "solve":
        return _am_dense(case["fid"], st["par"], st["A"], st["X0"], case["maxit"])
    if op == "group":
        return [_am_dense(q["formulation"], q["s_or_gamma"], q["A"], q["X0"], q["maxit"])
                for q in st["reqs"]]
    D = st["D"]
    A = torch.zeros(case["n"], case["p"], dtype=torch.float64, device=DEV)
    cols = torch.repeat_interleave(torch.arange(case["p"], device=DEV),
                                   D["col_ptr"][1:] - D["col_ptr"][:-1])
    A[D["row_idx"].long(), cols] = D["col_val"].double()
    At = A.t().contiguous()
    return _am(case["fid"], float(case["s"]), st["X0"].double(), case["maxit"],
               lambda X: X @ At, lambda Y: Y @ A)
