"""x-update rows of any leading dimension and alignment, and the selections
over them at the edges of their paths: candidate counts around the 1024
entries a selection goes on with alone, ties at the threshold, rows whose
root lies far below or above the first guess."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def spca():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1212_4137_amd as m

    m.load()
    return m


def _rows(p, rng):
    """Rows that start the searches at different places."""
    V = rng.standard_normal((6, p)).astype(np.float32)
    V[1, rng.choice(p, min(p, 40), replace=False)] *= 50.0   # a few large entries
    V[2] = rng.integers(-3, 4, size=p)                       # ties everywhere
    V[3] = np.exp(3.0 * V[3]).astype(np.float32)             # heavy tail
    V[4, p // 3:] = 0.0
    V[5, p // 4:p // 4 + p // 9] *= 20.0                     # large entries crowded together
    return V


def _check(spca, fid, V_h, par, offset, pad):
    """V_h inside a wider buffer: ld = p + offset + pad, rows off by offset."""
    r, p = V_h.shape
    buf = torch.full((r, p + offset + pad), float("nan"), device="cuda")
    V = buf[:, offset:offset + p]
    V.copy_(torch.from_numpy(V_h))
    X, phi, nnz = (t.cpu().numpy() for t in spca.x_update(fid, V, par))
    for j, v in enumerate(V_h.astype(np.float64)):
        w, ph = oracle.x_operator(fid, v, par)
        nrm = np.linalg.norm(w)
        x = w / nrm if nrm > 0 else w
        # FP64 sums of p terms in another order, and one FP32 rounding of x
        # (|x| <= 1: half an ulp is 2^-25)
        assert abs(phi[j] - ph) <= 1e-11 * abs(ph)
        assert np.max(np.abs(X[j] - x)) <= 2.0 ** -24
        if fid != 3:  # lambda_s: an entry equal to the root may go either way
            assert nnz[j] == np.count_nonzero(w)
            np.testing.assert_array_equal(X[j] != 0, x != 0)


@pytest.mark.parametrize("offset,pad", [(0, 0), (1, 2), (3, 0)])
@pytest.mark.parametrize("p", [7, 1023, 2049, 4099, 12287, 12289, 20001, 70003])
def test_rows_of_any_alignment(spca, p, offset, pad):
    V_h = _rows(p, np.random.default_rng(p))
    for fid, par in ((1, max(1, p // 40)), (3, max(1.0, p / 90)), (5, 4.0), (7, 1.5)):
        _check(spca, fid, V_h, par, offset, pad)


@pytest.mark.parametrize("p", [1025, 4099, 12288, 13001, 40000])
@pytest.mark.parametrize("s", [1, 2, 700, 1023, 1024, 1025, 2500])
def test_selection_counts(spca, p, s):
    V_h = _rows(p, np.random.default_rng(p + s))
    s = min(s, p)
    _check(spca, 1, V_h, s, 1, 0)
    _check(spca, 3, V_h, float(s), 1, 0)


@pytest.mark.parametrize("p", [5001, 20001])
@pytest.mark.parametrize("fid,par", [(1, 40), (1, 3000), (3, 30.0), (5, 4.0), (7, 1.5)])
def test_in_place(spca, fid, par, p):
    """X = V: long rows then take the paths that do not keep state in X."""
    V_h = _rows(p, np.random.default_rng(p + fid))
    V = torch.from_numpy(V_h).cuda()
    X, phi, nnz = spca.x_update(fid, V, par)
    W = V.clone()
    out = (W, torch.empty_like(phi), torch.empty_like(nnz))
    spca.x_update(fid, W, par, out=out)
    torch.cuda.synchronize()
    assert torch.equal(out[2], nnz) and torch.allclose(out[1], phi, rtol=1e-13, atol=0)
    # the same decisions and values; norms summed in another order
    assert torch.equal(W != 0, X != 0)
    assert float((W - X).abs().max()) <= 2.0 ** -24
