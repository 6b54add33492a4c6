"""Rows that the x-update's searches could handle wrongly or slowly: lambda_s
constraints that are inactive or nearly so, and ties."""
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


@pytest.mark.parametrize("p,k", [(500, 500), (9999, 9999), (12287, 3000), (20001, 20001),
                                 (70003, 70003), (20001, 5000), (9999, 1)])
def test_lambda_s_of_s_equal_entries(spca, p, k):
    """s = k equal entries: ||(|v| - t)_+||_1 = sqrt(s) ||(|v| - t)_+||_2 at
    every t below them, so that a search compares equal sums, which round
    either way, and has to end all the same."""
    print(f"equal entries p={p} k={k}", flush=True)
    V = np.zeros((3, p), dtype=np.float32)
    at = np.linspace(0, p - 1, k).astype(int)
    for j, a in enumerate((1.0, 0.3, -7.7e5)):
        V[j, at] = a
    X, phi, _ = (t.cpu().numpy() for t in spca.x_update(3, torch.from_numpy(V).cuda(), float(k)))
    want = np.abs(V.astype(np.float64)[:, at[0]]) * np.sqrt(k)
    np.testing.assert_allclose(phi, want, rtol=1e-11)
    # any lambda below the entries is a root, and they end equal
    assert np.max(np.abs(X - np.sign(V) / np.sqrt(k))) <= 2.0 ** -24
