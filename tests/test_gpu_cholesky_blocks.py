"""The Cholesky factorisation at the edges of its tiles (16 columns, 128-row
blocks, 256-column panels, 128-row update tiles), odd leading dimensions,
pivots that are not positive in every kind of place.  Reference: K itself."""
import numpy as np
import pytest

from conftest import ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ensure_built()

from paper_2501_14911_amd import cholesky  # noqa: E402

DEV = "cuda"
EPS = 2.0 ** -52


def spd(n, cond):
    rng = np.random.default_rng(n)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    K = (Q * np.geomspace(1.0, cond, n)) @ Q.T
    return 0.5 * (K + K.T)


@pytest.mark.parametrize("scale", [1.0, 1e-200, 1e200])
@pytest.mark.parametrize("n", [1, 15, 17, 127, 128, 129, 145, 256, 257, 385, 513, 700])
def test_factor(n, scale):
    print(f"[cholesky] n={n} scale={scale:g}", flush=True)
    K = spd(n, 1e8) * scale
    A = torch.full((n, n + 3), float("nan"), dtype=torch.float64, device=DEV)        # lda = n + 3
    A[:, :n] = torch.from_numpy(np.triu(K)).to(DEV)                                  # tensor row j = column j of K
    A[:, :n] += torch.tril(torch.full((n, n), float("nan"), dtype=torch.float64, device=DEV), -1)   # never read
    f = cholesky(A[:, :n]).cpu().numpy()
    assert torch.isnan(A[:, n:]).all()
    L = np.triu(f).T
    assert np.array_equal(f, f.T)                                                     # L and L^T agree to the bit
    # backward error of Cholesky: (n + 1) eps |L| |L^T| / 2 entry by entry, doubled for the blocked solves
    bound = (n + 1) * EPS * (np.abs(L) @ np.abs(L.T)) + EPS * np.abs(K)
    assert (np.abs(L @ L.T - K) <= bound).all()


@pytest.mark.parametrize("bad", [0, 7, 16, 127, 128, 200, 256, 299])
@pytest.mark.parametrize("value", [-1.0, 0.0, float("nan")])
def test_first_bad_pivot(bad, value):
    K = np.eye(300) * 4.0
    K[bad, bad] = value
    with pytest.raises(ValueError, match=rf"pivot {bad} "):
        cholesky(torch.from_numpy(K).to(DEV))
