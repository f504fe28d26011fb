"""The triangular solves with K's factor and Q d at the edges of their tiles:
64-row blocks, 128-row panels, 16 right-hand sides per matrix-core tile and
16, 32 or 64 per pass; odd leading dimensions.  Reference: numpy in FP64."""
import numpy as np
import pytest

from conftest import ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ensure_built()

from paper_2501_14911_amd import cholesky_solve, d2q_apply  # noqa: E402

DEV = "cuda"
EPS = 2.0 ** -52


@pytest.mark.parametrize("nrhs", [1, 2, 16, 17, 33, 65])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 128, 129, 192, 255, 257, 389])
def test_solve_pair(n, nrhs):
    print(f"[solve] n={n} nrhs={nrhs}", flush=True)
    rng = np.random.default_rng(n * 100 + nrhs)
    A = rng.standard_normal((n, n + 5))
    K = A @ A.T + n * np.eye(n)
    L = np.linalg.cholesky(K)
    both = torch.full((n, n + 3), float("nan"), dtype=torch.float64, device=DEV)     # ldl = n + 3
    both[:, :n] = torch.from_numpy(L + L.T - np.diag(np.diag(L))).to(DEV)
    b = rng.standard_normal((nrhs, n)) * 10.0 ** (np.arange(nrhs) % 5 - 2)[:, None]
    X = torch.full((nrhs, n + 1), float("nan"), dtype=torch.float64, device=DEV)     # ldx = n + 1
    X[:, :n] = torch.from_numpy(b).to(DEV)
    x = cholesky_solve(both[:, :n], X[:, :n]).cpu().numpy()
    assert torch.isnan(X[:, n:]).all()
    # substitution's backward error: 2 n eps |L| |L^T| |x| over both solves, entry by entry (and numpy's in L)
    bound = 4 * n * EPS * (np.abs(L) @ np.abs(L.T) @ np.abs(x.T)).T + EPS * np.abs(b)
    assert (np.abs(x @ K - b) <= bound).all()


@pytest.mark.parametrize("nrhs", [1, 3])
@pytest.mark.parametrize("nq,N", [(1, 1), (3, 255), (5, 256), (7, 2047), (2, 2048), (300, 2309)])
def test_qoi_product(nq, N, nrhs):
    print(f"[Q d] {nq} x {N}, {nrhs}", flush=True)
    rng = np.random.default_rng(nq * N)
    Q = torch.full((nq, N + 1), float("nan"), dtype=torch.float64, device=DEV)       # ldq = N + 1
    q0, d = rng.standard_normal((nq, N)), rng.standard_normal((nrhs, N))
    Q[:, :N] = torch.from_numpy(q0).to(DEV)
    q = d2q_apply(Q[:, :N], torch.from_numpy(d).to(DEV)).cpu().numpy()
    assert (np.abs(q - d @ q0.T) <= N * EPS * (np.abs(d) @ np.abs(q0.T))).all()
