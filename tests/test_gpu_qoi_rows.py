"""Q d with short rows, four to a workgroup: the edges of the wavefront's sweeps
(64 columns, 256 and 512 in its unrolled steps), a last workgroup with idle
wavefronts, one, two and more right-hand sides, and the first length that a whole
workgroup takes.  Reference: numpy in FP64."""
import numpy as np
import pytest

from conftest import ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ensure_built()

from paper_2501_14911_amd import d2q_apply  # noqa: E402

DEV = "cuda"
EPS = 2.0 ** -52


@pytest.mark.parametrize("nrhs", [1, 2, 3, 9])
@pytest.mark.parametrize("nq,N", [(1, 1), (5, 63), (4, 64), (1001, 65), (6, 255), (7, 256), (3, 511), (9, 513), (2, 1023),
                                  (3, 1024)])
def test_short_rows(nq, N, nrhs):
    print(f"[Q d rows] {nq} x {N}, {nrhs}", flush=True)
    rng = np.random.default_rng(nq * N)
    Q = torch.full((nq, N + 3), float("nan"), dtype=torch.float64, device=DEV)       # ldq = N + 3
    q0, d = rng.standard_normal((nq, N)), rng.standard_normal((nrhs, N))
    Q[:, :N] = torch.from_numpy(q0).to(DEV)
    q = d2q_apply(Q[:, :N], torch.from_numpy(d).to(DEV)).cpu().numpy()
    assert (np.abs(q - d @ q0.T) <= N * EPS * (np.abs(d) @ np.abs(q0.T))).all()
