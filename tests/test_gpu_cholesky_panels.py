"""The Cholesky factorisation where its panels are 512 columns wide (more than 6144
columns left) and change to 256: updates inside a panel over several column
tiles, the trailing update with 512 columns, a last block of an odd size and an
odd leading dimension.  Reference: K itself, in FP64 on the GPU."""
import pytest

from conftest import ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ensure_built()

from paper_2501_14911_amd import cholesky  # noqa: E402

DEV = "cuda"
EPS = 2.0 ** -52
N = 6144 + 512 + 77


def spd():
    g = torch.Generator(device=DEV).manual_seed(1)
    A = torch.randn((N, 400), generator=g, dtype=torch.float64, device=DEV)
    K = A @ A.T
    K = 0.5 * (K + K.T)                                   # (the product's halves differ by its own rounding)
    K.diagonal().add_(torch.logspace(-2, 2, N, dtype=torch.float64, device=DEV))
    return K


def test_factor_of_wide_panels():
    K = spd()
    A = torch.full((N, N + 3), float("nan"), dtype=torch.float64, device=DEV)        # lda = N + 3
    A[:, :N] = torch.triu(K)                                                         # tensor row j = column j of K
    A[:, :N] += torch.tril(torch.full((N, N), float("nan"), dtype=torch.float64, device=DEV), -1)   # never read
    f = cholesky(A[:, :N])
    assert torch.isnan(A[:, N:]).all()
    assert torch.equal(f, f.T)                                                       # L and L^T agree to the bit
    U = torch.triu(f)                                                                # L^T
    # backward error of Cholesky: (N + 1) eps |L| |L^T| / 2 entry by entry, doubled for the blocked solves
    bound = (N + 1) * EPS * (U.abs().T @ U.abs()) + EPS * K.abs()
    assert ((U.T @ U - K).abs() <= bound).all()


@pytest.mark.parametrize("bad", [0, 127, 128, 300, 511, 512, 640, N - 1])
def test_first_bad_pivot_of_wide_panels(bad):
    K = torch.eye(N, dtype=torch.float64, device=DEV) * 4.0
    K[bad, bad] = -1.0
    with pytest.raises(ValueError, match=rf"pivot {bad} "):
        cholesky(K)
