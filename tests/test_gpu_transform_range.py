"""Series near the top of the precision's range pass through every transform:
an impulse A with M A just below the largest finite number, M the complex
transform length, whose unscaled inverse transform holds M A at one place.  At
compiled lengths, at a runtime length with few and with many series, with the
truncation between two products."""
import pytest

from conftest import ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ensure_built()

from paper_2501_14911_amd import P2OOperator  # noqa: E402

DEV = "cuda"
TOL = {torch.float64: 1e-12, torch.float32: 1e-5}         # of all parity tests, relative to the impulse


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("Nt, Nm", [(16, 40), (128, 40), (420, 40), (420, 2100), (500, 40), (500, 2100), (60, 40),
                                    (60, 8200), (243, 8200)])
def test_impulse_near_the_largest_number(Nt, Nm, precision):
    print(f"[transform range] Nt={Nt} Nm={Nm} {precision}", flush=True)
    op = P2OOperator(2, Nm, Nt, precision, max_rhs=1, device=DEV)

    def blocks(c0, n):                                    # F_0 = 1 at (sensor 1, column 5), all else 0
        F = torch.zeros((Nt, 2, n), dtype=torch.float64, device=DEV)
        if c0 == 0:
            F[0, 1, 5] = 1.0
        return F

    op.load(blocks)
    A = 0.75 * torch.finfo(op.dtype).max / (op.L // 2)
    for t in (0, 7, Nt - 1):
        m = torch.zeros((1, Nt, Nm), dtype=op.dtype, device=DEV)
        d = torch.zeros((1, Nt, 2), dtype=op.dtype, device=DEV)
        m[0, t, 5] = A
        d[0, t, 1] = A
        for got, want in ((op.apply_F(m), d), (op.apply_Ft(d), m), (op.apply_FFt(d), d)):
            assert torch.isfinite(got).all()
            assert float((got / A - want / A).abs().max()) <= TOL[op.dtype]
