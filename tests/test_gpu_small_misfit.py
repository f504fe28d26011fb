"""GPU parity of the misfit and its gradient around the number of sensors that
one transform tile holds (32 at these lengths), where the misfit comes from
the transform itself instead of a reduction over tiles, at a compiled and a
runtime length, with active lengths down to 0."""
import numpy as np
import pytest

from conftest import ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ensure_built()

import oracle  # noqa: E402
import synth  # noqa: E402
from paper_2501_14911_amd import P2OOperator  # noqa: E402

DEV = "cuda"
TOL = {"fp64": 1e-12, "fp32": 1e-5}       # of all parity tests; 16-bit spectra use the FP32 transforms


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("Nt", [16, 20])
@pytest.mark.parametrize("Nd", [1, 31, 32, 33])
def test_misfit_around_one_tile(Nd, Nt, precision):
    print(f"[small misfit] Nd={Nd} Nt={Nt} {precision}", flush=True)
    Nm, nrhs = 70, 3
    w = synth.Workload("small", Nd=Nd, Nm=Nm, Nt=Nt, tau=Nt / 4)
    F = synth.operator_blocks(w, device=DEV, backend="torch")
    op = P2OOperator(Nd, Nm, Nt, precision, max_rhs=nrhs, device=DEV)
    op.load(lambda c0, n: F[:, :, c0:c0 + n])
    F = F.cpu().numpy()
    m, d = (torch.from_numpy(x).to(DEV, op.dtype) for x in (synth.param_series(w, nrhs), synth.data_series(w, nrhs)))
    mh, dh = m.double().cpu().numpy(), d.double().cpu().numpy()
    var = np.array([0.25])
    for nt in (None, [Nt - 1, 0, 1]):
        op.workspace.fill_(0xFF)                          # NaN: nothing may be read before it is written
        phi, g = op.misfit_grad(m, d, torch.from_numpy(var).to(DEV), nt)
        phi, g = phi.double().cpu().numpy(), g.double().cpu().numpy()
        for b in range(nrhs):
            n = Nt if nt is None else nt[b]
            if n == 0:
                assert phi[b] == 0 and not g[b].any()
                continue
            mb, db = mh[b:b + 1].copy(), dh[b:b + 1].copy()
            mb[:, n:], db[:, n:] = 0, 0
            r = oracle.apply_F(F, mb, [n]) - db
            ref = 0.5 * float((r ** 2).sum()) / var[0]
            g_ref = oracle.apply_Ft(F, r / var[0], [n])
            assert abs(phi[b] - ref) <= TOL[precision] * ref, (b, nt)
            assert oracle.rel_l2(g[b:b + 1], g_ref) <= TOL[precision], (b, nt)
