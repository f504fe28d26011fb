"""GPU parity of the FP64 and FP32 products that serve several right-hand
sides per pass, against the FP64 oracle: sizes at the edges of the row blocks
(16 and 32 sensors, 64 from 9 right-hand sides on), of the 128-byte column
steps (8 FP64, 16 FP32 columns), of the adjoint's column tiles and of the
right-hand-side groups (8, 16 and, in FP32, 32)."""
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
TOL = {"fp64": 1e-12, "fp32": 1e-5}       # the per-right-hand-side path's tolerances

# (Nd, Nm, Nt, nrhs)
SIZES = [(1, 1, 1, 2), (15, 9, 3, 3), (16, 17, 5, 8), (17, 63, 6, 9), (33, 130, 4, 16), (64, 257, 7, 17), (65, 515, 5, 33)]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_products_of_several_right_hand_sides(size, precision):
    Nd, Nm, Nt, nrhs = size
    print(f"[full products] {precision} {size}", flush=True)
    w = synth.Workload("full", Nd=Nd, Nm=Nm, Nt=Nt, tau=4.0)
    F = synth.operator_blocks(w)
    op = P2OOperator(Nd, Nm, Nt, precision, max_rhs=nrhs, device=DEV)
    Fd = torch.from_numpy(F).to(DEV)
    op.load(lambda c0, n: Fd[:, :, c0:c0 + n])
    # right-hand sides of very different sizes stay apart
    size_of = 10.0 ** (np.arange(nrhs) % 7 - 3)[:, None, None]
    m, d = synth.param_series(w, nrhs) * size_of, synth.data_series(w, nrhs) * size_of
    md, dd = (torch.from_numpy(x).to(DEV, op.dtype) for x in (m, d))
    m, d = md.double().cpu().numpy(), dd.double().cpu().numpy()
    op.workspace.fill_(0xFF)                              # NaN: nothing may be read before it is written
    y, x, h = op.apply_F(md), op.apply_Ft(dd), op.apply_FFt(dd)
    torch.cuda.synchronize()
    for b in range(nrhs):
        for got, ref in ((y, oracle.apply_F(F, m[b])), (x, oracle.apply_Ft(F, d[b])),
                         (h, oracle.apply_F(F, oracle.apply_Ft(F, d[b])))):
            err = oracle.rel_l2(got[b].double().cpu().numpy(), ref)
            assert err <= TOL[precision], (size, precision, b, err)
