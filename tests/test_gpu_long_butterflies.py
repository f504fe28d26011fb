"""GPU parity of the compiled transforms of 420 and 500 complex points in FP32,
whose passes are butterflies of 10, 20, 21 and 25, against the FP64 oracle: on
the narrow and on the wide tiles, with a last tile that is nearly empty, active
lengths down to 0 and the re-pad on FP32 and on FP16 pairs."""
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
TOL = {"fp32": 1e-5, "fp16": 2e-3}                         # the tolerances of all parity tests


@pytest.mark.parametrize("precision", ["fp32", "fp16"])
@pytest.mark.parametrize("Nd, Nm", [(2, 33), (3, 16385)])  # narrow; wide tiles
@pytest.mark.parametrize("Nt", [420, 499, 500])
def test_long_butterflies(Nt, Nd, Nm, precision):
    print(f"[long butterflies] Nt={Nt} Nd={Nd} Nm={Nm} {precision}", flush=True)
    nrhs = 3
    w = synth.Workload("long", Nd=Nd, Nm=Nm, Nt=Nt, tau=Nt / 4)
    F = synth.operator_blocks(w, device=DEV, backend="torch")
    op = P2OOperator(Nd, Nm, Nt, precision, max_rhs=nrhs, device=DEV)
    op.load(lambda c0, n: F[:, :, c0:c0 + n])
    F = F.cpu().numpy()
    m, d = (torch.from_numpy(x).to(DEV, op.dtype) for x in (synth.param_series(w, nrhs), synth.data_series(w, nrhs)))
    mh, dh = m.double().cpu().numpy(), d.double().cpu().numpy()
    for nt in (None, [Nt - 1, 0, Nt // 2 + 1]):
        op.workspace.fill_(0xFF)                          # NaN: nothing may be read before it is written
        calls = [(op.apply_F(m, nt), oracle.apply_F, mh), (op.apply_Ft(d, nt), oracle.apply_Ft, dh),
                 (op.apply_FFt(d, nt), oracle.data_space_hessian, dh)]
        torch.cuda.synchronize()
        for got, ref, x in calls:
            got, ref = got.double().cpu().numpy(), ref(F, x, nt)
            # over all right-hand sides together: an empty one has no norm of its own
            err = oracle.rel_l2(got.reshape(1, -1), ref.reshape(1, -1))
            assert err <= TOL[precision], (Nt, precision, nt, err)
            for b in range(nrhs):
                if nt is not None:
                    assert not got[b, nt[b]:].any()
