"""GPU parity of the FP32 transforms on tiles of 32 series, which take 512 of them
over all right-hand sides (4 x 129 here): on workgroups of 256 threads (up to
128 points) and of 512 (up to 256 points, odd and even numbers of bins), for
complex FP32, quad BF16 and FP16-scaled outputs, with the truncation between two
products and active lengths down to 0, against the FP64 oracle."""
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
TOL = {"fp32": 1e-5, "fp16": 2e-3, "bf16": 2e-3}          # the tolerances of all parity tests


@pytest.mark.parametrize("precision", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("Nt", [60, 126, 135, 189, 250, 256])
def test_tiles_of_32_series(Nt, precision):
    print(f"[wide tiles] Nt={Nt} {precision}", flush=True)
    Nd, Nm, nrhs = 2, 4097, 4
    w = synth.Workload("tiles", Nd=Nd, Nm=Nm, Nt=Nt, tau=Nt / 4)
    F = synth.operator_blocks(w, device=DEV, backend="torch")
    op = P2OOperator(Nd, Nm, Nt, precision, max_rhs=nrhs, device=DEV)
    op.load(lambda c0, n: F[:, :, c0:c0 + n])
    F = F.cpu().numpy()
    m, d = (torch.from_numpy(x).to(DEV, op.dtype) for x in (synth.param_series(w, nrhs), synth.data_series(w, nrhs)))
    mh, dh = m.double().cpu().numpy(), d.double().cpu().numpy()
    for nt in (None, [Nt - 1, 0, Nt // 2 + 1, 1]):
        op.workspace.fill_(0xFF)                          # NaN: nothing may be read before it is written
        calls = [(op.apply_F(m, nt), oracle.apply_F, mh), (op.apply_Ft(d, nt), oracle.apply_Ft, dh)]
        if precision != "bf16":                           # (data-space columns need more than BF16)
            calls.append((op.apply_FFt(d, nt), oracle.data_space_hessian, dh))
        torch.cuda.synchronize()
        for got, ref, x in calls:
            got, ref = got.double().cpu().numpy(), ref(F, x, nt)
            for b in range(nrhs):
                if nt is not None:
                    assert not got[b, nt[b]:].any()
                if nt is None or nt[b] > 1:
                    err = oracle.rel_l2(got[b], ref[b])
                    assert err <= TOL[precision], (Nt, precision, nt, b, err)
            assert np.isfinite(got).all()
