"""GPU parity of the transforms of many series (the parameter side) at lengths
without a compiled kernel, against the FP64 oracle: every radix as the first
and as the last pass, the smallest length with two passes, the tile widths of
32, 16, 8 and (FP64) 4 series with 256- and 512-thread workgroups, the longest
length, active lengths down to 0, a last tile that is nearly empty."""
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
TOL = {"fp64": 1e-12, "fp32": 1e-5, "fp16": 2e-3, "bf16": 2e-3}       # the tolerances of all parity tests

LENGTHS = [9, 14, 35, 60, 127, 189, 250, 256, 288, 375, 486, 512, 756]


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("Nt", LENGTHS)
def test_transforms_of_many_series(Nt, precision):
    print(f"[wide fft] Nt={Nt} {precision}", flush=True)
    Nd, Nm, nrhs = 2, 4097, 2                             # 2 x 129 tiles of 32 series
    w = synth.Workload("wide", Nd=Nd, Nm=Nm, Nt=Nt, tau=max(2.0, Nt / 4))
    F = synth.operator_blocks(w, device=DEV, backend="torch")
    op = P2OOperator(Nd, Nm, Nt, precision, max_rhs=nrhs, device=DEV)
    op.load(lambda c0, n: F[:, :, c0:c0 + n])
    F = F.cpu().numpy()
    m, d = (torch.from_numpy(x).to(DEV, op.dtype) for x in (synth.param_series(w, nrhs), synth.data_series(w, nrhs)))
    mh, dh = m.double().cpu().numpy(), d.double().cpu().numpy()
    for nt in (None, [Nt - 1, 0], [1, Nt // 2 + 1]):
        op.workspace.fill_(0xFF)                          # NaN: nothing may be read before it is written
        calls = [(op.apply_F(m, nt), oracle.apply_F, mh), (op.apply_Ft(d, nt), oracle.apply_Ft, dh)]
        if precision != "bf16":                           # (data-space columns need more than BF16)
            calls.append((op.apply_FFt(d, nt), oracle.data_space_hessian, dh))
        torch.cuda.synchronize()
        for got, ref, x in calls:
            got, ref = got.double().cpu().numpy(), ref(F, x, nt)
            # over both right-hand sides together: an empty one has no norm of its own
            err = oracle.rel_l2(got.reshape(1, -1), ref.reshape(1, -1))
            assert err <= TOL[precision], (Nt, precision, nt, err)
            for b in range(nrhs):
                if nt is not None:
                    assert not got[b, nt[b]:].any()
