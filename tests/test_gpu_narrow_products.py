"""GPU parity of the BF16 and FP16 products of few right-hand sides or sensors
(the built-in choice there) against the FP64 oracle and against a forced LDS-ring
variant: sizes at the edges of the row blocks (16, 32, 48, 64 sensors), the
16-row steps of the adjoint and their pairs, the 32-column steps and 4096-column
blocks, the right-hand-side tiles (8, 16, and 32 with at most 16 sensors)."""
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
TOL = 2e-3             # BF16 or FP16 spectrum, FP32 accumulation (as in all parity tests)
SAME = 1e-5            # same rounded operands, FP32 sums in another order: 2^-24 sqrt(8192 products) = 5.4e-6

# (Nd, Nm, Nt, nrhs)
SIZES = [(1, 1, 1, 2), (4, 31, 6, 33), (16, 33, 5, 8), (17, 100, 7, 9), (32, 4095, 2, 3), (33, 4097, 2, 16),
         (49, 130, 16, 5), (65, 257, 9, 16), (128, 64, 4, 8), (255, 300, 3, 7)]


@pytest.mark.parametrize("precision", ["fp16", "bf16"])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_products_of_few_right_hand_sides(size, precision):
    Nd, Nm, Nt, nrhs = size
    print(f"[narrow products] {precision} {size}", flush=True)
    w = synth.Workload("narrow", Nd=Nd, Nm=Nm, Nt=Nt, tau=4.0)
    F = synth.operator_blocks(w)
    op = P2OOperator(Nd, Nm, Nt, precision, max_rhs=nrhs, device=DEV)
    Fd = torch.from_numpy(F).to(DEV)
    op.load(lambda c0, n: Fd[:, :, c0:c0 + n])
    # right-hand sides of very different sizes stay apart
    size_of = 10.0 ** (np.arange(nrhs) % 7 - 3)[:, None, None]
    m, d = (torch.from_numpy(x * size_of).to(DEV, torch.float32)
            for x in (synth.param_series(w, nrhs), synth.data_series(w, nrhs)))
    got = []
    for tile in (-1, 17):                                 # built-in choice; a ring (its own direction's, else built-in ring)
        op.set_gemm_tile(tile)
        op.workspace.fill_(0xFF)                          # NaN: nothing may be read before it is written
        calls = [op.apply_F(m), op.apply_Ft(d)]
        if precision == "fp16":                           # (data-space columns need more than BF16)
            calls.append(op.apply_FFt(d))
        got.append([c.double().cpu().numpy() for c in calls])
    mh, dh = m.double().cpu().numpy(), d.double().cpu().numpy()
    ref = [oracle.apply_F(F, mh), oracle.apply_Ft(F, dh), oracle.data_space_hessian(F, dh)]
    few = Nd * Nm < 2000                                  # a handful of terms: all right-hand sides together
    for here, ring, r in zip(got[0], got[1], ref):
        for b in range(nrhs):
            assert oracle.rel_l2(here[b], ring[b]) <= SAME
        if Nd * Nm * Nt == 1 and precision == "bf16":
            continue                                      # one stored value: its own rounding is up to 2^-8
        if few:
            here, r = here / size_of, r / size_of
            assert oracle.rel_l2(here, r) <= TOL
        else:
            assert max(oracle.rel_l2(here[b], r[b]) for b in range(nrhs)) <= TOL
