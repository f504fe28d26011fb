"""The stored spectrum of chunks with many tiles, against the oracle's DFT of the
blocks: transform lengths on 256- and 512-thread workgroups and tiles of 16, 8
and 4 columns, two scale blocks of very different magnitude, a nearly empty last
tile, and a non-finite value in each corner."""
import numpy as np
import pytest

from conftest import ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ensure_built()

import oracle  # noqa: E402
import synth  # noqa: E402
from paper_2501_14911_amd import P2OError, P2OOperator  # noqa: E402

DEV = "cuda"
DT = {"fp64": torch.float64, "fp32": torch.float32, "bf16": torch.bfloat16, "fp16": torch.float16}
# unit roundoff, and the absolute part where FP16 is subnormal (2^-25 of its largest stored 2^15)
U = {"fp64": 0.0, "fp32": 2.0 ** -24, "bf16": 2.0 ** -8, "fp16": 2.0 ** -11}


def load(op, F):
    op.load(lambda c0, n: F[:, :, c0:c0 + n])


@pytest.mark.parametrize("precision", list(DT))
@pytest.mark.parametrize("Nt", [32, 60, 128, 243, 420, 500])
def test_stored_spectrum(Nt, precision):
    print(f"[wide load] Nt={Nt} {precision}", flush=True)
    Nd, Nm = 4, 4096 + 2049                               # the second chunk: 4 x 129 tiles of 16 columns
    w = synth.Workload("load", Nd=Nd, Nm=Nm, Nt=Nt, tau=max(2.0, Nt / 4))
    F = synth.operator_blocks(w, backend="torch", device=DEV)
    F[:, :, 4096:] *= 1e-3
    op = P2OOperator(Nd, Nm, Nt, precision, device=DEV)
    op.fhat.fill_(0xFF)                                   # NaN: everything has to be written
    load(op, F)
    s = op.spectrum_view().view(DT[precision]).double().reshape(op.nfreq, Nd, op.pitch, 2).cpu().numpy()
    assert not s[:, :, Nm:].any()                         # zero padding
    m = np.repeat(op.scales_view().double().cpu().numpy(), 4096, axis=1)[:, None, :Nm]
    assert (m == 2.0 ** np.round(np.log2(m))).all()
    got = (s[:, :, :Nm, 0] + 1j * s[:, :, :Nm, 1]) * m
    ref = oracle.spectrum(F.cpu().numpy(), op.L)
    # the FFT's FP64 rounding (relative to a bin row's size) and one rounding to the stored format
    fft = 1e-14 * np.sqrt((np.abs(ref) ** 2).mean())
    for part in (np.real, np.imag):
        a, b = part(got), part(ref)
        tiny = m * 2.0 ** -25 if precision == "fp16" else 0.0
        assert (np.abs(a - b) <= U[precision] * np.abs(b) + tiny + 8 * fft).all()


@pytest.mark.parametrize("at", [(0, 0, 0), (249, 3, 2099), (100, 0, 2099), (249, 3, 0)])
def test_non_finite_blocks_are_refused(at):
    F = torch.ones((250, 4, 2100), device=DEV)
    F[at] = float("inf")
    op = P2OOperator(4, 2100, 250, "fp16", device=DEV)
    with pytest.raises(P2OError):
        load(op, F)
    F[at] = 1.0
    load(op, F)                                           # and a finite load afterwards is accepted
