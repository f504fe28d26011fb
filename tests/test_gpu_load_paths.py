"""The stored spectrum does not depend on how a chunk's tiles are shared out: rows
loaded together (persistent workgroups with several items, several scale blocks
each) and a row at a time (tiles too few for them) give the same multipliers and
the same stored bits, at lengths with an odd and an even number of bins, a length
whose tiles are small, and past the row count where that length's tiles change."""
import pytest

from conftest import ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ensure_built()

from paper_2501_14911_amd import P2OOperator  # noqa: E402

DEV = "cuda"


def stored(F, precision):
    Nt, Nd, Nm = F.shape
    op = P2OOperator(Nd, Nm, Nt, precision, device=DEV)
    op.fhat.fill_(0xFF)                                   # NaN: everything has to be written
    op.load(lambda c0, n: F[:, :, c0:c0 + n], chunk_cols=Nm)
    return op.spectrum_view().clone(), op.scales_view().clone()


@pytest.mark.parametrize("precision", ["bf16", "fp16"])
@pytest.mark.parametrize("Nt, Nd, Nm", [(32, 5, 8192 + 100), (48, 3, 9000), (125, 9, 8192 + 7), (243, 4, 8200),
                                        (420, 6, 4097), (32, 140, 4096)])
def test_maxima_and_bits_by_rows(Nt, Nd, Nm, precision):
    print(f"[load paths] {Nd} x {Nm} x {Nt} {precision}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(Nt)
    F = torch.randn((Nt, Nd, Nm), generator=g, device=DEV)
    F *= 10.0 ** (torch.arange(Nd, device=DEV) % 5 - 2)[None, :, None]
    F[:, :, 4096:] *= 1e-4
    together, scales = stored(F, precision)
    rows = [0, Nd // 2, Nd - 1]
    each = {r: stored(F[:, r:r + 1].contiguous(), precision)[1] for r in range(Nd)} if Nd < 20 else None
    if each is not None:                                  # multiplier = power of two by the largest: exact over rows
        assert torch.equal(scales, torch.stack(list(each.values())).amax(0))
    dt = torch.bfloat16 if precision == "bf16" else torch.float16
    got = together.view(dt).float().view(together.shape[0], Nd, -1, 2)[:, rows, :Nm]
    mult = scales.repeat_interleave(4096, dim=1)[:, None, :Nm, None]
    spec = torch.fft.rfft(F[:, rows].double(), n=2 * (together.shape[0] - 1), dim=0)
    want = torch.view_as_real(spec) / mult
    # one rounding to the stored format, FP16 subnormals below 2^-14, and the transforms' FP64 rounding
    u = 2.0 ** -8 if precision == "bf16" else 2.0 ** -11
    bound = u * want.abs() + (2.0 ** -25 if precision == "fp16" else 0.0) + 1e-12 * want.abs().max()
    assert ((got.double() - want).abs() <= bound).all()
