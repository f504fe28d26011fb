"""BF16 and FP16 forward products of few right-hand sides or sensors: short rows (their
columns rounded up to 8) run the LDS ring, as if its variant were set; longer
ones the kernels without LDS tiles, with 4 wavefronts per work item (rows shorter
than a scale block, or thousands of items) or 8, which agree with the ring.  Short rows of many sensors
run the ring of 16 columns, except with FP16 right-hand sides.  Spectra that the
last-level cache holds run the 16-column ring of 128 rows, larger ones the whole-line
rings; the FP16 adjoint takes the tile whose workgroups need fewer rounds."""
import pytest

from conftest import ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ensure_built()

from paper_2501_14911_amd import P2OOperator  # noqa: E402

DEV = "cuda"
SAME = 1e-5            # same rounded operands, FP32 sums in another order: 2^-24 sqrt(8192 products) = 5.4e-6


def setup(Nd, Nm, Nt, nrhs, precision):
    print(f"[narrow choice] {Nd} x {Nm} x {Nt}, {nrhs} {precision}", flush=True)
    op = P2OOperator(Nd, Nm, Nt, precision, max_rhs=nrhs, device=DEV)
    g = torch.Generator(device=DEV).manual_seed(Nd * 1000 + nrhs)
    op.load(lambda c0, n: torch.randn((Nt, Nd, n), generator=g, device=DEV))
    size_of = (10.0 ** (torch.arange(nrhs, device=DEV) % 7 - 3))[:, None, None]
    return op, torch.randn((nrhs, Nt, Nm), generator=g, device=DEV) * size_of


def forward(op, m, tile):
    op.set_gemm_tile(tile)
    op.workspace.fill_(0xFF)                              # NaN: nothing may be read before it is written
    return op.apply_F(m).clone()


@pytest.mark.parametrize("precision", ["fp16", "bf16"])
@pytest.mark.parametrize("Nd, Nm, nrhs, ring", [(200, 128, 9, 12), (65, 192, 3, 12), (33, 100, 16, 11),
                                                (16, 192, 17, 11), (7, 400, 33, 11)])
def test_short_rows_run_the_ring(Nd, Nm, nrhs, ring, precision):
    op, m = setup(Nd, Nm, 60, nrhs, precision)
    assert torch.equal(forward(op, m, -1), forward(op, m, ring))


@pytest.mark.parametrize("precision", ["fp16", "bf16"])
@pytest.mark.parametrize("Nd, Nm, Nt, nrhs", [(200, 200, 60, 9), (64, 4095, 243, 8), (64, 4096, 60, 5), (49, 20513, 420, 9),
                                              (16, 8200, 500, 33), (33, 12300, 243, 16)])
def test_work_items_of_4_and_8_wavefronts(Nd, Nm, Nt, nrhs, precision):
    op, m = setup(Nd, Nm, Nt, nrhs, precision)
    a, b = forward(op, m, -1).double().flatten(1), forward(op, m, 11 if Nd <= 64 else 18).double().flatten(1)
    assert not torch.equal(a, b)                          # two kernels
    err = ((a - b).norm(dim=1) / b.norm(dim=1)).max().item()
    assert err <= SAME, err


@pytest.mark.parametrize("Nd, Nm, Nt, nrhs, ring", [(600, 400, 260, 8, 8), (300, 440, 500, 32, 8), (600, 449, 243, 3, 14),
                                                    (600, 800, 125, 5, 14), (520, 1000, 135, 33, 13),
                                                    (600, 200, 135, 8, 12), (300, 7, 250, 33, 18), (450, 201, 50, 33, 12),
                                                    (300, 304, 45, 17, 18), (300, 400, 45, 17, 12)])
def test_short_rows_of_many_sensors(Nd, Nm, Nt, nrhs, ring):
    op, m = setup(Nd, Nm, Nt, nrhs, "fp16")
    assert torch.equal(forward(op, m, -1), forward(op, m, ring))


@pytest.mark.parametrize("precision, Nd, Nm, Nt, nrhs, ring", [
    ("bf16", 300, 304, 45, 17, 12), ("bf16", 450, 200, 60, 33, 18), ("bf16", 450, 500, 420, 17, 8), ("bf16", 200, 1000, 420, 17, 18),
    ("fp16", 100, 1000, 420, 17, 12), ("fp16", 129, 8, 250, 64, 18)])
def test_spectra_in_and_past_the_cache(precision, Nd, Nm, Nt, nrhs, ring):
    op, m = setup(Nd, Nm, Nt, nrhs, precision)
    assert torch.equal(forward(op, m, -1), forward(op, m, ring))


@pytest.mark.parametrize("Nd, Nm, Nt, nrhs, tile", [(300, 128, 420, 64, 9), (300, 128, 420, 65, 9), (200, 700, 420, 33, 9),
                                                    (200, 1000, 420, 33, 15), (300, 128, 128, 17, 15), (160, 128, 128, 17, 9),
                                                    (161, 128, 128, 17, 15), (160, 128, 420, 17, 9), (128, 128, 128, 17, 10)])
def test_adjoint_tile_by_rounds(Nd, Nm, Nt, nrhs, tile):
    op, _ = setup(Nd, Nm, Nt, nrhs, "fp16")
    d = torch.randn((nrhs, Nt, Nd), generator=torch.Generator(device=DEV).manual_seed(3), device=DEV)
    out = []
    for t in (-1, tile, 15):
        op.set_gemm_tile(t)
        op.workspace.fill_(0xFF)
        out.append(op.apply_Ft(d).double().flatten(1))
    assert torch.equal(out[0], out[1])
    assert ((out[0] - out[2]).norm(dim=1) / out[2].norm(dim=1)).max().item() <= SAME


def test_short_rows_with_fp16_operands():
    op, _ = setup(600, 200, 420, 8, "fp16")               # (FP16 right-hand sides: whole-line rings only)
    e = torch.randn((8, 420, 600), generator=torch.Generator(device=DEV).manual_seed(2), device=DEV)
    op.workspace.fill_(0xFF)
    a = op.apply_FFt(e).double().flatten(1)
    op.set_fp16_operands(False)
    b = op.apply_FFt(e).double().flatten(1)
    assert ((a - b).norm(dim=1) / b.norm(dim=1)).max().item() <= 2e-3      # the tolerance of all FP16 parity tests
