"""BF16 and FP16 forward products of few right-hand sides or sensors: short rows (their
columns rounded up to 8) run the LDS ring, as if its variant were set; longer
ones the kernels without LDS tiles, with 4 wavefronts per work item (rows shorter
than a scale block, or thousands of items) or 8, which agree with the ring."""
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
@pytest.mark.parametrize("Nd, Nm, nrhs, ring", [(200, 128, 9, 18), (65, 192, 3, 18), (33, 100, 16, 11),
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
