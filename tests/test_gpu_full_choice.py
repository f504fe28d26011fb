"""FP64 and FP32 products of several right-hand sides: where sensors and
right-hand sides are few and rows are long, a call runs one streaming pass per
right-hand side, as if that mode were set; elsewhere the passes over 16 and 32
right-hand sides and over the wider column and row tiles (which take thousands of
work items) agree with it."""
import pytest

from conftest import ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ensure_built()

from paper_2501_14911_amd import P2OOperator  # noqa: E402

DEV = "cuda"
TOL = {"fp64": 1e-12, "fp32": 1e-5}                       # of all parity tests


def calls(op, m, d, mode):
    op.set_batched(mode)
    op.workspace.fill_(0xFF)                              # NaN: nothing may be read before it is written
    return op.apply_F(m).clone(), op.apply_Ft(d).clone(), op.apply_FFt(d).clone()


def setup(Nd, Nm, Nt, nrhs, precision):
    print(f"[full choice] {Nd} x {Nm} x {Nt}, {nrhs} {precision}", flush=True)
    op = P2OOperator(Nd, Nm, Nt, precision, max_rhs=nrhs, device=DEV)
    g = torch.Generator(device=DEV).manual_seed(Nd * 1000 + nrhs)
    op.load(lambda c0, n: torch.randn((Nt, Nd, n), generator=g, device=DEV))
    size_of = (10.0 ** (torch.arange(nrhs, device=DEV) % 7 - 3))[:, None, None]
    return (op, *((torch.randn((nrhs, Nt, n), generator=g, device=DEV) * size_of).to(op.dtype) for n in (Nm, Nd)))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("Nd, nrhs", [(1, 2), (1, 9), (2, 6), (4, 3), (6, 2)])
def test_few_sensors_stream(Nd, nrhs, precision):
    op, m, d = setup(Nd, 3000, 100, nrhs, precision)
    auto, gemv = calls(op, m, d, "auto"), calls(op, m, d, "gemv")
    assert torch.equal(auto[1], gemv[1])                  # F*
    if precision == "fp64" and nrhs * (Nd + 1) < 15:
        assert torch.equal(auto[0], gemv[0]) and torch.equal(auto[2], gemv[2])


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("Nd, Nm, Nt, nrhs", [(7, 3000, 100, 2), (16, 4097, 128, 16), (24, 4097, 128, 9),
                                              (32, 2049, 60, 33), (33, 1000, 128, 17), (65, 4097, 128, 33),
                                              (65, 4090, 128, 24), (4, 9001, 128, 17), (1, 33, 406, 33),
                                              (3, 128, 60, 2), (1, 200, 250, 9)])
def test_passes_agree_with_streaming(Nd, Nm, Nt, nrhs, precision):
    op, m, d = setup(Nd, Nm, Nt, nrhs, precision)
    for a, b in zip(calls(op, m, d, "auto"), calls(op, m, d, "gemv")):
        err = ((a - b).double().flatten(1).norm(dim=1) / b.double().flatten(1).norm(dim=1)).max().item()
        assert err <= TOL[precision], err


@pytest.mark.parametrize("Nd, Nm, Nt, nrhs, streams", [(33, 600, 60, 2, True), (40, 600, 60, 2, True), (41, 600, 60, 2, False),
                                                       (40, 600, 60, 3, False), (2, 4096, 16, 17, True),
                                                       (5, 1000, 16, 9, True), (5, 4096, 60, 9, False)])
def test_padded_rows_and_tiles_stream(Nd, Nm, Nt, nrhs, streams):
    op, m, d = setup(Nd, Nm, Nt, nrhs, "fp64")
    auto, gemv = calls(op, m, d, "auto"), calls(op, m, d, "gemv")
    assert torch.equal(auto[0], gemv[0]) == streams       # F
    if Nd <= 5:
        assert torch.equal(auto[1], gemv[1]) == streams   # F*
    for a, b in zip(auto, gemv):
        err = ((a - b).flatten(1).norm(dim=1) / b.flatten(1).norm(dim=1)).max().item()
        assert err <= TOL["fp64"], err
