"""What the autotuner reports is what later calls run, also where the kernels
without LDS tiles beat every listed variant: at 8 sensors and 2 right-hand
sides they are two to four times as fast, and the report is -1, the value that
selects them (but for the BF16 adjoint, where a listed variant is as fast and
either may be reported)."""
import pytest

from conftest import ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ensure_built()

from paper_2501_14911_amd import P2OOperator, gemm_tiles  # noqa: E402

DEV = "cuda"


@pytest.mark.parametrize("precision", ["fp16", "bf16"])
@pytest.mark.parametrize("Nd, nrhs, built_in", [(8, 2, True), (300, 40, False)])
def test_reported_choice_is_the_one_that_runs(Nd, nrhs, built_in, precision):
    print(f"[autotune choice] Nd={Nd} nrhs={nrhs} {precision}", flush=True)
    Nm, Nt = (16384, 250) if built_in else (2048, 60)
    op = P2OOperator(Nd, Nm, Nt, precision, max_rhs=nrhs, device=DEV)
    g = torch.Generator(device=DEV).manual_seed(1)
    op.load(lambda c0, n: torch.randn((Nt, Nd, n), generator=g, device=DEV))
    m = torch.randn((nrhs, Nt, Nm), generator=g, device=DEV)
    d = torch.randn((nrhs, Nt, Nd), generator=g, device=DEV)
    got = op.autotune(nrhs, reps=5)
    for direction, call in (("fwd", lambda: op.apply_F(m)), ("adj", lambda: op.apply_Ft(d))):
        tile, ms = got[direction]
        assert ms > 0
        assert -1 <= tile < len(gemm_tiles())
        if not built_in:
            assert tile >= 0
        elif (precision, direction) != ("bf16", "adj"):
            assert tile == -1
        op.set_gemm_tile(-1)
        tuned = call()
        op.set_gemm_tile(tile)                            # the reported number, forced: the same kernel
        assert torch.equal(call(), tuned)
    op.set_gemm_tile(-1)
