"""State in from FP32 and from FP64 fields of the same values: the rows of the two types
take different ways into the row pass of an FP32 run up to 128^3, and the same bits
must come out.  State out in FP64 is the FP32 state, widened."""
import pytest

from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [64, 96, 128, 192])
@pytest.mark.parametrize("precision", ["fp32", "mixed"])
def test_same_bits_from_either_type(n, precision):
    from paper_1810_12707_amd.mhd import Solver

    log(f"[row types] n={n} {precision}")
    g = torch.Generator(device="cuda:0").manual_seed(n)
    U = torch.randn(8, n, n, n, dtype=torch.float32, device="cuda:0", generator=g)
    S = Solver(n, precision)
    out = []
    for V in (U, U.double()):
        S.set_state(V)
        a = S.get_state(torch.float32)
        assert torch.equal(S.get_state(torch.float64), a.double())
        out.append(a)
    assert torch.isfinite(out[0]).all()
    assert torch.equal(out[0], out[1])
    S.close()
