"""The flux pass of runs whose viscous force is the Laplacian takes no strain fields.
With nu = 0 neither form adds anything, so both flux passes must give the same states
bit for bit."""
import pytest

from paper_1810_12707_amd import inputs as I
from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("scheme", ["ab2", "rk4"])
@pytest.mark.parametrize("n,precision", [(24, "fp64"), (48, "fp32"), (64, "fp64"), (96, "fp32"), (96, "fp64"),
                                         (128, "fp32"), (128, "mixed"), (192, "fp64"), (256, "fp32")])
def test_laplacian_form_equals_stress_form_without_viscosity(n, precision, scheme):
    from paper_1810_12707_amd.mhd import Solver

    log(f"[no strain] n={n} {precision} {scheme}")
    c = I.random_turbulence(n, b_rms=0.3, seeds=(61, 62, 63))
    U = torch.from_numpy(c.U).to("cuda:0")
    out = []
    for flags in (0, 4):
        S = Solver(n, precision, gamma=c.gamma, nu=0.0, eta=3e-3, dt=c.dt, scheme=scheme, flags=flags)
        S.set_state(U)
        S.step(3)
        out.append(S.get_state())
        S.close()
    assert torch.isfinite(out[0]).all()
    assert torch.equal(out[0], out[1])
