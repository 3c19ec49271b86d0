"""Small grids: the fused z and y passes (one workgroup per kx plane) against the
pass-by-pass kernels, which run while mhd_profile records.  Both evaluate the
same operations in the same order, so the states agree bit for bit."""
import pytest

from paper_1810_12707_amd import inputs as I
from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

VARIANTS = {"ab2": {}, "rk4_forced": {"scheme": "rk4", "force": 0.1},
            "pc_laplacian": {"scheme": "pc", "flags": 4}, "kinematic": {"flags": 8}}


@pytest.mark.parametrize("variant", list(VARIANTS))
@pytest.mark.parametrize("precision", ["fp32", "fp64", "mixed"])
@pytest.mark.parametrize("n", [8, 12, 16, 24, 32])
def test_fused_equals_pass_by_pass(n, precision, variant):
    from paper_1810_12707_amd.mhd import Solver

    log(f"[fused] n={n} {precision} {variant}")
    c = I.random_turbulence(n, b_rms=0.3, seeds=(71, 72, 73))
    U = torch.from_numpy(c.U).to("cuda:0")
    out = []
    for record in (False, True):
        S = Solver(n, precision, gamma=c.gamma, nu=2e-3, eta=3e-3, dt=c.dt, **VARIANTS[variant])
        S.set_state(U)
        S.profile(record)
        S.step(3)
        S.profile(False)
        out.append(S.get_state())
        S.close()
    assert torch.isfinite(out[0]).all()
    assert torch.equal(out[0], out[1])
