"""mhd_step_bytes of kinematic runs: the launches of one step, each array counted once.
Written out from the update each stage makes."""
import pytest

from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# Spectra moved by the updates of one steady step: of the three evolved fields B, and of
# the five frozen ones.  AB2: state and history in and out; a frozen history read.
# PC predictor: state and history in, stage state and history out, frozen fields too;
# corrector: state, R^n and the stage's B in, state out.  RK4: state in, stage sum and
# stage state out, frozen fields too; twice state, sum and the stage's B in, sum and stage
# state out; state, sum and the stage's B in, state out.
UPDATES = {"ab2": 3 * 4 + 5, "pc": 8 * 4 + 3 * 4, "rk4": 8 * 3 + 2 * 3 * 5 + 3 * 4}
EVALS = {"ab2": 1, "pc": 2, "rk4": 4}


@pytest.mark.parametrize("scheme", list(UPDATES))
@pytest.mark.parametrize("n,precision", [(32, "fp32"), (48, "fp64"), (64, "mixed")])
def test_kinematic(n, precision, scheme):
    from paper_1810_12707_amd.mhd import MHD_FLAG_KINEMATIC, Solver

    log(f"[step bytes] n={n} {precision} {scheme}")
    S = Solver(n, precision, scheme=scheme, flags=MHD_FLAG_KINEMATIC)
    K = (n - 1) // 3
    nh, nb, size = K + 1, 2 * K + 1, 16 if precision == "fp64" else 8
    sc, iz, iy = nb * nb * nh, n * nb * nh, n * n * nh
    # rho, m, B, E to the grid, e = u x B, and back
    evaluation = 8 * sc + (8 + 8 + 3 + 3) * iz + (8 + 8 + 3 + 3) * iy
    want = size * (EVALS[scheme] * evaluation + UPDATES[scheme] * sc)
    assert S.step_bytes == pytest.approx(want, rel=1e-12)
    S.close()
