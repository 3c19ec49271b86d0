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


@pytest.mark.parametrize("n,precision", [(16, "fp64"), (32, "fp32"), (48, "fp64"), (64, "mixed"), (96, "fp32")])
def test_kinematic_run_continued_from_a_full_one(n, precision):
    """Frozen fields of a kinematic run: the first step after a checkpoint of a
    full run still applies its history, U <- U - dt/2 R^{n-1}; from then on they
    stay bit for bit.  The induction equation is the full run's."""
    from paper_1810_12707_amd.mhd import Solver

    log(f"[kinematic] n={n} {precision}")
    c = I.compressive_state(n, 5)
    kw = dict(gamma=5.0 / 3.0, nu=2e-3, eta=3e-3, dt=1e-2)
    U0 = torch.from_numpy(c).to("cuda:0")
    F = Solver(n, precision, **kw)
    F.set_state(U0)
    F.step(1)
    U1 = F.get_state()
    R0 = F.rhs(F_state(F, U0))
    K = Solver(n, precision, flags=8, **kw)
    assert K.load(F.save()) == 0
    K.step(1)
    F.step(1)
    U2, want_b = K.get_state(), F.get_state()[4:7]
    tol = {"fp64": 1e-12, "fp32": 1e-5, "mixed": 1e-3}[precision]
    for f in (0, 1, 2, 3, 7):
        want = U1[f] - 0.5 * kw["dt"] * R0[f]
        assert float((U2[f] - want).norm() / (kw["dt"] * R0[f]).norm()) < tol * float(
            U1[f].norm() / (kw["dt"] * R0[f]).norm())
    assert float((U2[4:7] - want_b).norm() / want_b.norm()) < tol
    K.step(3)
    U5 = K.get_state()
    for f in (0, 1, 2, 3, 7):
        assert torch.equal(U5[f], U2[f])
    assert not torch.equal(U5[4:7], U2[4:7])
    F.close()
    K.close()


def F_state(S, U):
    """Real fields U as the solver holds them (D F[U] back on the grid)."""
    T = type(S)(S.n, S.precision)
    T.set_state(U)
    out = T.get_state()
    T.close()
    return out
