"""State out and diagnostics at 768^3, whose row passes have thread counts and an LDS
layout of their own, against the fields the state was set from (trigonometric, so
exactly band-limited) and their FP64 means."""
import math

import pytest

from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["fp32", "mixed"])
def test_state_and_diagnostics(precision):
    from paper_1810_12707_amd.mhd import Solver

    n = 768
    log(f"[768] {precision}")
    x = torch.arange(n, device="cuda:0", dtype=torch.float64) * (2 * math.pi / n)
    X, Y, Z = x[None, None, :], x[None, :, None], x[:, None, None]
    fields = [lambda: 1.0 + 0.2 * torch.sin(X + 2 * Y) * torch.cos(Z),
              lambda: 0.3 * torch.sin(Z) + 0.1 * torch.cos(3 * X - Y), lambda: 0.2 * torch.cos(X + Z) - 0.1 * Y.cos(),
              lambda: 0.1 * torch.sin(2 * X) * torch.sin(Y + Z), lambda: 0.2 * torch.cos(Y) + 0.05 * torch.sin(Z),
              lambda: 0.1 * torch.sin(X - Z), lambda: 0.3 + 0.1 * torch.cos(2 * X + Y),
              lambda: 2.0 + 0.1 * torch.sin(X) * torch.sin(Y) * torch.sin(Z)]
    U = torch.empty(8, n, n, n, dtype=torch.float32, device="cuda:0")
    for f, make in enumerate(fields):
        U[f] = make().expand(n, n, n).float()
    S = Solver(n, precision)
    S.set_state(U)
    got = S.get_state(torch.float32)
    # two transforms within eps log2(n^3) of their rms each (29 eps at 768); the mixed
    # path's split products keep 16 bits (2^-16 per radix-16 pass, four of them)
    bar = {"fp32": 58 * 2.0 ** -24, "mixed": 4 * 2.0 ** -16}[precision]
    for f in range(8):
        err = float((got[f] - U[f]).norm() / U[f].norm())
        log(f"  field {f}: {err:.2e}")
        assert err <= bar, f
    rc, d = S.diagnostics()
    assert rc == 0
    rho, m, B, E = U[0], U[1:4], U[4:7], U[7]

    def mean(v):
        return float(sum(p.double().sum() for p in v)) / n ** 3  # plane by plane

    kin = (m[0] * m[0] + m[1] * m[1] + m[2] * m[2]) / rho * 0.5
    mag = (B[0] * B[0] + B[1] * B[1] + B[2] * B[2]) * 0.5
    want = {"mass": mean(rho), "e_kin": mean(kin), "e_mag": mean(mag), "e_tot": mean(E),
            "h_cross": mean((m[0] * B[0] + m[1] * B[1] + m[2] * B[2]) / rho),
            "e_int": mean(E - kin - mag)}
    # a mean is off by at most its integrand's relative error against its mean square's
    # root: the products double the fields' own bound
    scale = {"mass": 1.0, "e_tot": 2.0, "e_int": 2.0}
    for key, w in want.items():
        log(f"  {key}: {d[key]:.9f} {w:.9f}")
        assert abs(d[key] - w) <= 4 * bar * scale.get(key, 1.0), key
    S.close()
