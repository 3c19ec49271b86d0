"""Tracer positions outside the box, on cell faces and at the wrap: the same
velocities and pushes as from the positions taken modulo 2 pi."""
import numpy as np
import pytest

from paper_1810_12707_amd import inputs as I
from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,precision", [(8, "fp64"), (12, "fp32"), (48, "fp64")])
def test_positions_are_periodic(n, precision):
    from paper_1810_12707_amd.mhd import Solver

    log(f"[tracers] n={n} {precision}")
    S = Solver(n, precision)
    S.set_state(torch.from_numpy(I.compressive_state(n, 3)).to("cuda:0"))
    two_pi = 2.0 * np.pi
    rng = np.random.default_rng(1)
    p = rng.uniform(0.0, two_pi, (257, 3))
    p[0], p[1] = 0.0, np.nextafter(two_pi, 0.0)
    p[2:10] = np.arange(8)[:, None] * (two_pi / n)  # cell faces
    k = rng.integers(-3, 4, p.shape)
    k[20:30] *= 1000
    shifted = p + two_pi * k
    a, b = (torch.from_numpy(x.copy()).to("cuda:0") for x in (p, shifted))
    va, vb = S.tracer_velocity(a), S.tracer_velocity(b)
    # the shifted positions differ from p by their own rounding, |x| 2^-53, and
    # the interpolant's slope is at most max |du| / dx
    slope = float(va.abs().max()) * 2.0 * n / two_pi
    tol = 4.0 * slope * two_pi * 3000 * 2.0 ** -53
    assert float((va - vb).abs().max()) <= tol
    S.tracer_push(a, va, 0.05, 1)
    S.tracer_push(b, vb, 0.05, 1)
    for x in (a, b):
        assert float(x.min()) >= 0.0 and float(x.max()) <= two_pi
    d = (a - b).abs()
    d = torch.minimum(d, (d - two_pi).abs())
    assert float(d.max()) <= 4.0 * (tol + two_pi * 3000 * 2.0 ** -53)
    S.close()
