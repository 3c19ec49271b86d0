"""Short tracer calls gather from the planes of the synthesised fields, long ones from
the interleaved grid: both against the oracle, on either side of the line."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1810_12707_amd import inputs as I
from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# 96^3 FP64: velocities interleave from 36000 particles, short pushes from three steps;
# 128^3 FP32: from 41000 particles and three steps; 64^3 FP32: always
@pytest.mark.parametrize("n,precision", [(96, "fp64"), (128, "fp32"), (64, "fp32")])
@pytest.mark.parametrize("count,steps", [(1, 1), (999, 2), (999, 3), (50000, 1), (50000, 4)])
def test_velocity_and_push(n, precision, count, steps):
    from paper_1810_12707_amd.mhd import Solver

    log(f"[tracer routes] n={n} {precision} {count} x {steps}")
    S = Solver(n, precision)
    S.set_state(torch.from_numpy(I.compressive_state(n, 4)).to("cuda:0"))
    G = S.get_state(torch.float64).cpu().numpy()
    p0 = np.random.default_rng(count + steps).uniform(0.0, 2.0 * np.pi, (count, 3))
    pos = torch.from_numpy(p0.copy()).to("cuda:0")
    vel = S.tracer_velocity(pos)
    want = O.cic(G[1:4] / G[0], p0)
    tol = 1e-12 if precision == "fp64" else 1e-6  # the bounds of tests/test_gpu_tracers.py
    v0 = vel.cpu().numpy()
    assert np.abs(v0 - want).max() <= tol * np.abs(want).max()
    S.tracer_push(pos, vel, 0.05, steps)
    p1, v1 = O.tracer_push(G[4:7], p0, v0, 0.05, steps)
    d = (pos.cpu().numpy() - p1 + np.pi) % (2.0 * np.pi) - np.pi
    assert np.abs(d).max() <= 10 * tol
    assert np.abs(vel.cpu().numpy() - v1).max() <= 10 * tol * np.abs(v1).max()
    S.close()
