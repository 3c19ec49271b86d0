"""Tracers that start far outside the box, at up to 4 x 10^17: the cell index taken
in whole numbers, the weights in FP64, as for any other position."""
import numpy as np
import pytest

from paper_1810_12707_amd import inputs as I
from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def cic(field, pos):
    """Cloud-in-cell values of field [z][y][x] at pos (np, 3), indices in Python integers."""
    n = field.shape[0]
    s = pos / (2.0 * np.pi / n)
    fl = np.floor(s)
    i0 = np.array([[int(v) % n for v in row] for row in fl])
    w1 = s - fl
    out = np.zeros(len(pos))
    for c in range(8):
        b = [(c >> a) & 1 for a in range(3)]
        w = np.prod([w1[:, a] if b[a] else 1.0 - w1[:, a] for a in range(3)], axis=0)
        i = [(i0[:, a] + b[a]) % n for a in range(3)]
        out += w * field[i[2], i[1], i[0]]
    return out


@pytest.mark.parametrize("n,precision", [(12, "fp64"), (48, "fp32"), (64, "fp64")])
def test_positions_of_any_size(n, precision):
    from paper_1810_12707_amd.mhd import Solver

    log(f"[far tracers] n={n} {precision}")
    S = Solver(n, precision)
    S.set_state(torch.from_numpy(I.compressive_state(n, 3)).to("cuda:0"))
    G = S.get_state(torch.float64).cpu().numpy()
    rng = np.random.default_rng(2)
    # 4e17: within 2^62 cells at every size here
    p = rng.uniform(-1.0, 1.0, (600, 3)) * 10.0 ** rng.uniform(0.0, np.log10(4e17), (600, 3))
    pos = torch.from_numpy(p.copy()).to("cuda:0")
    vel = S.tracer_velocity(pos)
    want = np.stack([cic(G[1 + i] / G[0], p) for i in range(3)], axis=1)
    tol = 1e-12 if precision == "fp64" else 1e-6  # the bounds of positions inside the box
    assert np.abs(vel.cpu().numpy() - want).max() <= tol * np.abs(want).max()
    # one push: the field at the start, the rotation it makes, the position wrapped
    dt, v = 0.05, vel.cpu().numpy()
    t = 0.5 * dt * np.stack([cic(G[4 + i], p) for i in range(3)], axis=1)
    s = 2.0 * t / (1.0 + (t * t).sum(1, keepdims=True))
    v = v + np.cross(v + np.cross(v, t), s)
    S.tracer_push(pos, vel, dt, 1)
    assert np.abs(vel.cpu().numpy() - v).max() <= tol * np.abs(v).max()
    x = pos.cpu().numpy()
    assert (x >= 0.0).all() and (x <= 2.0 * np.pi).all()
    # a second step from there, with a particle that is nowhere beside them
    pos[0] = float("nan")
    S.tracer_push(pos, vel, dt, 2)
    assert torch.isnan(vel[0]).all() and torch.isfinite(vel[1:]).all() and torch.isfinite(pos[1:]).all()
    S.close()
