"""Column passes that store past the caches: chosen by a launch's output bytes, so a
group of runs takes them where a run by itself does not.  The values stored are the
same, so the states agree bit for bit."""
import pytest

from paper_1810_12707_amd import inputs as I
from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# output bytes of a launch at 128^3: 25 MB per FP32 run and 4 fields, 75 MB per 12
# fields, twice that in FP64; the rule turns at 256 MiB
@pytest.mark.parametrize("precision,members", [("fp32", 3), ("fp32", 4), ("fp32", 12), ("fp64", 4), ("mixed", 4)])
def test_group_equals_runs_alone(precision, members):
    from paper_1810_12707_amd.mhd import Ensemble, Solver

    log(f"[stream] 128 {precision} {members}")
    n = 128
    cases = [I.random_turbulence(n, b_rms=0.3, seeds=(81 + s, 91 + s, 101 + s)) for s in range(2)]
    fields = [torch.from_numpy(c.U).to("cuda:0") for c in cases]
    par = [dict(gamma=cases[i % 2].gamma, nu=1e-3 * (1 + i), eta=2e-3, dt=cases[i % 2].dt) for i in range(members)]
    E = Ensemble([dict(n=n, precision=precision, **p) for p in par])
    for i in range(members):
        E.set_state(i, fields[i % 2])
    E.step(3)
    schedule = E.groups()[0]["schedule"]
    for i in (0, members - 1):
        S = Solver(n, precision, **par[i])
        S.set_state(fields[i % 2])
        S.set_schedule(schedule)
        S.step(3)
        S.set_schedule(0)
        got = E.get_state(i)
        assert torch.isfinite(got).all()
        assert torch.equal(got, S.get_state()), f"member {i}"
        S.close()
    E.close()
