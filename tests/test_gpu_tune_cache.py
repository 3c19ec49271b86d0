"""The ensemble's tuning cache holds choices measured for one build's kernels: a line
that another build wrote (or one that names no build) is not applied to these."""
import pytest

from paper_1810_12707_amd import inputs as I
from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def ensemble(path):
    from paper_1810_12707_amd.mhd import Ensemble

    c = I.random_turbulence(32, b_rms=0.3, seeds=(11, 12, 13))
    E = Ensemble([dict(n=32, precision="fp32", gamma=c.gamma, nu=1e-3, eta=1e-3, dt=c.dt)] * 2, tune_cache=str(path))
    U = torch.from_numpy(c.U).to("cuda:0")
    for i in range(2):
        E.set_state(i, U)
    return E


def test_lines_of_other_builds_are_not_applied(tmp_path):
    log("[tune cache]")
    path = tmp_path / "tune.txt"
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    old = f"mhd-ens-tune 32 1 2 {cus} 0.2500 0.5000 1"
    other = old + " 0"
    from paper_1810_12707_amd.mhd import MHD_FP32
    assert MHD_FP32 == 1
    path.write_text(f"{old}\n{other}\n")
    E = ensemble(path)
    g = E.groups()[0]
    assert (g["col_scale"], g["row_scale"], g["schedule"]) == (1.0, 1.0, 0)
    E.step(2)  # tunes, and appends this build's choice
    g = E.groups()
    E.close()
    lines = path.read_text().splitlines()
    assert lines[:2] == [old, other] and len(lines) == 3
    # this build's own line is: with its choices replaced by others, those come back
    words = lines[2].split()
    words[5:8] = ["0.2500", "0.5000", "1"]
    path.write_text(" ".join(words) + "\n")
    E = ensemble(path)
    g = E.groups()[0]
    assert (g["col_scale"], g["row_scale"], g["schedule"]) == (0.25, 0.5, 1)
    E.close()
