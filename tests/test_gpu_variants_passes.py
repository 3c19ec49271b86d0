"""The integrators and the Section V variants against the FP64 oracle on the grids that
run pass by pass: 48^3 (the first mixed plan) and 64^3 (the wave-mapped row passes).
Up to 32^3 the fused passes run instead (tests/test_gpu_integrators.py, whose start and
bounds these are)."""
import functools

import numpy as np
import pytest

from oracle import oracle as O
from paper_1810_12707_amd import inputs as I
from tests.gpu_helpers import log, per_field_rel_l2
from tests.test_gpu_integrators import BAR, dev, flags_of, oracle_options, solver

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

STEPS = 4


def start(n):
    return I.abc_dynamo(n, nu=2e-2, eta=3e-2, dt=2e-3, b_rms=0.2, seed=9)


@functools.lru_cache(maxsize=None)
def reference(n, variant, force, scheme):
    c = start(n)
    return O.run(c.U, STEPS, c.dt, c.gamma, c.nu, c.eta, scheme=scheme, options=oracle_options(variant), force=force)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "mixed"])
@pytest.mark.parametrize("variant,force,scheme", [("plain", 0.0, "rk4"), ("plain", 0.0, "pc"), ("lap", 0.0, "ab2"),
                                                  ("plain", 0.3, "ab2"), ("kin", 0.0, "ab2"), ("lap", 0.3, "rk4"),
                                                  ("kin", 0.2, "pc")])
@pytest.mark.parametrize("n", [48, 64])
def test_steps_against_oracle(n, variant, force, scheme, prec):
    log(f"[variant] {variant} force={force} {scheme} n={n} prec={prec}")
    c, ref = start(n), reference(n, variant, force, scheme)
    S = solver(n, prec, gamma=c.gamma, nu=c.nu, eta=c.eta, dt=c.dt, scheme=scheme, flags=flags_of(variant),
               force=force)
    S.set_state(dev(c.U))
    S.step(STEPS)
    got = S.get_state(torch.float64).cpu().numpy()
    S.close()
    errs = per_field_rel_l2(got, ref)
    log("  ", ["%.2e" % e for e in errs])
    assert max(errs) <= BAR[prec]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "mixed"])
@pytest.mark.parametrize("variant,force", [("lap", 0.0), ("plain", 0.4), ("kin", 0.0)])
@pytest.mark.parametrize("n", [48, 64])
def test_rhs_against_oracle(n, variant, force, prec):
    log(f"[variant rhs] {variant} force={force} n={n} prec={prec}")
    gamma, nu, eta = 5.0 / 3.0, 3e-3, 5e-3
    U = I.compressive_state(n, 300 + n, gamma)
    ref = O.rhs(U, gamma, nu, eta, options=oracle_options(variant), force=force)
    S = solver(n, prec, gamma=gamma, nu=nu, eta=eta, flags=flags_of(variant), force=force)
    got = S.rhs(dev(U).to(torch.float64 if prec == "fp64" else torch.float32)).double().cpu().numpy()
    S.close()
    live = [f for f in range(8) if np.abs(ref[f]).max() > 0]
    errs = [float(np.linalg.norm(got[f] - ref[f]) / np.linalg.norm(ref[f])) for f in live]
    log("  ", ["%.2e" % e for e in errs])
    assert max(errs) <= BAR[prec]
    for f in set(range(8)) - set(live):
        assert np.abs(got[f]).max() == 0.0
