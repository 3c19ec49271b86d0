"""Large grids in the forms tests/test_gpu_fullsize.py leaves out: the right-hand side of
the radix-3 sizes in FP64 and mixed precision, of kinematic runs and runs with the
Laplacian viscous force at each thread count of their flux passes, and the stage updates
of every scheme where the z-RHS pass loads both flux groups up front.

The plans at these sizes: 192 (6,4,8), 384 (6,8,8), 768 (8,8,4,3); the mixed path's
column passes 192 (4,3,16), 384 (3,8,16), 768 (16,3,16)."""
import numpy as np
import pytest

from oracle import oracle as O
from tests import test_gpu_fullsize as F
from tests.gpu_helpers import log
from tests.test_gpu_integrators import flags_of, oracle_options

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GAMMA, NU, ETA = 5.0 / 3.0, 2e-3, 3e-3


@pytest.mark.parametrize("n,prec", [(192, "fp64"), (384, "fp64"), (192, "mixed"), (384, "mixed"), (768, "mixed")])
def test_rhs_exact(n, prec):
    F.test_rhs_exact_lowmode_state(n, prec)


def lowmode_fields(n, dtype):
    U0 = F.lowmode_state(32)
    U = torch.empty((8, n, n, n), dtype=dtype, device="cuda:0")
    for f in range(8):
        U[f] = F.upsample_field_gpu(U0[f], n).to(dtype)
    return U0, U


# threads of the kinematic pass: 96 128, 128 128, 192 256, 256 256, 384 and 512 512
@pytest.mark.parametrize("n,prec", [(96, "fp32"), (128, "fp64"), (128, "mixed"), (192, "fp32"), (192, "fp64"),
                                    (256, "fp32"), (256, "fp64"), (384, "fp64"), (384, "mixed"), (512, "fp32"),
                                    (512, "fp64")])
@pytest.mark.parametrize("variant", ["kin", "lap"])
def test_variant_rhs_exact(variant, n, prec):
    """rho = 1 and modes up to 2: the exact right-hand side is a trigonometric polynomial
    of modes up to 6, the oracle's at 32^3.  What rounding leaves: a flux is off by
    eps log2(n^3) of its size per transform (27 eps at 512, two transforms and the
    products: 64 eps; mixed: 2^-16 per radix-16 pass, four of them), white over the band,
    and the divergence or curl multiplies it by up to sqrt(3) K.  In FP32 most of that lies
    outside the 13^3 modes that hold the answer; those are held to the bounds of
    tests/test_gpu_fullsize.py."""
    log(f"[fullsize {variant}] n={n} {prec}")
    U0, U = lowmode_fields(n, torch.float64 if prec == "fp64" else torch.float32)
    R0 = O.rhs(U0, GAMMA, NU, ETA, options=oracle_options(variant))
    S = F.solver(n, prec, gamma=GAMMA, nu=NU, eta=ETA, flags=flags_of(variant))
    out = S.rhs(U)
    S.close()
    K = (n - 1) // 3
    eps = {"fp64": 64 * 2.0 ** -53, "fp32": 64 * 2.0 ** -24, "mixed": 4 * 2.0 ** -16}[prec]
    idx = np.r_[-6:7] % 32
    exact = (np.fft.fftn(R0, axes=(-3, -2, -1)) / 32 ** 3)[:, idx[:, None, None], idx[None, :, None], idx[None, None, :]]
    low = F.low_mode_coefficients(out, 6).cpu().numpy()
    low_tol = {"fp64": 1e-11, "fp32": 1e-5, "mixed": 1e-3}[prec]
    flux = 10.0  # (E + P_tot) u, the largest of them: 3 + 2 times a velocity of rms 0.5
    for f in range(8):
        want = F.upsample_field_gpu(R0[f], n, kmax=6)
        if not np.any(R0[f]):
            assert float(out[f].abs().max()) == 0.0  # frozen
            continue
        err = float((out[f].double() - want).pow(2).mean().sqrt())
        log(f"  field {f}: rms error {err:.2e}, bound {eps * flux * 3.0 ** 0.5 * K:.2e}, rms {float(want.pow(2).mean().sqrt()):.2e}")
        assert err <= eps * flux * 3.0 ** 0.5 * K, f
        rel = np.linalg.norm(low[f] - exact[f]) / np.linalg.norm(exact[f])
        log(f"  field {f}: low modes rel {rel:.2e}")
        assert rel <= low_tol, f


@pytest.mark.parametrize("scheme", ["ab2", "pc", "rk4"])
@pytest.mark.parametrize("n,prec", [(512, "fp64"), (512, "fp32"), (384, "fp64"), (48, "fp64")])
def test_stage_updates(n, prec, scheme):
    """Two steps against the scheme written out over the library's own right-hand sides,
    which take no update."""
    log(f"[stages] n={n} {prec} {scheme}")
    dt = 4e-3
    dtype = torch.float64 if prec == "fp64" else torch.float32
    U = lowmode_fields(n, dtype)[1]
    S = F.solver(n, prec, gamma=GAMMA, nu=NU, eta=ETA, dt=dt, scheme=scheme)
    S.set_state(U)
    U = S.get_state(dtype)
    prev = None
    for step in range(2):
        R = S.rhs(U)
        if scheme == "rk4":
            acc, k = R.clone(), R
            for h, w in ((0.5 * dt, 2.0), (0.5 * dt, 2.0), (dt, 1.0)):
                k = S.rhs(U + h * k)
                acc += w * k
            U = U + (dt / 6.0) * acc
            continue
        new = U + dt * (R if prev is None else 1.5 * R - 0.5 * prev)
        U = U + 0.5 * dt * (R + S.rhs(new)) if scheme == "pc" else new
        prev = R
    S.step(2)
    got = S.get_state(dtype)
    S.close()
    # Rounding, which adds like random steps: eps (log2 n^3)^1/2 of the state's rms per
    # transform, two transforms in and out; and dt times the noise of the right-hand sides
    # (eps |P| max |k|, as in tests/test_gpu_fullsize.py), up to eight of them.  A stage left
    # out or weighed wrongly would show as (dt k c)^2 / 2 ~ 1e-4 of the state.
    K = (n - 1) // 3
    eps = 2.0 ** (-52 if prec == "fp64" else -23)
    for f in range(8):
        rms = float(U[f].double().pow(2).mean().sqrt())
        bound = 4 * np.log2(n ** 3) ** 0.5 * eps * rms + 8 * dt * eps * 3.0 * 3.0 ** 0.5 * K
        err = float((got[f].double() - U[f].double()).pow(2).mean().sqrt())
        log(f"  field {f}: rms error {err:.2e}, bound {bound:.2e}, rms {rms:.2e}")
        assert err <= bound, f
