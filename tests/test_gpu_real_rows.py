"""State in and out (the x passes from and to real fields) against the 2/3-dealiased
projection by an FP64 FFT, at sizes on both sides of the register prefetch of real
rows and at each thread count, from fields of either real type."""
import pytest

from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("n,precision", [(8, "fp64"), (64, "fp32"), (96, "fp32"), (96, "fp64"), (192, "fp64"),
                                         (256, "mixed"), (384, "fp32")])
def test_state_round_trip_is_the_projection(n, precision, dtype):
    from paper_1810_12707_amd.mhd import Solver

    log(f"[real rows] n={n} {precision} {dtype}")
    g = torch.Generator(device="cuda:0").manual_seed(n)
    U = torch.randn(8, n, n, n, dtype=torch.float64, device="cuda:0", generator=g).to(getattr(torch, dtype))
    S = Solver(n, precision, nu=1e-3, eta=1e-3, dt=1e-3)
    S.set_state(U)
    got = S.get_state(getattr(torch, dtype)).double()
    K = (n - 1) // 3
    k = torch.arange(n, device="cuda:0")
    keep = torch.minimum(k, n - k) <= K
    mask = keep[:, None, None] & keep[None, :, None] & keep[None, None, :n // 2 + 1]
    # a transform's rounding error is within eps log2(n^3) of its rms: twice 27 eps at 384;
    # the mixed path's split products keep 16 bits (2^-16 per radix-16 pass, four of them)
    fp32 = 54 * 2.0 ** -24
    bar = {"fp64": 54 * 2.0 ** -53, "fp32": fp32, "mixed": 4 * 2.0 ** -16}[precision]
    if dtype == "float32":
        bar = max(bar, fp32)
    for f in range(8):
        want = torch.fft.irfftn(torch.fft.rfftn(U[f].double()) * mask, s=(n, n, n))
        err = float((got[f] - want).norm() / want.norm())
        assert err <= bar, (f, err)
    S.close()
