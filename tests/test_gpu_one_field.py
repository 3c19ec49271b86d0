"""Transforms of one field (mhd_fft3d), which run row passes of their own, against an
FP64 FFT at every grid size."""
import pytest

from tests.gpu_helpers import band, log, pitch

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = (8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512)


@pytest.mark.parametrize("n,precision", [(n, p) for n in SIZES for p in ("fp32", "fp64")] +
                         [(48, "mixed"), (256, "mixed"), (768, "fp32")])
def test_one_field_both_ways(n, precision):
    from paper_1810_12707_amd.mhd import Solver

    log(f"[one field] n={n} {precision}")
    S = Solver(n, precision)
    g = torch.Generator(device="cuda:0").manual_seed(n)
    f = torch.randn(n, n, n, dtype=S.real_dtype, device="cuda:0", generator=g)
    spec = S.fft_forward(f)
    K, nb, idx = band(n)
    keep = torch.from_numpy(idx).to("cuda:0")
    want = torch.fft.rfftn(f.double())[keep][:, keep][:, :, :K + 1]
    got = torch.view_as_complex(spec.double().reshape(nb, nb, pitch(n), 2)[:, :, :K + 1].contiguous())
    # a transform's rounding error is within eps log2(n^3) of its rms: 29 eps at 768; the
    # mixed path's split products keep 16 bits (2^-16 per radix-16 pass, two of them)
    bar = {"fp64": 29 * 2.0 ** -53, "fp32": 29 * 2.0 ** -24, "mixed": 2 * 2.0 ** -16}[precision]
    assert float((got - want).norm() / want.norm()) <= bar
    full = torch.zeros(n, n, n // 2 + 1, dtype=torch.complex128, device="cuda:0")
    full[keep[:, None, None], keep[None, :, None], torch.arange(K + 1, device="cuda:0")[None, None, :]] = got
    back = torch.fft.irfftn(full, s=(n, n, n))
    out = S.fft_inverse(spec)
    assert float((out.double() - back).norm() / back.norm()) <= bar
    S.close()
