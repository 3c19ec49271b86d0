"""Launch shapes and scratch of the built kernels (CPU only: read from the library)."""
import pytest

from tests.kernel_table import kernel_table

SIZES = (8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024)
RM_XDIAG, RM_XFWD_ONE, RM_XINV_ONE = 4, 7, 8


@pytest.fixture(scope="module")
def table():
    return kernel_table()


@pytest.mark.parametrize("mode", [RM_XFWD_ONE, RM_XINV_ONE])
def test_one_field_passes_take_one_wave(table, mode):
    """A call on one field has N / r_0 <= 128 butterflies per row pair: one wave's work."""
    for n in SIZES:
        for t in ("float", "double") if n <= 512 else ("float",):
            k = table[f"sched0::k_row<{t}, {n}, {mode}>"]
            assert k["threads"] == 64 and k["scratch"] == 0, (t, n, k)


def test_diagnostics_pass_does_not_spill(table):
    """28 FP64 accumulators beside the butterflies: the pass that comes nearest to 256
    registers.  The mixed path runs the FP32 one."""
    for n in SIZES:
        for t in ("float", "double") if n <= 512 else ("float",):
            k = table[f"sched0::k_row<{t}, {n}, {RM_XDIAG}>"]
            assert k["scratch"] == 0, (t, n, k)


def test_column_passes_stream_only_where_that_pays(table):
    """Stores past the caches (the last argument of k_col): not at 1024, nor from the
    mixed path's one-term inverse z pass at 768."""
    streamed = [k for k in table if k.startswith("sched0::k_col<") and k.endswith(", true>")]
    assert any("<float, 512, 1, 1, false, true, true>" in k for k in streamed)
    assert not [k for k in streamed if "<float, 1024, " in k or "<float, 768, 1, 1, true, true," in k]
