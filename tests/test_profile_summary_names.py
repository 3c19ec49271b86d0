"""The rocprofv3 summary tool on the kernel names the library has: launch classes found
under either way of storing, and no size taken for another that begins like it."""
import csv
import re

import pytest

from paper_1810_12707_amd import profile_summary as P
from tests.kernel_table import kernel_table
from tests.test_profile_summary import HEAD


def names_of(table, n, mixed):
    """The kernel of every launch class of a step, as the library's metadata has it."""
    mx = "true" if mixed else "false"
    out = {}
    for cls, start in P.STEP_SEQUENCE:
        start = start.format(n=n, mx=mx)
        hits = [k for k in table if P.is_kernel(k, start) and not k.startswith("sched1::")]
        assert hits, (cls, start)
        out[cls] = hits
    return out


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("n", [48, 128, 256, 384, 512, 1024])
def test_every_class_is_found(tmp_path, n, mixed):
    table = kernel_table()
    names = names_of(table, n, mixed)
    for cls, hits in names.items():
        # one kernel, or the two ways a column pass stores
        assert len({re.sub(r", (true|false)>$", "", k) if "k_col" in k else k for k in hits}) == 1, hits
    rows = []
    for step in range(2):
        for i, cls in enumerate(c for c, _ in P.STEP_SEQUENCE):
            rows.append((f"void mhd::{names[cls][step % len(names[cls])]}(mhd::Args)", 10.0 * i + step))
    path = tmp_path / "c.csv"
    with open(path, "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(HEAD)
        for i, (name, value) in enumerate(rows):
            row = dict.fromkeys(HEAD, 1)
            row.update(Dispatch_Id=i + 1, Kernel_Name=name, Counter_Name="FETCH_SIZE", Counter_Value=value)
            w.writerow([row[h] for h in HEAD])
    got = P.per_class_kib(str(path), "FETCH_SIZE", n, mixed)
    assert got == {c: (10.0 * i + 0.5, 2) for i, (c, _) in enumerate(P.STEP_SEQUENCE)}


def test_a_size_is_matched_whole():
    for cls, start in P.class_kernels(12).items():
        if "12" in start:
            assert not P.is_kernel(start.replace("12", "128") + ">", start), cls
            assert P.is_kernel(start + ">", start) and P.is_kernel(start + ", false>", start), cls
