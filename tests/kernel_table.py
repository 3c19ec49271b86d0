"""Kernels of the built library: the metadata (registers, scratch, LDS, workgroup
size) the compiler wrote into the gfx950 code objects that libmhd.so carries."""
import os
import re
import struct
import subprocess
import tempfile

import pytest

from paper_1810_12707_amd.build_lib import LIB

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
CXXFILT = "/usr/bin/c++filt"
KEYS = {"scratch": "private_segment_fixed_size", "vgprs": "vgpr_count", "threads": "max_flat_workgroup_size",
        "lds": "group_segment_fixed_size"}
EM_AMDGPU = 224


def _code_objects(data):
    at = data.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            shoff, = struct.unpack_from("<Q", data, at + 40)
            shentsize, shnum = struct.unpack_from("<HH", data, at + 58)
            yield data[at:at + shoff + shentsize * shnum]
        at = data.find(b"\x7fELF", at + 4)


def kernel_table():
    """Kernel name without its parameters -> {scratch, vgprs, threads, lds}."""
    for tool in (LIB, READELF, CXXFILT):
        if not os.path.exists(tool):
            pytest.skip(f"{tool} not available")
    with open(LIB, "rb") as f:
        data = f.read()
    found = {}
    for obj in _code_objects(data):
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(obj)
            f.flush()
            notes = subprocess.run([READELF, "--notes", f.name], capture_output=True, text=True, check=True).stdout
        for block in re.split(r"\n  - (?=\.a)", notes)[1:]:
            name = re.search(r"\.name:\s+(\S+)", block)
            if name and ".max_flat_workgroup_size" in block:
                found[name.group(1)] = {k: int(re.search(rf"\.{v}:\s+(\d+)", block).group(1)) for k, v in KEYS.items()}
    plain = subprocess.run([CXXFILT], input="\n".join(found), capture_output=True, text=True, check=True).stdout
    return {p.replace("void ", "").replace("mhd::", "").split("(")[0]: found[n]
            for n, p in zip(found, plain.splitlines())}
