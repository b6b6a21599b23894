"""Registers and scratch memory of kernels whose launchers or comments count on
them, from the built library's own metadata.  Needs no GPU."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_29707_amd import binding as bd

LLVM = "/opt/rocm/llvm/bin/"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled name: (vector registers, scratch bytes a lane)} of every kernel."""
    if not os.path.exists(LLVM + "llvm-objdump"):
        pytest.skip("no LLVM tools")
    d = tmp_path_factory.mktemp("co")
    shutil.copy(bd.LIB_PATH, d / "lib.so")
    subprocess.run([LLVM + "llvm-objdump", "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    out = {}
    for f in d.glob("*gfx950*"):
        notes = subprocess.run([LLVM + "llvm-readelf", "--notes", str(f)], capture_output=True, text=True).stdout
        for block in re.split(r"\n\s+- \.agpr_count:", notes)[1:]:
            get = {k: v for k, v in re.findall(r"\.(name|vgpr_count|private_segment_fixed_size):\s+(\S+)", block)
                   if k != "name" or v.startswith("_Z")}
            name = subprocess.run(["c++filt", get["name"]], capture_output=True, text=True).stdout.strip()
            out[re.sub(r"^void ", "", name).split("(")[0]] = (int(get["vgpr_count"]), int(get["private_segment_fixed_size"]))
    assert len(out) > 50
    return out


# (name, most registers, most scratch): 256 registers leave two waves a SIMD, 64 eight
@pytest.mark.parametrize("pattern,count,regs,spill", [
    # two workgroups of four waves a CU, one of eight
    (r"dk::attn_flash_kernel<", 4, 256, 0),
    # eight workgroups of four waves a CU; five with 16 single values a thread
    (r"dk::argmax_partial_kernel<\w+, [01]>", 4, 64, 0),
    (r"dk::argmax_partial_kernel<\w+, 16>", 2, 102, 0),
    # the operands in flight in registers: one fragment spills, no array of them lies in private memory
    (r"dk::train_ce_kernel<", 6, 256, 32),
])
def test_registers_and_scratch(kernels, pattern, count, regs, spill):
    found = {n: v for n, v in kernels.items() if re.match(pattern, n)}
    assert len(found) == count, sorted(kernels)
    for name, (vgprs, scratch) in found.items():
        assert vgprs <= regs and scratch <= spill, (name, vgprs, scratch)
