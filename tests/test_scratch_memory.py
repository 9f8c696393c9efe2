"""The contraction kernels keep everything in registers and LDS: the built
library's own kernel descriptors (no GPU) ask for no scratch memory.  Register
spills there would also take part in the memory counters that the FP64 form's
written-out waits count.  One kernel is left out: the BF16x6 batch of problems
that leave products out and problems that do not."""
import re
import shutil
import subprocess

import pytest

import paper_1504_04653_amd.build as build

TOOLS = "/opt/rocm/lib/llvm/bin/"


def test_contraction_kernels_use_no_scratch(tmp_path):
    if shutil.which(TOOLS + "llvm-readelf") is None:
        pytest.skip("llvm-readelf not available")
    lib = tmp_path / "lib.so"
    shutil.copy(build.LIB, lib)
    subprocess.run([TOOLS + "llvm-objdump", "--offloading", lib.name], cwd=tmp_path, check=True, capture_output=True)
    scratch = {}
    for obj in sorted(tmp_path.glob("*gfx950")):
        notes = subprocess.run([TOOLS + "llvm-readelf", "--notes", str(obj)], check=True, capture_output=True, text=True).stdout
        name = None
        for line in notes.splitlines():
            if m := re.match(r"\s+\.name:\s+(\S*k_(?:class|batch)_\S+)", line):
                name = m.group(1)
            elif re.match(r"\s+\.name:", line):
                name = None
            elif name and (m := re.match(r"\s+\.private_segment_fixed_size:\s+(\d+)", line)):
                scratch[name] = int(m.group(1))
    assert sum("k_class" in n for n in scratch) >= 8 and sum("k_batch" in n for n in scratch) >= 4
    mixed = [n for n in scratch if "k_batch_bf16ILi3ELi2E" in n]
    assert len(mixed) == 1 and scratch.pop(mixed[0]) <= 128
    assert not {n: b for n, b in scratch.items() if b}
