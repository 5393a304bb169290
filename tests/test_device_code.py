"""What the compiler made of code whose order matters between the waves of a workgroup, read from the library as it is built (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2602_06694_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def kernels(lib, tmp_path, pattern):
    """{kernel: its LDS accesses, matrix instructions and workgroup barriers, in the order of the code}"""
    here = shutil.copy(lib, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", here], check=True, capture_output=True, cwd=tmp_path)
    found = {}
    for name in sorted(os.listdir(tmp_path)):
        if "amdgcn" not in name:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(tmp_path / name)], check=True, capture_output=True, text=True).stdout
        events = None
        for line in text.splitlines():
            head = re.match(r"[0-9a-f]+ <(.+)>:", line)
            if head:
                events = found.setdefault(head.group(1), "") if re.search(pattern, head.group(1)) else None
                kernel = head.group(1)
            elif events is not None:
                op = line.split()[0] if line.split() else ""
                kind = "|" if op == "s_barrier" else "r" if op.startswith("ds_read") else "W" if op.startswith("ds_write") else "m" if "mfma" in op or "smfmac" in op else ""
                found[kernel] += kind
    return found


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_accumulators_handed_over_are_read_before_the_barrier(tmp_path):
    """Dense GEMM with the reduction halved inside the workgroup: in each of two rounds the second part's waves write 16 accumulators to LDS and
    the first part's read them, each between barriers.  Reads that the compiler moves past the last one race with
    other waves' epilogues, which write there."""
    if not os.path.exists(build.LIB):
        pytest.skip("library not built")
    found = kernels(build.LIB, tmp_path, r"prefill_gemm_kernelILi\dELi4ELi2E")
    assert len(found) == 6, sorted(found)
    for kernel, events in found.items():
        tail = events[events.rindex("m") + 1:]
        assert re.match(r"\|W{16}\|r{16}\|W{16}\|r{16}\|", tail), (kernel, tail[:100])
