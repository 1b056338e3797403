"""The matrix-core kernels keep survivor words in v128..v255 (with 4 metric
registers: v64..v127), which they move by asm that names them: the compiler must
not use those registers itself.  This compiles each source to assembly and looks
at every instruction outside asm."""
import importlib.util
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _assembly(job):
    hipcc_args, src, asm = job
    subprocess.run([HIPCC] + hipcc_args + ["--cuda-device-only", "-S", "-x", "hip", src, "-o", asm], check=True,
                   capture_output=True)
    return asm


@pytest.mark.skipif(not shutil.which(HIPCC), reason="no hipcc")
def test_named_registers_are_the_kernels_own(tmp_path):
    spec = importlib.util.spec_from_file_location("vit_build", os.path.join(ROOT, "paper_2011_09337_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    jobs = [(build.COMMON, os.path.join(build.CSRC, f"vit_kernels_mx_k{k}.hip"), str(tmp_path / f"k{k}.s"))
            for k in range(3, 10)]
    with ThreadPoolExecutor(7) as pool:
        for asm in pool.map(_assembly, jobs):
            _check(asm)


def _check(asm):
    inside, first, own, named, counts = False, 0, [], {}, {}
    for line in open(asm):
        label = re.match(r"(_ZN\S*vit_\w+_(quad|mx)_kernel\S*):", line)
        if label:
            kernel, first = label.group(1), {"quad": 64, "mx": 128}[label.group(2)]
            named[kernel] = 0
        elif re.match(r"\s+\.name:\s+_ZN", line):
            kernel = line.split()[-1]
        elif "#ASMSTART" in line:
            inside = True
        elif "#ASMEND" in line:
            inside = False
        elif ".vgpr_count:" in line:
            counts[kernel] = int(line.split()[-1])
        elif line.startswith("\t") and not line.strip().startswith((".", ";")):
            code = line.split(";")[0]
            regs = [int(x) for group in re.findall(r"\bv(?:(\d+)|\[(\d+):(\d+)\])", code) for x in group if x]
            if any(r >= first for r in regs) or re.search(r"\ba(\d+|\[)", code):
                if inside:
                    named[kernel] += 1
                else:
                    own.append(line)
    assert not own, (asm, own[:5])
    assert named.keys() == counts.keys() and counts
    for kernel, count in counts.items():  # each names its registers, and claims them from the hardware
        size = 64 if "_quad_" in kernel else 128
        assert named[kernel] >= 2 * size and count == 2 * size, (kernel, named[kernel], count)
