"""Build the HIP library paper_2011_09337_amd/libvit.so for gfx950.

Every call recompiles.  Sources are compiled in parallel (one hipcc per file),
then linked into a shared library next to this file.
"""
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libvit.so")
BUILD_DIR = os.path.join(ROOT, "_build")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

SOURCES = ["vit_api.cpp", "vit_batch.cpp", "vit_batch_static.cpp", "vit_server.cpp", "vit_launch.hip", "vit_quantize.hip", "vit_copy.hip", "vit_expand.hip", "vit_depuncture.hip", "vit_check.hip"] + [f"vit_kernels_k{k}.hip" for k in range(3, 10)] + [f"vit_kernels_sub_k{k}.hip" for k in range(3, 10)] + [f"vit_kernels_int_k{k}.hip" for k in range(3, 10)] + [f"vit_kernels_mx_k{k}.hip" for k in range(3, 10)] + [f"vit_kernels_row_k{k}.hip" for k in range(3, 7)] + [f"vit_kernels16_k{k}.hip" for k in range(3, 10)]

COMMON = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off",                   # every add rounded once, as written
    "-fno-gpu-flush-denormals-to-zero",    # keep fp32 denormals (IEEE, like the oracle)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def check_named_registers(asm):
    """The matrix-core kernels keep survivor words in v128..v255 (4 metric
    registers: v64..v127), which they move by asm that names them
    (vit_decoder_mx.h): an instruction of the compiler's own on one of those, or
    on an AGPR, would destroy them.  Raises RuntimeError if the assembly file
    holds one."""
    kernel, first, inside = None, 0, False
    with open(asm) as f:
        for line in f:
            label = re.match(r"(\S*vit_\w+_(quad|mx)_kernel\S*):", line)
            if label:
                kernel, first = label.group(1), 64 if label.group(2) == "quad" else 128
            elif "#ASMSTART" in line:
                inside = True
            elif "#ASMEND" in line:
                inside = False
            elif kernel and not inside and line.startswith("\t") and not line.strip().startswith((".", ";")):
                code = line.split(";")[0]
                regs = [int(x) for m in re.findall(r"\bv(?:(\d+)|\[(\d+):(\d+)\])", code) for x in m if x]
                if any(r >= first for r in regs) or re.search(r"\ba(\d+|\[)", code):
                    raise RuntimeError(f"{asm}: {kernel}: the compiler uses a register that the kernel names: {code.strip()}")
    if kernel is None:
        raise RuntimeError(f"{asm}: no matrix-core kernel found")


def _compile(src, verbose):
    obj = os.path.join(BUILD_DIR, os.path.basename(src) + ".o")
    lang = ["-x", "hip"] if src.endswith(".hip") else ["-x", "hip"]
    mx = src.startswith("vit_kernels_mx")
    if mx:
        lang = ["-save-temps=obj"] + lang
    cmd = [HIPCC] + COMMON + lang + ["-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    # hipcc's host pass warns about the device-only target feature; drop that noise
    msg = "\n".join(ln for ln in (res.stdout + res.stderr).splitlines()
                    if "packed-fp32-ops" not in ln and ln.strip())
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{msg}")
    if msg and verbose:
        print(msg)
    if mx:
        check_named_registers(os.path.join(BUILD_DIR, f"{os.path.splitext(src)[0]}-hip-amdgcn-amd-amdhsa-{ARCH}.s"))
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 4)) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-q" not in sys.argv))
