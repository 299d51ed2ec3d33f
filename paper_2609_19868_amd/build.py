"""Build libzarya.so (HIP, gfx950 only) in-tree with hipcc.

Usage: python -m paper_2609_19868_amd.build   (or call build()).
"""

from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import re
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD_DIR = os.path.join(PKG, "_build")
LIB_NAME = "libzarya.so"
LIB_PATH = os.path.join(PKG, LIB_NAME)

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # no packed fp32 instructions anywhere in the device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-I", INCLUDE,
    "-I", CSRC,
]
RESOURCE_FLAG = "-Rpass-analysis=kernel-resource-usage"


def _hipcc():
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the HIP toolchain is required to build libzarya")


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l and "not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"command failed ({r.returncode}): {' '.join(cmd)}\n{without_remarks(out)}")
    return out


def without_remarks(text):
    """Compiler output without its remarks and the source lines quoted under them."""
    keep, lines = True, []
    for l in text.splitlines():
        if re.search(r"(?:^|: )(remark|warning|error|note): ", l):
            keep = "remark: " not in l
        if keep:
            lines.append(l)
    return "\n".join(lines)


def kernel_resources(text):
    """{kernel: {field: number}} from the compiler's kernel-resource-usage remarks."""
    kernels, name = {}, None
    for field, value in re.findall(r"remark: +([^:\n]+): (\S+) \[-Rpass-analysis=kernel-resource-usage\]", text):
        if field == "Function Name":
            name = value
            kernels[name] = {}
        elif value.isdigit():
            kernels[name][field] = int(value)
    return kernels


def check_kernels(text):
    """Refuse kernels with scratch memory or spilled vector registers.  Their LDS
    reads are inline assembly whose results are in flight until a later wait, which
    the compiler does not know: a spill in between would store stale data."""
    for name, r in kernel_resources(text).items():
        if r["ScratchSize [bytes/lane]"] or r["VGPRs Spill"]:
            raise RuntimeError(f"{name}: {r['ScratchSize [bytes/lane]']} bytes of scratch, "
                               f"{r['VGPRs Spill']} spilled vector registers; no kernel may have either")


def build(verbose: bool = False) -> str:
    """Compile every HIP source under csrc/ and link libzarya.so next to this file."""
    hipcc = _hipcc()
    os.makedirs(BUILD_DIR, exist_ok=True)
    sources = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    objs = [os.path.join(BUILD_DIR, os.path.basename(s) + ".o") for s in sources]
    with cf.ThreadPoolExecutor(max_workers=min(8, len(sources))) as ex:
        outs = list(ex.map(lambda so: _run([hipcc, *HIPCC_FLAGS, RESOURCE_FLAG, "-c", so[0], "-o", so[1]]),
                           zip(sources, objs)))
    if not any(map(kernel_resources, outs)):
        raise RuntimeError(f"the compiler reported no kernel resources ({RESOURCE_FLAG})")
    for o in outs:
        check_kernels(o)
    tmp = LIB_PATH + ".tmp"
    # -z defs: a kernel whose host launch stub was not emitted fails the link here
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,-z,defs", "-o", tmp, *objs])
    os.replace(tmp, LIB_PATH)
    if verbose:
        for o in outs:
            o = without_remarks(o)
            if o.strip():
                print(o)
        print(f"built {LIB_PATH}")
    return LIB_PATH


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
