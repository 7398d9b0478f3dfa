"""Builds libdcpq.so (hand-written HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libdcpq.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# -ffp-contract=off and the correctly rounded divide keep the fp32 stages that decide integers
# bit-reproducible; packed-fp32 code generation is switched off for the whole library.
HIP_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-ffp-contract=off",
    "-fhip-fp32-correctly-rounded-divide-sqrt", "-fno-fast-math",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


# The double-precision matrix kernels keep 64 accumulator registers per lane over their k loops.  Left to
# itself the compiler holds them in ordinary registers across the loop edge and copies all 64 into and out
# of the accumulation registers in every iteration (128 copies around 8 matrix instructions); this option
# makes the matrix instructions work on ordinary registers directly.
EXTRA_FLAGS = {
    "tables_full.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    "assign.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    "assign_middle.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    "assign_long.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    # a few lanes of a wavefront count their hits with an LDS atomic each; the compiler's scan over all 64
    # lanes in its place costs several times the instructions
    "scan_cells.hip": ["-mllvm", "-amdgpu-atomic-optimizer-strategy=None"],
}


def sources() -> list[str]:
    return sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")))


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *HIP_FLAGS, *EXTRA_FLAGS.get(src, []), "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    p = subprocess.run(cmd, capture_output=True, text=True)
    if p.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, p.stdout, p.stderr))
    warn = "\n".join(l for l in p.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
    return warn


def build(verbose: bool = False) -> str:
    """Compile every source for gfx950 and link the shared library; always recompiles."""
    os.makedirs(OBJ, exist_ok=True)
    srcs = sources()
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        for src, warn in zip(srcs, ex.map(_compile, srcs)):
            if verbose and warn:
                print("[%s]\n%s" % (src, warn))
    objs = [os.path.join(OBJ, os.path.splitext(s)[0] + ".o") for s in srcs]
    tmp = LIB + ".tmp%d" % os.getpid()
    p = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp],
                       capture_output=True, text=True)
    if p.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (p.stdout, p.stderr))
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
