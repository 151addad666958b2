"""Builds libbbmm.so (HIP, gfx950) in-tree with hipcc.  Run: python -m paper_1809_11165_amd.build"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB_PATH = os.path.join(HERE, "libbbmm.so")
SOURCES = ["kernels_vec.hip", "kernels_mm.hip", "kernels_sym.hip", "kernels_sgpr.hip", "kernels_dig.hip",
           "kernels_words.hip", "bbmm_api.hip"]
# packed fp32 VALU ops are switched off for all device code
FLAGS = ["-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]

# The on-the-fly kernels use every fp32 MFMA result on the vector unit at once: with the results in
# ordinary registers the accumulator-register moves go (config 4 product 34.0 -> 32.3 ms; the other
# kernels of the file time the same).  The triangle kernel needs the accumulation registers and stays as it is.
EXTRA_FLAGS = {"kernels_mm.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
               "kernels_dig.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
               "kernels_words.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


def _run(cmd):
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in proc.stdout.splitlines() if "packed-fp32-ops" not in l)
    if proc.returncode != 0:
        raise RuntimeError("command failed: %s\n%s" % (" ".join(cmd), out))
    return out


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = [os.path.join(OBJ_DIR, s.replace(".hip", ".o")) for s in SOURCES]
    cmds = [[hipcc] + FLAGS + EXTRA_FLAGS.get(s, []) + ["-c", os.path.join(CSRC, s), "-o", o]
            for s, o in zip(SOURCES, objs)]
    with ThreadPoolExecutor(max_workers=len(cmds)) as ex:
        for out in ex.map(_run, cmds):
            if verbose and out.strip():
                print(out)
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH] + objs)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
