"""Builds the HIP library (csrc/*.hip -> libqzo.so) for gfx950 with hipcc."""
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libqzo.so")
OBJ = os.path.join(HERE, "_build")
SOURCES = ["qzo_elementwise.hip", "qzo_gemm.hip", "qzo_gemm_wide.hip", "qzo_w4.hip", "qzo_lmhead.hip", "qzo_skinny.hip", "qzo_few.hip", "qzo_mid.hip", "qzo_expand.hip", "qzo_attention.hip", "qzo_api.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# -ffp-contract=off: the noise recipe is defined operation by operation; fused
# steps are written as explicit fma.  packed-fp32 code generation is disabled.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument"]
# Kernel arguments that the command processor puts into scalar registers before a wavefront starts (scalars and pointers at the
# head of a kernel's list): behind 100 MB of weights the first read of an argument takes 1.2 us.
PRELOAD = ["-mllvm", "-amdgpu-kernarg-preload-count=14"]


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(OBJ, src.replace(".hip", ".o"))
        cmd = [HIPCC] + FLAGS + PRELOAD + ["-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
        if verbose and r.stderr.strip():
            print(r.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs,
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    return LIB


if __name__ == "__main__":
    print(build())
