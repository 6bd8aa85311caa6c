"""Build the HIP library libmf.so for gfx950: generate the amplitude headers,
compile each kernel instance in parallel and check its assembly, link in-tree."""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

from . import check_asm

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmf.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-I", CSRC,
         # no packed FP32 instructions anywhere in the device code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def compile_one(src: str, extra=()) -> str:
    name = os.path.basename(src)[:-4]
    obj = os.path.join(OBJ, name + ".o")
    cmd = [HIPCC, *FLAGS, *extra, "-save-temps=obj", "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr[-4000:]}")
    # of the intermediate files only the device assembly is kept
    asm = os.path.join(OBJ, name + "-hip-amdgcn-amd-amdhsa-gfx950.s")
    for f in os.listdir(OBJ):
        path = os.path.join(OBJ, f)
        if path != asm and f.startswith((name + "-hip-", name + "-host-", name + ".hip-")):
            os.remove(path)
    with open(asm) as f:
        found = check_asm.join_copies(f.read())
    if found:
        raise RuntimeError(f"{src}: registers are copied ahead of the execution mask's restore:\n"
                           + "\n".join(f"  {fn} {label}: {'; '.join(code[:4])}" for fn, label, code in found))
    return obj


def build(jobs: int | None = None, extra=()) -> str:
    sys.path.insert(0, os.path.join(HERE, "gen"))
    import gen_me  # noqa: E402

    gen_me.main(os.path.join(CSRC, "gen"))
    os.makedirs(OBJ, exist_ok=True)
    srcs = sources()
    jobs = jobs or min(len(srcs), os.cpu_count() or 4)
    with cf.ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(lambda s: compile_one(s, extra), srcs))
    tmp = LIB + ".tmp"
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":  # python -m paper_2105_10529_amd.build_lib
    extra = sys.argv[1:]
    print(build(extra=extra))
