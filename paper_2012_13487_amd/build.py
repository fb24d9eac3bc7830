"""Build step for the gfx950 library ``libdgbgk.so`` (C ABI in include/dgbgk.h).

Compiles the HIP kernels, the C-ABI layer and the host set-up code with hipcc
for gfx950 only, into ``libdgbgk.so`` beside this file.
"""
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdgbgk.so")
SOURCES = ["dgbgk_api.hip", "kernels.hip", "kernels32.hip", "rows_64.hip", "rows_32.hip", "rows_ref.hip", "linalg.hip",
           "moments.hip", "init.hip", "host_math.cpp", "server.cpp"]

# Sources whose kernels must not use scratch memory: a build of the row kernels
# that spilled vector registers computed wrong rates, and the occupancy they ask
# for is set just short of that, so another compiler or a small change could
# bring it back unseen.
NO_SCRATCH = ("rows_64.hip", "rows_32.hip", "rows_ref.hip")
RESOURCE_REMARKS = "-Rpass-analysis=kernel-resource-usage"

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared",
    # keep the compiler from forming packed FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def hipcc():
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    path = os.path.join(rocm, "bin", "hipcc")
    return path if os.path.exists(path) else "hipcc"


def scratch_users(remarks):
    """(kernel, scratch bytes per lane, spilled vector registers) of every kernel in the compiler's
    resource remarks that has either; raises if there are no remarks."""
    kernels = re.split(r"remark: +Function Name: ", remarks)[1:]
    if not kernels:
        raise RuntimeError("the compiler gave no kernel resource remarks")
    out = []
    for k in kernels:
        scratch = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", k)
        spills = re.search(r"VGPRs Spill: (\d+)", k)
        if not scratch or not spills:
            raise RuntimeError(f"incomplete kernel resource remark:\n{k}")
        if int(scratch[1]) or int(spills[1]):
            out.append((k.split()[0], int(scratch[1]), int(spills[1])))
    return out


OBJDIR = os.path.join(HERE, "_build")


def compile_sources(sources, csrc, objdir, verbose=False):
    """Compiles the sources to objects in parallel; returns their paths.  Raises
    for a failed compile and for scratch memory in a kernel of NO_SCRATCH."""
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    compile_flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    procs, objs = [], []
    for src in sources:
        obj = os.path.join(objdir, src + ".o")
        checked = src in NO_SCRATCH
        cmd = [hipcc()] + compile_flags + ([RESOURCE_REMARKS] if checked else []) + inc
        cmd += ["-c", "-o", obj, os.path.join(csrc, src)]
        if verbose:
            print(" ".join(cmd), flush=True)
        log = open(obj + ".log", "w+") if checked else None
        procs.append((subprocess.Popen(cmd, stderr=log), cmd, src, log))
        objs.append(obj)
    failed, spilled = [], []
    for p, cmd, src, log in procs:
        rc = p.wait()
        text = ""
        if log:
            log.seek(0)
            text = log.read()
            log.close()
            # (all but the remarks and the source lines quoted below them)
            other = re.sub(r"(?m)^.*\[" + RESOURCE_REMARKS + r"\]\n(?: *\d* \|.*\n)*", "", text).strip()
            if other:
                print(other, file=sys.stderr, flush=True)
        if rc != 0:
            failed.append(cmd)
        elif log:
            spilled += [(src,) + u for u in scratch_users(text)]
    if failed:
        raise subprocess.CalledProcessError(1, failed[0])
    if spilled:
        raise RuntimeError("kernels that must not use scratch memory do (source, kernel, bytes per lane, spilled "
                           "registers): " + "; ".join(map(str, spilled)))
    return objs


def build(verbose: bool = False) -> str:
    """Compiles every source to an object in parallel, then links."""
    os.makedirs(OBJDIR, exist_ok=True)
    objs = compile_sources(SOURCES, CSRC, OBJDIR, verbose)
    tmp = LIB + ".tmp"
    cmd = [hipcc()] + HIPCC_FLAGS + ["-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-q" not in sys.argv))
