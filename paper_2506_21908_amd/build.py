"""Build libnct.so (hand-written HIP for gfx950) in-tree with hipcc."""
import os
import shutil
import subprocess
import sys

ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libnct.so")
# (source, defines, object): the kernels are compiled once per precision, side by side
SOURCES = [("nct_kernels.hip", ["-DNCT_FP64_TU=1"], "nct_kernels_f64.o"),
           ("nct_kernels.hip", ["-DNCT_FP64_TU=0"], "nct_kernels_f32.o"),
           ("nct_api.cpp", [], "nct_api.o")]
ARCH = "gfx950"


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def flags():
    return ["-x", "hip", f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wno-unused-result", "-I", os.path.join(HERE, "..", "include")]


def build(verbose: bool = False) -> str:
    """Compile every source to an object (in parallel) and link libnct.so; returns its path."""
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    cc = hipcc()
    procs = []
    objs = []
    for src, defines, name in SOURCES:
        obj = os.path.join(bdir, name)
        objs.append(obj)
        cmd = [cc] + flags() + defines + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((name, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
    failed = []
    for src, p in procs:
        out, _ = p.communicate()
        if p.returncode != 0:
            failed.append((src, out.decode(errors="replace")))
        elif verbose and out:
            print(out.decode(errors="replace"))
    if failed:
        msg = "\n".join(f"--- {s} ---\n{o}" for s, o in failed)
        raise RuntimeError("hipcc failed:\n" + msg)
    tmp = LIB + ".tmp"
    cmd = [cc, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs + [
        "-Wl,-rpath," + os.path.join(ROCM, "lib")]
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    build_c_example()
    return LIB


EXAMPLE_SRC = os.path.join(HERE, "examples", "c_step.c")
EXAMPLE_BIN = os.path.join(HERE, "examples", "c_step")


def build_c_example() -> str:
    """Compile the plain C client (examples/c_step.c) against libnct.so with the host compiler."""
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None:
        raise RuntimeError("no C compiler for the C example")
    cmd = [cc, "-O2", "-std=c99", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(HERE, "..", "include"),
           "-I", os.path.join(ROCM, "include"), EXAMPLE_SRC, "-o", EXAMPLE_BIN, "-L", HERE, "-lnct",
           "-L", os.path.join(ROCM, "lib"), "-lamdhip64", "-lm",
           "-Wl,-rpath,$ORIGIN/..", "-Wl,-rpath," + os.path.join(ROCM, "lib")]
    subprocess.run(cmd, check=True)
    return EXAMPLE_BIN


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
