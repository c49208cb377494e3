"""Builds the HIP library in-tree: paper_2506_17974_amd/liblqsgd.so (gfx950)."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblqsgd.so")
SOURCES = ["lqsgd_plan.cpp", "lqsgd_api.cpp", "lqsgd_kernels.hip"]
KERNEL_PARTS = 6        # the kernel file is compiled in this many parts side by side (LQSGD_PART in the file)


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose: bool = True, extra=(), out: str = LIB) -> str:
    """Compiles every source for gfx950 and links the shared library.  Always
    recompiles (the sources are few)."""
    objs = []
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    common = ["-O3", "-std=c++17", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
              "-Wall", "-Wno-unused-command-line-argument", "-Wno-unused-function"]
    # Packed-fp32 instructions are switched off for device code (they have
    # given wrong results on the test machines); the host pass does not know
    # the feature and says so, which is harmless.
    dev = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
    procs = []
    units = [(s, None) for s in SOURCES if not s.endswith(".hip")]
    units += [(s, k) for s in SOURCES if s.endswith(".hip") for k in range(KERNEL_PARTS)]
    for src, part in units:
        obj = os.path.join(bdir, os.path.splitext(src)[0] + ("" if part is None else "_%d" % part) + ".o")
        objs.append(obj)
        cmd = [hipcc()] + common + (dev + ["-DLQSGD_PART=%d" % part] if part is not None else []) + list(extra) + \
              ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src, p in procs:
        log, _ = p.communicate()
        log = "\n".join(l for l in log.splitlines() if "packed-fp32-ops" not in l)
        if verbose and log.strip():
            print(log)
        if p.returncode != 0:
            raise RuntimeError("compiling %s failed:\n%s" % (src, log))
    cmd = [hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950"] + objs + ["-o", out]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return out


def build_host_sanitize(verbose: bool = True) -> str:
    """The planner and the argument-checking half of the ABI as a host-only program with
    AddressSanitizer and UndefinedBehaviorSanitizer: lqsgd_plan.cpp and lqsgd_api.cpp compiled for
    the CPU, the kernel launchers replaced by stand-ins, csrc/host_check.cpp as its main.  No device
    code is built or sanitized.  Returns the path of the executable; it needs no GPU."""
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    out = os.path.join(bdir, "lqsgd_host_check")
    srcs = [os.path.join(CSRC, f) for f in ("lqsgd_plan.cpp", "lqsgd_api.cpp", "host_check_stubs.cpp", "host_check.cpp")]
    cmd = [hipcc(), "-O1", "-g", "-std=c++17", "-fno-omit-frame-pointer", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=undefined", "-fno-gpu-sanitize", "-Wall", "-Wno-unused-command-line-argument",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC] + srcs + ["-o", out]
    if verbose:
        print(" ".join(cmd), flush=True)
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if p.returncode != 0:
        raise RuntimeError("host sanitizer build failed:\n" + p.stdout)
    return out


if __name__ == "__main__":
    if "--sanitize" in sys.argv[1:]:
        exe = build_host_sanitize()
        # the HIP runtime's own start-up allocations are not this library's: no leak report at exit
        env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")
        sys.exit(subprocess.call([exe], env=env))
    build(extra=sys.argv[1:])
