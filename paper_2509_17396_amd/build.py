"""Build libepicache.so (gfx950) in-tree with hipcc.  `python -m paper_2509_17396_amd.build`."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "lib", "libepicache.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden",
    # packed-fp32 VALU forms are kept out of all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
]


def build(verbose: bool = False) -> str:
    srcs = sorted(glob.glob(os.path.join(PKG, "csrc", "*.hip")))
    os.makedirs(os.path.dirname(LIB), exist_ok=True)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    base = [hipcc, *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc")]
    with tempfile.TemporaryDirectory() as objdir:  # one compiler per source, the long ones side by side
        objs = [os.path.join(objdir, os.path.basename(src) + ".o") for src in srcs]
        jobs = [subprocess.Popen([*(f for f in base if f != "-shared"), "-c", "-o", obj, src], stdout=subprocess.PIPE,
                                 stderr=subprocess.STDOUT, text=True) for src, obj in zip(srcs, objs)]
        out = [job.communicate()[0] for job in jobs]
        code = max(abs(job.returncode) for job in jobs)
        if code == 0:
            link = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs],
                                  capture_output=True, text=True)
            out.append(link.stdout + link.stderr)
            code = link.returncode
    noise = "is not a recognized feature for this target"  # host pass, harmless
    log = "\n".join(l for l in "".join(out).splitlines() if noise not in l)
    if code != 0:
        raise RuntimeError("hipcc failed:\n" + log)
    if verbose and log.strip():
        print(log, file=sys.stderr)
    return LIB


def build_selftests(verbose: bool = False):
    """Compile the shared objects under csrc/selftest: internal launchers with arguments that the library fixes, for the
    tests (not part of the library)."""
    outdir = os.path.join(PKG, "lib", "selftest")
    os.makedirs(outdir, exist_ok=True)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    built = []
    for src in sorted(glob.glob(os.path.join(PKG, "csrc", "selftest", "*.hip"))):
        so = os.path.join(outdir, "lib" + os.path.splitext(os.path.basename(src))[0] + ".so")
        cmd = [hipcc, *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"), "-o", so, src]
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
        built.append(so)
    return built


def build_microbench(verbose: bool = False):
    """Compile the stand-alone microbenchmarks under csrc/microbench (not part of the library)."""
    outdir = os.path.join(PKG, "lib", "microbench")
    os.makedirs(outdir, exist_ok=True)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    built = []
    for src in sorted(glob.glob(os.path.join(PKG, "csrc", "microbench", "*.hip"))):
        exe = os.path.join(outdir, os.path.splitext(os.path.basename(src))[0])
        cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-w", "-Xclang", "-target-feature", "-Xclang",
               "-packed-fp32-ops", "-o", exe, src]
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
        built.append(exe)
    return built


if __name__ == "__main__":
    print(build(verbose=True))
    print("\n".join(build_selftests(verbose=True)))
    print("\n".join(build_microbench(verbose=True)))
