"""Build the gfx950 shared library ``libftp.so`` in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libftp.so")
SOURCES = ["ftp_nfft.hip", "ftp_solve.hip", "ftp_qr.hip", "ftp_learned.hip", "ftp_aberth.hip", "ftp_mlp.hip", "ftp_train.hip", "ftp_capi.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-munsafe-fp-atomics",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]
# Per-file code generation flags (each file's device code is compiled on its
# own: no kernel calls device code of another file).  The assembly, scoring
# and Aberth kernels are built without machine-level loop-invariant
# code motion, which otherwise keeps constants of their loop bodies in vector
# registers for the whole loop and pushes them past their register budgets
# (measured: assembly, scoring and the Aberth tier faster without it); the
# Newton kernel's short loops gain from the motion and keep it, and so does the
# companion QR, far from its budget (with / without: H = 13 uniform, 65 matrices of
# N = 76, 2.77 / 2.95 ms; N = 16 166 / 169 us; N = 34 and 28 the same; N = 58 24.9 /
# 24.7 ms).
FILE_FLAGS = {
    "ftp_solve.hip": ["-mllvm", "-disable-machine-licm"],
    "ftp_aberth.hip": ["-mllvm", "-disable-machine-licm"],
}


def build(verbose: bool = False, jobs: int = 4) -> str:
    srcs = [os.path.join(CSRC, s) for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    for s in srcs:
        o = os.path.join(objdir, os.path.basename(s) + ".o")
        objs.append(o)
        cmd = [HIPCC] + [f for f in FLAGS if f != "-shared"] + FILE_FLAGS.get(os.path.basename(s), []) + \
            ["-c", s, "-o", o]
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
        if len(procs) >= jobs:
            _wait(procs, verbose)
            procs = []
    _wait(procs, verbose)
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    _run(cmd, verbose)
    os.replace(tmp, LIB)
    return LIB


def _wait(procs, verbose):
    for cmd, p in procs:
        out, _ = p.communicate()
        if verbose or p.returncode:
            sys.stderr.write(" ".join(cmd) + "\n" + out.decode(errors="replace"))
        if p.returncode:
            raise RuntimeError("hipcc failed: " + " ".join(cmd))


def _run(cmd, verbose):
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    if verbose or p.returncode:
        sys.stderr.write(" ".join(cmd) + "\n" + p.stdout.decode(errors="replace"))
    if p.returncode:
        raise RuntimeError("link failed")


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
