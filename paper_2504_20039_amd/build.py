"""Build libaj.so (hand-written HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import concurrent.futures
import glob
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libaj.so")
OBJDIR = os.path.join(HERE, "_build")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _stale(target, deps):
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def build(force: bool = False, verbose: bool = False, check: bool = False) -> str:
    """Compile every csrc/*.hip to an object and link them into libaj.so.  check: also verify the generated code of the
    hand-scheduled kernels (check_isa.py); raises if a loop holds spills, register-file moves or foreign waits, or if a kernel
    whose tiles use nearly all registers spills any."""
    from . import check_isa
    os.makedirs(OBJDIR, exist_ok=True)
    headers = glob.glob(os.path.join(CSRC, "*.h")) + [os.path.join(HERE, "..", "include", "aj.h")]
    jobs = []
    objs = []
    for src in sources():
        obj = os.path.join(OBJDIR, os.path.basename(src)[:-4] + ".o")
        objs.append(obj)
        if force or _stale(obj, [src] + headers):
            report = ["-Rpass-analysis=kernel-resource-usage"] if check and os.path.basename(src) in check_isa.SPILL_FREE else []
            jobs.append([HIPCC, *FLAGS, *report, "-c", src, "-o", obj])

    def run(cmd):
        r = subprocess.run(cmd, capture_output=True, text=True)
        # the host pass does not know the packed-fp32 feature flag and says so: harmless
        err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed: " + " ".join(cmd) + "\n" + r.stdout + err)
        if verbose and err.strip() and "-Rpass-analysis=kernel-resource-usage" not in cmd:
            print(err)
        return err

    with concurrent.futures.ThreadPoolExecutor(max_workers=4) as ex:
        reports = list(ex.map(run, jobs))
    if force or jobs or _stale(LIB, objs):
        run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    if check:
        check_isa.check_spills("\n".join(reports))
        check_isa.check(HIPCC, FLAGS, verbose)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True, check=True))
