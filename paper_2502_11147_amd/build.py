"""Compiles the HIP sources of the decode path into ``libraas.so`` (gfx950)."""
from __future__ import annotations

import hashlib
import os
import shutil
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB_PATH = os.path.join(HERE, "libraas.so")
KERNELS = os.path.join(CSRC, "raas_kernels.hip")
# translation units of libraas.so: the kernels' file once per RAAS_PART, and the runtime
KERNEL_PARTS = 15
UNITS = [(KERNELS, ["-DRAAS_PART=%d" % i]) for i in range(KERNEL_PARTS)] + [(os.path.join(CSRC, "raas_runtime.hip"), [])]
# the streaming probe (measurement only) is a library of its own
PROBE_SOURCES = [os.path.join(CSRC, "raas_probe.hip")]
PROBE_LIB_PATH = os.path.join(HERE, "libraas_probe.so")
ARCH = "gfx950"


def hipcc_command(out: str, sources, *more: str) -> list[str]:
    return [
        "hipcc", "--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", *more,
        # packed fp32 vector instructions stay off on this target
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-I", INCLUDE, "-I", CSRC, *sources, "-o", out,
    ]


def _code_text(src: str) -> str:
    """C++ source without its comments and with whitespace runs collapsed
    (the kernels' sources hold no comment markers inside literals)."""
    out, i, n = [], 0, len(src)
    while i < n:
        if src.startswith("//", i):
            j = src.find("\n", i)
            i = n if j < 0 else j
        elif src.startswith("/*", i):
            j = src.find("*/", i + 2)
            i = n if j < 0 else j + 2
            out.append(" ")
        else:
            out.append(src[i])
            i += 1
    return " ".join("".join(out).split())


def kernel_digest() -> str:
    """sha256 over the kernel sources' code (comments and layout left out)
    and the compile flags: identifies the kernels that a stored
    hardware-counter measurement was taken on."""
    h = hashlib.sha256()
    for p in (KERNELS, os.path.join(CSRC, "raas_internal.h")):
        with open(p, encoding="utf-8") as f:
            h.update(_code_text(f.read()).encode())
    h.update(" ".join(a for a in hipcc_command("lib", (), "-shared") if not os.path.isabs(a) and a not in ("-I", "-o", "lib")).encode())
    return h.hexdigest()


def _hipcc(cmd: list[str], verbose: bool):
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
    if verbose:
        print(" ".join(cmd))


def build(verbose: bool = False) -> str:
    """Builds libraas.so (the decode path) and libraas_probe.so (the
    streaming probe of the measurements)."""
    with tempfile.TemporaryDirectory(prefix="raas_build_") as tmp:
        objects = [os.path.join(tmp, "unit%d.o" % i) for i in range(len(UNITS))]
        lib, probe = os.path.join(tmp, "libraas.so"), os.path.join(tmp, "libraas_probe.so")
        compiles = [hipcc_command(o, [src], "-c", *flags) for o, (src, flags) in zip(objects, UNITS)]
        compiles.append(hipcc_command(probe, PROBE_SOURCES, "-shared"))
        with ThreadPoolExecutor(max(1, min(8, os.cpu_count() or 1))) as pool:
            list(pool.map(lambda c: _hipcc(c, verbose), compiles))
        _hipcc(hipcc_command(lib, objects, "-shared"), verbose)
        for src, dst in ((lib, LIB_PATH), (probe, PROBE_LIB_PATH)):
            part = dst + ".tmp%d" % os.getpid()
            shutil.copyfile(src, part)
            os.replace(part, dst)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
