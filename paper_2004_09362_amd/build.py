"""Build libar.so (HIP kernels for gfx950 + host plan generator + C ABI).

Run ``python -m paper_2004_09362_amd.build`` or call :func:`build`.  Every
translation unit is compiled in parallel into ``_build/`` and linked into
``libar.so`` next to this file.
"""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libar.so")
SOURCES = [os.path.join(CSRC, f) for f in ["plan.cpp", "capi.cpp", "kernels.hip", "fused_lo.hip", "fused_group.hip",
                                           "fused_free.hip", "fused_small.hip",
                                           "broadcast.hip", "noalloc.hip"]]
HEADERS = [os.path.join(CSRC, f) for f in ("ar_internal.hpp", "device_common.hpp", "fused_col.hpp",
                                               "fused_free.hpp", "free_shape.hpp")] + [
    os.path.join(ROOT, "include", "ar.h")]
# The native part of the Python binding: host code only, against torch's and Python's headers.
BIND_SOURCE = os.path.join(CSRC, "bind.cpp")
BIND_LIB = os.path.join(HERE, "_arbind.so")
OBJDIR = os.path.join(HERE, "_build")
GENDIR = os.path.join(OBJDIR, "gen")

# The column-fused kernels (fused_col.hpp) are instantiated once per P =
# 2..128 -- bandwidth-optimal, shifted and rank-slot launchers, and the int32
# kernel of fused_free.hpp -- in COL_UNITS
# generated units that share the P values round-robin, so that they compile
# in parallel.  Fifteen of them (about 90 s each) and fused_group.hip (about
# 60 s), started first, keep eight cores busy to the end: about 180 s in all,
# where eight column units (160 s) followed by fused_group.hip took 216 s.
COL_UNITS = 15
COL_KINDS = ("bo", "mid", "rot")


def col_unit_text(i: int) -> str:
    """Source of generated unit i: the explicit instantiations for P = 2 + i,
    2 + i + COL_UNITS, ..."""
    lines = ["// Generated by paper_2004_09362_amd/build.py: instantiations of the column-fused",
             "// kernels of fused_col.hpp for every %d-th P starting at %d." % (COL_UNITS, 2 + i),
             '#include "fused_col.hpp"', '#include "fused_free.hpp"', "", "namespace ar {", ""]
    for P in range(2 + i, 129, COL_UNITS):
        for kind in COL_KINDS:
            lines.append("template int launch_fused_%s<%d>(const ColArgs&, int, int, bool, int, void*);" % (kind, P))
        lines.append("template int launch_free_at<%d>(const FreeArgs&, int, int, bool, int, uint32_t, void*);" % P)
    lines += ["", "}  // namespace ar", ""]
    return "\n".join(lines)


def col_units() -> list[str]:
    """Write the generated units (only where their text changed, so that an
    incremental build keeps their objects) and return their paths."""
    os.makedirs(GENDIR, exist_ok=True)
    out = []
    for i in range(COL_UNITS):
        path = os.path.join(GENDIR, "fused_col_u%d.hip" % i)
        text = col_unit_text(i)
        old = None
        if os.path.exists(path):
            with open(path) as fh:
                old = fh.read()
        if old != text:
            with open(path, "w") as fh:
                fh.write(text)
        out.append(path)
    return out

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=" + ARCH,
    # device code objects stored compressed in libar.so (unpacked at load)
    "--offload-compress",
    # packed fp32 instructions stay off in all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-ffp-contract=off", "-fno-fast-math",
    "-Wall", "-Wno-unused-function",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]


def _compile(src: str, incremental: bool = False) -> tuple[str, str]:
    obj = os.path.join(OBJDIR, os.path.basename(src) + ".o")
    if incremental and os.path.exists(obj):
        t = os.path.getmtime(obj)
        if all(os.path.getmtime(f) <= t for f in [src] + HEADERS):
            return obj, ""
    res = subprocess.run([HIPCC] + FLAGS + ["-c", src, "-o", obj], capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s%s" % (src, res.stdout, res.stderr))
    warn = [ln for ln in res.stderr.splitlines() if "packed-fp32-ops" not in ln and ln.strip()]
    return obj, "\n".join(warn)


def _build_bind(incremental: bool = False) -> str:
    """Compile _arbind.so; returns the compiler's warnings."""
    if incremental and os.path.exists(BIND_LIB):
        t = os.path.getmtime(BIND_LIB)
        if all(os.path.getmtime(f) <= t for f in (BIND_SOURCE, os.path.join(ROOT, "include", "ar.h"))):
            return ""
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths

    tmp = BIND_LIB + ".tmp%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-I" + os.path.join(ROOT, "include"), "-I" + sysconfig.get_paths()["include"],
           "-isystem", os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")]
    for p in include_paths():
        cmd += ["-isystem", p]
    cmd += [BIND_SOURCE, "-o", tmp, "-L" + os.path.join(os.path.dirname(torch.__file__), "lib"), "-ltorch_python",
            "-ltorch_cpu", "-lc10"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("compiling %s failed:\n%s%s" % (BIND_SOURCE, res.stdout, res.stderr))
    os.replace(tmp, BIND_LIB)
    return res.stderr


def build(verbose: bool = False, incremental: bool = False) -> str:
    """Compile every source (in parallel) and link libar.so.  Rebuilds every
    unit unless ``incremental`` (then only units older than their sources)."""
    t0 = time.time()
    os.makedirs(OBJDIR, exist_ok=True)
    # the longest units first: the XOR/Ring unit, then the column units, then the rest
    group = [f for f in SOURCES if os.path.basename(f) == "fused_group.hip"]
    units = group + col_units() + [f for f in SOURCES if f not in group]
    workers = max(1, min(len(units), int(os.environ.get("MAX_JOBS", os.cpu_count() or 1))))
    with concurrent.futures.ThreadPoolExecutor(max_workers=workers) as ex:
        bind = ex.submit(_build_bind, incremental)
        results = list(ex.map(lambda src: _compile(src, incremental), units))
        bind_warn = bind.result()
    if verbose:
        for _, warn in results + [("", bind_warn)]:
            if warn:
                sys.stderr.write(warn + "\n")
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=" + ARCH, "-o", tmp] + [o for o, _ in results]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("linking libar.so failed")
    os.replace(tmp, LIB)
    if verbose:
        print("built %s in %.1fs (%d units, %d parallel)" % (LIB, time.time() - t0, len(units), workers))
    return LIB


# Sources of each kernel family (besides the common ones): a profile taken on
# one family stays valid while only another family's sources change.
COMMON = ["capi.cpp", "ar_internal.hpp", "device_common.hpp"]
FAMILIES = {
    "step": ["kernels.hip", "plan.cpp", "noalloc.hip"],
    "lo": ["fused_lo.hip"],
    "col": ["fused_col.hpp"],  # and the generated units (col_unit_text)
    "group": ["fused_group.hip"],
    "free": ["fused_free.hip", "fused_free.hpp", "free_shape.hpp"],
    "small": ["fused_small.hip"],
    "bcast": ["broadcast.hip"],
}


def kernel_families(kernel: str) -> list[str]:
    """Families of a kernel name as bench.py reports it; a split launch
    ("<reducing kernel>+broadcast") has both kernels' families."""
    out = []
    for part in kernel.split("+"):
        for prefix, fam in (("step_kernel", "step"), ("fused_lo_kernel", "lo"), ("fused_bo_kernel", "col"),
                            ("fused_mid_kernel", "col"), ("fused_rot_kernel", "col"), ("fused_xor_kernel", "group"),
                            ("fused_ring_kernel", "group"), ("fused_free_kernel", "free"),
                            ("fused_small_kernel", "small"), ("fused_wide_kernel", "col"),
                            ("fused_xor_wide_kernel", "group"), ("broadcast", "bcast")):
            if part.startswith(prefix):
                out.append(fam)
                break
        else:
            raise ValueError("unknown kernel %r" % kernel)
    return out


def code_text(text: str) -> str:
    """C++ source without comments and with whitespace collapsed: what the
    compiler sees, so that editing a comment does not count as a change."""
    import re

    text = re.sub(r"/\*.*?\*/", " ", text, flags=re.S)
    text = re.sub(r"//[^\n]*", " ", text)
    return " ".join(text.split())


def source_hash(families) -> str:
    """Short hash of the code (comments removed) of one kernel family, or a
    list of families: counter profiles taken on other code are not reported
    as current."""
    import hashlib

    if isinstance(families, str):
        families = [families]
    h = hashlib.sha256()
    for f in COMMON + [f for fam in families for f in FAMILIES[fam]]:
        with open(os.path.join(CSRC, f), encoding="utf-8") as fh:
            h.update(f.encode())
            h.update(code_text(fh.read()).encode())
    if "col" in families:
        # the generated units' code lines as a set: the instantiations count,
        # not how they are dealt out over units
        lines = {code_text(ln) for i in range(COL_UNITS) for ln in col_unit_text(i).splitlines()}
        for ln in sorted(lines - {""}):
            h.update(ln.encode())
    return h.hexdigest()[:16]


def stale() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(BIND_LIB):
        return True
    t = os.path.getmtime(LIB)
    return (any(os.path.getmtime(f) > t for f in SOURCES + HEADERS + [os.path.abspath(__file__)])
            or os.path.getmtime(BIND_SOURCE) > os.path.getmtime(BIND_LIB))


if __name__ == "__main__":
    build(verbose=True, incremental="--incremental" in sys.argv)
