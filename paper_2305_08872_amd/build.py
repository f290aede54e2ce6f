"""Builds libamulet.so (HIP, gfx950) in-tree with hipcc, and _marshal, the compiled part of the Python
binding, with the host compiler.  The library needs hipcc alone; where the module cannot be built (no
host compiler, no Python or torch headers) the binding does without it.

One hipcc invocation per translation unit, run in parallel, then one link.
Flags: -O3, fp contraction off (the compared product must be a separately
rounded fp32 multiply), packed-fp32 instruction selection disabled.
"""
from __future__ import annotations

import concurrent.futures
import glob
import importlib.machinery
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
OBJ_DIR = os.path.join(HERE, "_build")
LIB_PATH = os.path.join(HERE, "libamulet.so")
# (named for this Python's ABI: another one does not import it)
MARSHAL_PATH = os.path.join(HERE, "_marshal" + importlib.machinery.EXTENSION_SUFFIXES[0])

SOURCES = ["amulet_api.hip", "mmlike_valu_identity_col.hip"] + [
    "mmlike_valu_%s_%s.hip" % (task, form)
    for task in ("discount", "boost", "count_gt")
    for form in ("col", "row", "const", "elem")
] + ["mmlike_boost_%s.hip" % form for form in ("col", "row", "const", "elem")] + [
    "mmlike_critical_f64_%s.hip" % name for name in ("discount_col", "discount_const", "boost", "count_gt")
] + [
    "mmlike_tile_%s_%s.hip" % (elem, task)
    for elem in ("f64", "f32")
    for task in ("discount", "boost", "count_gt")
] + ["identity_mfma.hip", "identity_mfma_dma.hip", "identity_split.hip", "identity_split_waves.hip", "count_i8.hip", "count_i8_dma.hip", "count_i8_stream.hip", "count_i8_tile.hip", "valu_probe.hip", "mmlike_valu_f64.hip", "identity_mfma_f64.hip", "identity_mfma_f64_dma.hip", "pack.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-I", INCLUDE, "-I", CSRC,
]


def _hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found: cannot build libamulet.so")
    return exe


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc()] + HIPCC_FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    lines = [l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l]
    if res.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s" % (src, "\n".join(lines)))
    if lines:
        sys.stderr.write("\n".join(lines) + "\n")
    return obj


def torch_build() -> str:
    """Which torch this is: the module reads its tensors by the layout of the headers it was compiled with."""
    import torch
    return "%s %s" % (torch.__version__, torch.version.git_version)


def _compile_marshal() -> str:
    """The host-only extension module: this Python's and this torch's headers, no device code."""
    import torch
    root = os.path.dirname(torch.__file__)
    obj = os.path.join(OBJ_DIR, "marshal.o")
    inc = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
           sysconfig.get_paths()["include"]]
    subprocess.check_call([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden",
                           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-DBUILT_FOR_TORCH=\"%s\"" % torch_build(), "-I", INCLUDE]
                          + [x for d in inc for x in ("-isystem", d)]
                          + ["-c", os.path.join(CSRC, "marshal.cpp"), "-o", obj])
    return obj


def _link_marshal(obj: str) -> None:
    # (torch's libraries are in the process before the module is: no path to them is kept in it)
    import torch
    subprocess.check_call([os.environ.get("CXX", "g++"), "-shared", "-o", MARSHAL_PATH, obj, "-L", HERE, "-l:libamulet.so",
                           "-Wl,-rpath,$ORIGIN", "-Wl,--allow-shlib-undefined",
                           "-L", os.path.join(os.path.dirname(torch.__file__), "lib"), "-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10"])


def build(jobs: int = 8) -> str:
    """Compile every HIP source for gfx950 and link libamulet.so, then the binding's module if that can be
    built; returns the library's path."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=jobs) as pool:
        marshal = pool.submit(_compile_marshal)
        objs = list(pool.map(_compile, SOURCES))
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH] + objs
    subprocess.check_call(cmd)
    for old in glob.glob(os.path.join(os.path.dirname(MARSHAL_PATH), "_marshal*.so")):
        os.remove(old)
    try:
        _link_marshal(marshal.result())
    except (ImportError, OSError, AttributeError, subprocess.CalledProcessError) as e:
        sys.stderr.write("the binding's compiled module was not built (%s: %s): calls cost some 3 us more on the host\n" % (type(e).__name__, e))
    return LIB_PATH


if __name__ == "__main__":
    print(build())
