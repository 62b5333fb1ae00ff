"""Build the HIP library (gfx950 only) in-tree: paper_2009_13062_amd/libnetfuse.so.

Each .hip translation unit is compiled by its own hipcc process (they run side by side), then
the objects are linked into one shared library with a plain C ABI (include/netfuse.h)."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libnetfuse.so")
BINDING = os.path.join(HERE, "_binding.so")
SOURCES = ["netfuse_api.hip", "graph_merge.cpp", "gemm_inst_b8.hip", "gemm_inst_b2.hip", "gemm_inst_b24.hip", "gemm_inst_b22.hip", "gemm_inst_b21.hip", "gemm_inst_b27.hip", "gemm_inst_b1.hip",
           "gemm_inst_b0.hip", "gemm_inst_dma.hip", "gemm_inst_stream.hip", "gemm_inst_frag.hip", "gemm_inst_f32.hip", "gemm_inst_split.hip", "gemm_inst_ring.hip", "conv_patch_inst.hip", "conv_tap_inst.hip", "conv_wave_inst.hip", "conv_plane_inst.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 VALU forms are not to be generated on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-value",
]


def _hipcc() -> str:
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _newest_header() -> float:
    t = os.path.getmtime(os.path.join(HERE, "..", "include", "netfuse.h"))
    for f in os.listdir(CSRC):
        if f.endswith(".h"):
            t = max(t, os.path.getmtime(os.path.join(CSRC, f)))
    return t


def _compile(src: str, extra, verbose: bool, force: bool) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    path = os.path.join(CSRC, src)
    if not force and os.path.exists(obj) and os.path.getmtime(obj) > max(os.path.getmtime(path), _newest_header()):
        return obj
    cmd = [_hipcc()] + HIPCC_FLAGS + list(extra) + ["-c", path, "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops' is not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, out))
    if verbose and out.strip():
        print(out, flush=True)
    return obj


def binding_target() -> str:
    """The Python and torch that a binding built now is for: their inlined accessors and struct layouts are compiled in."""
    import torch
    return "python %d.%d, torch %s %s" % (sys.version_info[0], sys.version_info[1], torch.__version__, torch.version.git_version)


def _built_for(target: str) -> bool:
    with open(BINDING, "rb") as f:
        return target.encode() + b"\0" in f.read()


def _build_binding(verbose: bool, force: bool) -> None:
    """The call marshalling of the Python package (csrc/binding.cpp): a host-only extension against the installed torch.  The package runs
    without it, so a box without a host compiler or these headers gets a warning; code that does not compile is an error."""
    import shutil
    import sysconfig
    import warnings

    import torch
    src = os.path.join(CSRC, "binding.cpp")
    target = binding_target()
    if not force and os.path.exists(BINDING) and os.path.getmtime(BINDING) > max(os.path.getmtime(src), _newest_header()) and _built_for(target):
        return
    root = os.path.dirname(torch.__file__)                   # its libraries are found by name: the package imports torch first
    headers = [os.path.join(sysconfig.get_paths()["include"], "Python.h"), os.path.join(root, "include", "ATen", "ATen.h")]
    missing = ["g++"] * (shutil.which("g++") is None) + [h for h in headers if not os.path.exists(h)]
    if missing:
        warnings.warn("calls are marshalled in Python: csrc/binding.cpp is not built without " + ", ".join(missing))
        if os.path.exists(BINDING):
            os.remove(BINDING)                               # of other sources, or of another torch
        return
    # NDEBUG: without it a header keeps a thread-local counter.  A library with thread-local storage that is loaded late and whose storage is
    # never touched leaves glibc 2.35 on the slow path of every other library's (17 % on torch's small operators).
    cmd = ["g++", "-O2", "-DNDEBUG", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, '-DNETFUSE_BUILT_FOR="%s"' % target,
           "-isystem", os.path.join(root, "include"),
           "-isystem", sysconfig.get_paths()["include"], src, "-o", BINDING + ".tmp",
           "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(BINDING + ".tmp", BINDING)


def build(verbose: bool = False, extra=(), force: bool = True, jobs: int = 8) -> str:
    """Compile every translation unit (always, unless force=False and objects are newer) and link."""
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        binding = ex.submit(_build_binding, verbose, force)
        objs = list(ex.map(lambda s: _compile(s, extra, verbose, force), SOURCES))
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", LIB + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(LIB + ".tmp", LIB)
    binding.result()                                         # the library is there whatever became of it
    return LIB


if __name__ == "__main__":
    args = sys.argv[1:]
    force = "--incremental" not in args
    args = [a for a in args if a != "--incremental"]
    print(build(verbose=True, extra=args, force=force))
