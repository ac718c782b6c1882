"""Compile the HIP library for gfx950 into paper_2401_10187_amd/libkronmatmul.so (in-tree), and the binding's native part for
this Python and torch into paper_2401_10187_amd/_marshal.<this Python's suffix>.so.  The library is needed; without the native part
the binding marshals by ctypes.

The kernel instances are spread over one translation unit per kernel family (csrc/inst_*.hip) so that
they compile side by side; csrc/kronmatmul.hip holds the C-ABI, the planner and the two kernels
without compile-time shapes."""
import glob
import importlib.util
import os
import re
import subprocess
import sysconfig
import time
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libkronmatmul.so")
MARSHAL = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))
MARSHAL_SOURCE = os.path.join(CSRC, "marshal.cpp")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep hipcc from forming packed-fp32 instructions out of ordinary float code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    t0 = time.time()
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if verbose:
        print("%.0f s: %s" % (time.time() - t0, os.path.basename(cmd[-1])), flush=True)
    out = "\n".join(l for l in proc.stdout.splitlines() if "packed-fp32-ops" not in l)
    if proc.returncode != 0:
        raise RuntimeError("%s failed:\n%s" % (os.path.basename(cmd[0]), out))
    if verbose and out.strip():
        print(out, flush=True)


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _stale(obj):
    """True unless `obj` is newer than every file its dependency list (written by -MD) names."""
    dep = obj[:-2] + ".d"
    if not (os.path.exists(obj) and os.path.exists(dep)):
        return True
    names = open(dep).read().replace("\\\n", " ").split(":", 1)[1].split()
    t = os.path.getmtime(obj)
    return any(not os.path.exists(n) or os.path.getmtime(n) > t for n in names)


def _torch_version(torch_dir):
    """torch.__version__, without the import."""
    return re.search(r"^__version__ = '(.*)'", open(os.path.join(torch_dir, "version.py")).read(), re.M).group(1)


def _marshal_stale():
    """True unless the native part is newer than its source and built for the torch at hand (whose version is kept beside the objects)."""
    try:
        torch_dir = os.path.dirname(importlib.util.find_spec("torch").origin)
        return (os.path.getmtime(MARSHAL) < os.path.getmtime(MARSHAL_SOURCE) or
                open(os.path.join(OBJ, "marshal.torch")).read() != _torch_version(torch_dir))
    except (OSError, AttributeError):
        return True


def build_marshal(verbose=False):
    """Host code only: the headers of Python and torch, linked against the torch libraries that `import torch` loads.  Returns
    whether that worked: a machine without a C++ compiler or these headers has the library all the same."""
    for old in {MARSHAL, os.path.join(HERE, "_marshal.so")}:       # (nothing older is left to be loaded in its place)
        if os.path.exists(old):
            os.remove(old)
    try:
        torch_dir = os.path.dirname(importlib.util.find_spec("torch").origin)
        version = _torch_version(torch_dir)
        _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I" + sysconfig.get_paths()["include"],
              "-isystem", os.path.join(torch_dir, "include"), "-isystem", os.path.join(torch_dir, "include/torch/csrc/api/include"),
              '-DKM_BUILT_FOR="%s"' % version,
              "-o", MARSHAL, MARSHAL_SOURCE, "-L" + os.path.join(torch_dir, "lib"), "-lc10", "-ltorch_cpu",
              "-ltorch_python"], verbose)
        with open(os.path.join(OBJ, "marshal.torch"), "w") as f:
            f.write(version)
    except (OSError, AttributeError, RuntimeError) as e:
        print("the binding's native part was not built, calls are marshalled by ctypes: %s" % e, flush=True)
        return False
    return True


def build(verbose=False, jobs=None, incremental=False):
    """Recompiles every translation unit (with incremental=True only those whose sources changed, a
    convenience while working on one kernel); returns the path of the shared library."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)
    srcs = sources()
    objs = [os.path.join(OBJ, os.path.basename(s)[:-4] + ".o") for s in srcs]
    todo = [(s, o) for s, o in zip(srcs, objs) if not incremental or _stale(o)]
    jobs = jobs or min(max(len(todo), 1), os.cpu_count() or 1, 16)
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        marshal = None
        if not incremental or _marshal_stale():
            marshal = pool.submit(build_marshal, verbose)
        list(pool.map(lambda so: _run([hipcc] + HIPCC_FLAGS + ["-MD", "-MF", so[1][:-2] + ".d", "-c", "-o", so[1], so[0]],
                                      verbose), todo))
        if marshal:
            marshal.result()
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs, verbose)
    return LIB


if __name__ == "__main__":
    import sys
    print(build(verbose=True, incremental="--incremental" in sys.argv[1:]))
