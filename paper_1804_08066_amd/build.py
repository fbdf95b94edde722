"""Build libmqgrad.so (gfx950 kernels + C ABI + host MDP) in-tree with hipcc, _marshal.<key>.so (the
Python binding's argument tables) and libmqgrad_bench.so
(the streaming kernels that bench.py uses as its measured ceilings; not part of the library)."""
import os
import shutil
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmqgrad.so")
BENCH_LIB = os.path.join(HERE, "libmqgrad_bench.so")
SOURCES = ["api.hip", "quantize_pack.hip", "quantize_wave.hip", "aggregate_update.hip", "minmax.hip", "requantize_cells.hip", "mdp.cpp"]
BENCH_SOURCES = ["bench_stream.hip"]
MARSHAL_SOURCE = "marshal.cpp"   # the binding's argument tables: host code against torch and Python

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# -ffp-contract=off: the kernels' only fused operations are their explicit fma calls, so that the
# fp32 results are reproducible to the bit.  Packed-fp32 instruction selection is switched off.
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off", "-fno-fast-math", "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-fno-gpu-flush-denormals-to-zero",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wextra", "-Wno-unused-parameter",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def needs_build():
    """True when a library is missing or older than any of its sources or headers, or there is no binding module of
    the present sources, Python and torch."""
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".h", ".hip", ".cpp"))] + \
        [os.path.join(ROOT, "include", "mqgrad.h")]
    if not os.path.exists(marshal_path()):
        return True
    for lib in (LIB, BENCH_LIB):
        if not os.path.exists(lib):
            return True
        t = os.path.getmtime(lib)
        if any(os.path.getmtime(d) > t for d in deps):
            return True
    return False


def _link(names, out, tmpdir, verbose, extra_flags):
    def compile_one(name):
        obj = os.path.join(tmpdir, name + ".o")
        cmd = [HIPCC, *FLAGS, *extra_flags, "-c", os.path.join(CSRC, name), "-o", obj]
        if verbose:
            print(" ".join(cmd))
        subprocess.check_call(cmd)
        return obj

    with ThreadPoolExecutor(max_workers=min(6, len(names))) as pool:
        objs = list(pool.map(compile_one, names))
    tmp = out + ".tmp.%d" % os.getpid()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,--no-undefined", *objs, "-o", tmp])
    os.replace(tmp, out)


def marshal_path():
    """The binding's module, named by what it was compiled from and against: its sources (the layout of the item structs
    among them), the Python it is loaded into and the torch whose classes it has inlined."""
    import hashlib
    import sysconfig
    import torch
    key = hashlib.sha256()
    for path in (os.path.join(CSRC, MARSHAL_SOURCE), os.path.join(ROOT, "include", "mqgrad.h")):
        with open(path, "rb") as f:
            key.update(f.read())
    key.update(repr((sysconfig.get_config_var("EXT_SUFFIX"), torch.__version__, torch.version.git_version,
                     torch.compiled_with_cxx11_abi())).encode())
    return os.path.join(HERE, "_marshal.%s.so" % key.hexdigest()[:16])


def _build_marshal(verbose):
    import sysconfig
    import torch
    at = os.path.dirname(torch.__file__)
    inc = [os.path.join(at, "include"), os.path.join(at, "include", "torch", "csrc", "api", "include"), sysconfig.get_paths()["include"]]
    out = marshal_path()
    tmp = out + ".tmp.%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch.compiled_with_cxx11_abi()), "-I", os.path.join(ROOT, "include"),
           *[x for d in inc for x in ("-isystem", d)], os.path.join(CSRC, MARSHAL_SOURCE),
           "-L", os.path.join(at, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-o", tmp]
    if verbose:
        print(" ".join(cmd))
    subprocess.check_call(cmd)
    os.replace(tmp, out)


def load_marshal():
    """The binding's module (built first only if there is none of the present sources, Python and torch), or None, with a
    warning, where it can be neither built nor loaded: the binding then makes its tables itself."""
    import importlib.machinery
    import importlib.util
    try:
        if not os.path.exists(marshal_path()):
            _build_marshal(False)
        loader = importlib.machinery.ExtensionFileLoader("_marshal", marshal_path())
        module = importlib.util.module_from_spec(importlib.util.spec_from_loader("_marshal", loader))
        loader.exec_module(module)
        return module
    except (OSError, ImportError, subprocess.CalledProcessError) as e:
        import warnings
        warnings.warn("the binding's native argument tables are not available (%s): each call takes longer" % e)
        return None


def build_libraries(verbose=False, extra_flags=()):
    """Compile the libraries' sources (one hipcc process per file, in parallel) and link them."""
    tmpdir = tempfile.mkdtemp(prefix="mqgrad_build_")
    try:
        _link(SOURCES, LIB, tmpdir, verbose, extra_flags)
        _link(BENCH_SOURCES, BENCH_LIB, tmpdir, verbose, extra_flags)
    finally:
        shutil.rmtree(tmpdir, ignore_errors=True)
    return LIB


def build(verbose=False, extra_flags=()):
    """Build everything: the libraries and the binding's module."""
    with ThreadPoolExecutor(max_workers=1) as pool:
        marshal = pool.submit(_build_marshal, verbose)
        build_libraries(verbose, extra_flags)
        marshal.result()
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
