"""Compile the HIP library for gfx950 into paper_2305_18627_amd/libgqsgd.so and the Python binding's argument
marshalling into _marshal.so beside it (in-tree)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libgqsgd.so")
SOURCES = [os.path.join(CSRC, f) for f in ("common.hip", "norm.hip", "quantize.hip", "aggregate.hip", "reduce.hip",
                                           "sparse.hip", "pipeline.hip")]
MARSHAL = os.path.join(HERE, "_marshal.so")
MARSHAL_SOURCE = os.path.join(CSRC, "marshal.cpp")
# for a test: gq_compact with a third of its spans mute (GQ_MUTE_SPANS in sparse.hip); nothing else loads it
MUTE_LIB = os.path.join(HERE, "libgqsgd_mute.so")
MUTE_SOURCES = [os.path.join(CSRC, f) for f in ("common.hip", "sparse.hip")]
HEADERS = [os.path.join(CSRC, "gq_device.hpp"), os.path.join(CSRC, "gq_host.hpp"),
           os.path.join(ROOT, "include", "gqsgd.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
    # the rounding decisions are single IEEE binary32 operations: no implicit fusing, exact division
    "-ffp-contract=off", "-fhip-fp32-correctly-rounded-divide-sqrt", "-fno-fast-math",
    # do not form packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def built_for():
    """The torch and the interpreter whose C++ and C interfaces _marshal.so is compiled against."""
    import platform

    import torch
    return "torch %s, python %s" % (torch.__version__, platform.python_version())


def is_stale():
    if not os.path.exists(LIB) or not os.path.exists(MARSHAL) or not os.path.exists(MUTE_LIB):
        return True
    with open(MARSHAL, "rb") as f:
        if built_for().encode() not in f.read():
            return True
    t = min(os.path.getmtime(f) for f in (LIB, MARSHAL, MUTE_LIB))
    return any(os.path.getmtime(f) > t for f in SOURCES + HEADERS + [MARSHAL_SOURCE])


def _build_marshal(verbose):
    import sysconfig

    import torch
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    tmp = MARSHAL + ".tmp.%d" % os.getpid()
    _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
          "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), '-DGQ_BUILT_FOR="%s"' % built_for(),
          "-I", os.path.join(ROOT, "include"), "-isystem", inc, "-isystem", sysconfig.get_paths()["include"],
          "-o", tmp, MARSHAL_SOURCE, "-L", lib, "-ltorch_python", "-ltorch_cpu", "-lc10"], verbose)
    os.replace(tmp, MARSHAL)


def _build_mute(verbose):
    tmp = MUTE_LIB + ".tmp.%d" % os.getpid()
    _run([HIPCC] + FLAGS + ["-DGQ_MUTE_SPANS=3", "-shared", "-o", tmp] + MUTE_SOURCES, verbose)
    os.replace(tmp, MUTE_LIB)


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # hipcc's host pass does not know the packed-fp32 feature and says so; that is harmless
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("%s failed:\n%s" % (os.path.basename(cmd[0]), out))
    if verbose and out.strip():
        print(out)


def build(force=True, verbose=False):
    """Compile every source (always, unless force=False and the library is newer than its sources),
    the translation units in parallel, then link them into one shared library."""
    if not force and not is_stale():
        return LIB
    from concurrent.futures import ThreadPoolExecutor
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = [os.path.join(objdir, os.path.basename(src)[:-4] + ".%d.o" % os.getpid()) for src in SOURCES]
    try:
        with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 2)) as ex:
            marshal, muted = ex.submit(_build_marshal, verbose), ex.submit(_build_mute, verbose)
            list(ex.map(lambda so: _run([HIPCC] + FLAGS + ["-c", "-o", so[1], so[0]], verbose), zip(SOURCES, objs)))
            marshal.result()
            muted.result()
        tmp = LIB + ".tmp.%d" % os.getpid()
        _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs, verbose)
        os.replace(tmp, LIB)
    finally:
        for o in objs:
            if os.path.exists(o):
                os.remove(o)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
