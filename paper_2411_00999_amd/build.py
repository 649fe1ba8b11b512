"""Build the lnpegn shared library for gfx950 with hipcc (cross-compiles without a GPU), and the CPython extension that
marshals arguments to it with the host compiler.

    python -m paper_2411_00999_amd.build          # rebuild liblnpegn.so in-tree
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblnpegn.so")
MARSHAL_SOURCE = os.path.join(CSRC, "marshal.cpp")
SOURCES = [os.path.join(CSRC, f) for f in ("lnpegn.hip", "lnpegn_rows_inst.hip", "linear_pegn.hip", "embedding_pegn.hip")]
HEADERS = [os.path.join(CSRC, h) for h in ("lnpegn_device.h", "lnpegn_rows.h", "lnpegn_finalize.h", "lnpegn_tracker.h",
                                           "lnpegn_launch.h", "linear_wide.h")]
# translation units: (source, extra defines, object tag).  The row kernels are one source compiled four times.
UNITS = [("lnpegn.hip", [], "abi"),
         ("lnpegn_rows_inst.hip", ["-DLNPEGN_INST_BF16=1", "-DLNPEGN_INST_SAVED=0"], "rows_bf16_recompute"),
         ("lnpegn_rows_inst.hip", ["-DLNPEGN_INST_BF16=1", "-DLNPEGN_INST_SAVED=1"], "rows_bf16_saved"),
         ("lnpegn_rows_inst.hip", ["-DLNPEGN_INST_BF16=0", "-DLNPEGN_INST_SAVED=0"], "rows_f32_recompute"),
         ("lnpegn_rows_inst.hip", ["-DLNPEGN_INST_BF16=0", "-DLNPEGN_INST_SAVED=1"], "rows_f32_saved"),
         ("linear_pegn.hip", [], "linear"),
         ("embedding_pegn.hip", [], "embedding")]
HEADERS.append(os.path.join(os.path.dirname(HERE), "include", "lnpegn.h"))

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # no packed-fp32 instructions: plain scalar fp32 code generation only
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def marshal_path() -> str:
    """Where the extension for the Python and the torch that run this belongs.  It unpacks both's objects by their layout, so
    both are part of its name: another interpreter or another torch over the same tree builds its own."""
    import sysconfig

    import torch
    commit = (torch.version.git_version or "")[:8]
    return os.path.join(HERE, f"_marshal.{sysconfig.get_config_var('SOABI')}.torch-{torch.__version__}.{commit}.so")


def is_stale() -> bool:
    marshal = marshal_path()
    if not os.path.exists(LIB) or not os.path.exists(marshal):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(f) > t for f in SOURCES + HEADERS) or \
        any(os.path.getmtime(f) > os.path.getmtime(marshal) for f in (MARSHAL_SOURCE, HEADERS[-1]))


def _marshal_command(out: str) -> list:
    """g++ on the extension, against the headers of the Python and the torch that run this."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            *("-I" + d for d in (*cpp_extension.include_paths(), sysconfig.get_paths()["include"])),
            MARSHAL_SOURCE, "-o", out, "-L" + lib, "-ltorch_python", "-ltorch_cpu", "-lc10", "-Wl,-rpath," + lib]


def build_marshal(verbose: bool = False) -> str:
    """Compile the extension alone."""
    path = marshal_path()
    tmp = path + f".tmp{os.getpid()}"
    cmd = _marshal_command(tmp)
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, path)
    return path


def build(verbose: bool = False, extra_flags=()) -> str:
    """Compile every HIP source (side by side, one hipcc each) and link liblnpegn.so, and the extension beside them; always
    recompiles."""
    import concurrent.futures as cf
    import shutil
    import tempfile
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmpdir = tempfile.mkdtemp(prefix="lnpegn_build_")
    try:
        def compile_one(unit):
            name, defines, tag = unit
            obj = os.path.join(tmpdir, tag + ".o")
            cmd = [hipcc, *HIPCC_FLAGS, *defines, *extra_flags, "-c", "-o", obj, os.path.join(CSRC, name)]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)
            return obj
        with cf.ThreadPoolExecutor(max_workers=min(len(UNITS) + 1, os.cpu_count() or 4)) as ex:
            marshal = ex.submit(build_marshal, verbose)
            objs = list(ex.map(compile_one, UNITS))
            marshal.result()
        tmp = LIB + f".tmp{os.getpid()}"
        cmd = [hipcc, "--offload-arch=gfx950", "-fPIC", "-shared", "-o", tmp, *objs]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        os.replace(tmp, LIB)
    finally:
        shutil.rmtree(tmpdir, ignore_errors=True)
    return LIB


def ensure_built() -> str:
    """Return the library path, building it and the extension only where they do not exist yet."""
    if not os.path.exists(LIB):
        build()
    elif not os.path.exists(marshal_path()):
        build_marshal()
    return LIB


if __name__ == "__main__":
    build(verbose=True, extra_flags=sys.argv[1:])
    print(LIB)
