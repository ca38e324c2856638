"""The library's host code over a CPU stand-in of the HIP runtime
(hip_standin.cpp): `load()` builds both into one shared library and returns
the Python binding on it, with the stand-in's controls beside it."""
import ctypes
import fcntl
import importlib.util
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
OUT = os.path.join(ROOT, "_build", "standin")
CSRC = os.path.join(ROOT, "paper_2106_06601_amd", "csrc")


def _by_path(name, path):
    spec = importlib.util.spec_from_file_location(name, path)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def build() -> str:
    """Host passes only (no device code)."""
    os.makedirs(OUT, exist_ok=True)
    with open(os.path.join(OUT, "lock"), "w") as lock:  # parallel test workers build in turn
        fcntl.flock(lock, fcntl.LOCK_EX)
        return _build()


def _build() -> str:
    b = _by_path("costa_build", os.path.join(ROOT, "paper_2106_06601_amd", "build.py"))
    # (the stand-in first: the library's objects register their kernels with it as they are loaded)
    sources = [os.path.join(HERE, "hip_standin.cpp")] + [os.path.join(CSRC, s) for s in b.SOURCES]
    objs = [os.path.join(OUT, os.path.basename(s) + ".o") for s in sources]
    flags = ["-O1" if f == "-O3" else f for f in b.COMMON]
    jobs = [[b.HIPCC, f"--offload-arch={b.ARCH}", *flags, "-x", "hip", "--cuda-host-only", "-c", s, "-o", o]
            for s, o in zip(sources, objs)]
    with ThreadPoolExecutor(max_workers=len(jobs)) as ex:
        list(ex.map(b._run, jobs))
    undefined = subprocess.run(["nm", "-u", *objs], stdout=subprocess.PIPE, text=True, check=True).stdout
    fatbins = sorted(set(re.findall(r"__hip_fatbin\w*", undefined)))  # the device code that is not there
    lib = os.path.join(OUT, "libcosta_standin.so")
    b._run(["g++", "-shared", "-Wl,-Bsymbolic", "-Wl,--no-undefined", "-o", lib + ".tmp", *objs,
            *[f"-Wl,--defsym,{s}=0" for s in fatbins], "-lpthread"])
    os.replace(lib + ".tmp", lib)
    return lib


class Standin:
    """The binding `C` and the stand-in's streams, graphs and memory."""

    def __init__(self, lib):
        old = os.environ.get("COSTA_LIB")
        os.environ["COSTA_LIB"] = lib
        try:
            name = "paper_2106_06601_amd_standin"
            spec = importlib.util.spec_from_file_location(
                name, os.path.join(ROOT, "paper_2106_06601_amd", "__init__.py"))
            self.C = sys.modules[name] = importlib.util.module_from_spec(spec)
            spec.loader.exec_module(self.C)
        finally:
            if old is None:
                del os.environ["COSTA_LIB"]
            else:
                os.environ["COSTA_LIB"] = old
        self.lib = ctypes.CDLL(lib)
        vp = ctypes.c_void_p
        for f, res, args in (("stream", vp, []), ("capture", None, [vp]), ("end_capture", vp, [vp]),
                             ("replay", None, [vp, vp]), ("nodes", ctypes.c_int, [vp]),
                             ("destroy_graph", None, [vp]), ("run", None, [vp]),
                             ("buffer", None, [vp, ctypes.c_size_t]),
                             ("refuse_implicit", None, [ctypes.c_int]),
                             ("lane_volume", ctypes.c_int64, [ctypes.c_int32] * 3),
                             ("divmod", None, [ctypes.c_int, vp, vp, vp, vp, ctypes.c_int64]),
                             ("xcd_order", None, [ctypes.c_int32, ctypes.c_int32, vp]),
                             ("tile_walk", None, [ctypes.c_int32] * 3 + [ctypes.c_int64] + [ctypes.c_int32] * 3 +
                              [vp, vp]), ("faults", ctypes.c_char_p, [])):
            fn = getattr(self.lib, "standin_" + f)
            fn.restype, fn.argtypes = res, args
            setattr(self, f, fn)

    def array(self, n, start=0.0):
        """n doubles of device memory: start, start + 1, ..."""
        a = np.arange(n, dtype=np.float64) + start
        self.buffer(a.ctypes.data, a.nbytes)
        return a

    def check(self):
        text = self.faults().decode()
        assert not text, text


_loaded = None


def load() -> Standin:
    global _loaded
    if _loaded is None:
        _loaded = Standin(build())
    return _loaded
