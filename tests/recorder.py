"""A host-only build of the library whose kernel launches are written down
instead of made (tests/recorder.cpp): what a call launches, seen without a GPU."""
import ctypes
import os
import re
import subprocess
from collections import namedtuple

import pytest

from paper_2506_15745_amd import build, ipv

HERE = os.path.dirname(os.path.abspath(__file__))
BASE = 1 << 40  # device addresses that nothing reads: every buffer gets a range of its own

Launch = namedtuple("Launch", "kernel grid_x grid_y threads lds")


class Recorder:
    def __init__(self, path, monkeypatch):
        monkeypatch.setattr(ipv, "_lib", None)
        monkeypatch.setattr(ipv, "LIB_PATH", path)
        self.lib = ipv.lib()
        self.lib.rec_count.restype = ctypes.c_long
        self.lib.rec_launch.restype = ctypes.c_char_p
        self.lib.rec_launch.argtypes = [ctypes.c_long, ctypes.POINTER(ctypes.c_uint * 4)]
        self.lib.rec_reset.argtypes = [ctypes.c_long]

    def start(self, fail=-1):
        self.lib.rec_reset(fail)

    def launches(self):
        out = []
        for i in range(self.lib.rec_count()):
            dims = (ctypes.c_uint * 4)()
            name = self.lib.rec_launch(i, ctypes.byref(dims)).decode()
            # mangled: the namespace, the name's length, the name
            length, kernel = re.search(r"(\d\d?)(k_\w+)", name.replace("12_GLOBAL__N_1", "")).groups()
            out.append(Launch(kernel[:int(length)], *dims))
        return out

    def kernels(self):
        return [x.kernel for x in self.launches()]


@pytest.fixture(scope="session")
def recorder_library(tmp_path_factory):
    folder = tmp_path_factory.mktemp("recorder")
    path, api, rec = (str(folder / f) for f in ("libipv_recorder.so", "api.o", "recorder.o"))
    include = os.path.join(os.path.dirname(os.path.dirname(build.HIPCC)), "include")
    subprocess.run([build.HIPCC, "--offload-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC",
                    "-fuse-cuid=none", "-c", *build.SOURCES, "-o", api], check=True)
    subprocess.run(["g++", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I" + include, "-c",
                    os.path.join(HERE, "recorder.cpp"), "-o", rec], check=True)
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", api, rec, "-o", path], check=True)
    return path


@pytest.fixture
def recorder(recorder_library, monkeypatch):
    return Recorder(recorder_library, monkeypatch)


class Stream:
    """ipv_ckv_stream on buffers at made-up addresses."""

    def __init__(self, L, H, D, grid, cap, budget, r, entry, rows=None, dtype=ipv.BF16, capacity=None):
        gh, gw = grid
        self.rows = rows or gh * gw
        self.shape = ipv.Shape(len(entry), L, H, D, capacity or cap + self.rows, gh, gw, dtype)
        self.cap, self.budget, self.r, self.entry = cap, budget, r, entry
        self.at = {k: BASE * (i + 1) for i, k in enumerate("K V fr pa fK fV tar van keep ws".split())}

    def call(self, frames, mode=0, tau=None, n=None):
        """(status, counts after, passes)"""
        i32 = ctypes.c_int32 * len(self.entry)
        n, passes = i32(*(n or self.entry)), i32(*[-7] * len(self.entry))
        t = None if tau is None else (ctypes.c_double * 3)(*tau)
        a = self.at
        rc = ipv.lib().ipv_ckv_stream(
            ctypes.byref(self.shape), a["K"], a["V"], a["fr"], a["pa"], n, a["fK"], a["fV"], frames, self.rows, 0, self.cap,
            self.budget, 0.5, self.r, mode, None if t is None else ctypes.addressof(t), a["tar"], a["van"], a["keep"],
            a["ws"], ipv.workspace_bytes(self.shape), passes, None)
        return rc, list(n), list(passes)
