"""The library's host side (api.cpp) on a CPU: compiled against the stand-in of
host_runtime.cpp for the HIP runtime and the kernels."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2102_01305_amd import _lib as L
from paper_2102_01305_amd.solver import make_config, make_wings

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2102_01305_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
PER_THREAD = 2                        # hipStreamPerThread


def build(folder):
    """Compile and load the library's host side; skips where that cannot be done."""
    cxx = shutil.which("g++")
    if cxx is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("no g++ or no HIP headers")
    so = os.path.join(str(folder), "libhostside.so")
    # -Bsymbolic: its calls stay with the stand-in, whatever runtime the process has mapped
    subprocess.run([cxx, "-O1", "-std=c++17", "-fPIC", "-shared", "-pthread", "-Wl,-Bsymbolic",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"),
                    "-I", CSRC, os.path.join(CSRC, "api.cpp"), os.path.join(ROOT, "tests", "host_runtime.cpp"),
                    "-o", so], check=True)
    lib = C.CDLL(so)
    for name, res, args in L.SIGNATURES:
        fn = getattr(lib, name)
        fn.restype, fn.argtypes = res, args
    lib.host_stream.restype = C.c_void_p
    lib.host_pinned.restype = C.c_longlong
    lib.host_calls.restype = C.c_char_p
    return lib


class Solve:
    """A handle on a workspace in host memory."""

    def __init__(self, lib, bx, wings=(), stream=None, **config):
        self.lib, self.h = lib, L.Handle()
        cfg, arr = make_config(bx, **config), make_wings(list(wings))
        n = lib.ibmlbm_workspace_bytes(C.byref(cfg), len(wings), arr)
        assert n, lib.ibmlbm_last_error(None)
        self.shape = (cfg.nz, cfg.ny, cfg.nx)
        self.ws = np.empty(n + 256, np.uint8)          # (touched only where a call writes)
        at = (self.ws.ctypes.data + 255) // 256 * 256
        self.check(lib.ibmlbm_create(C.byref(cfg), C.c_void_p(at), n, C.c_void_p(stream), C.byref(self.h)))
        self.state = [np.frombuffer((C.c_char * 8).from_address(at + k * self._state_bytes(cfg)), np.int64) for k in (0, 1)]
        if wings:
            self.check(lib.ibmlbm_set_kinematics(self.h, len(wings), arr))

    @staticmethod
    def _state_bytes(cfg):
        size = 4 if cfg.storage == L.FP32 else 2
        line = 128 // size
        px = -(-(cfg.nx + 2) // line) * line
        slabs = -(-((cfg.ny * cfg.nz + 1) * 19 * px * size) // 256) * 256
        return -(-(slabs + 64 * cfg.ny * cfg.nz) // 256) * 256

    def check(self, rc):
        assert rc == L.OK, self.lib.ibmlbm_last_error(self.h)

    def init(self, fdist=None, step0=0):
        p = None if fdist is None else fdist.ctypes.data_as(L._dp)
        self.check(self.lib.ibmlbm_init_fields(self.h, None, None, p, step0))

    def fields(self, which):
        n = {L.FIELD_RHO: 1, L.FIELD_U: 3, L.FIELD_FDIST: 19}[which]
        out = np.empty((n,) + self.shape)
        self.check(self.lib.ibmlbm_fields(self.h, which, out.ctypes.data_as(L._dp)))
        return out

    def step_count(self):
        return int(self.lib.ibmlbm_step_count(self.h))

    def close(self):
        self.check(self.lib.ibmlbm_destroy(self.h))
        self.h = None
