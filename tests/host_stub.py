"""Runs the library's host side on a HIP runtime that launches nothing (hip_stub.cpp), in
a process of its own: which kernels a call launches, what memory it takes, whether it
returns. No GPU and no torch in that process; kernels leave no results."""

import ctypes
import functools
import os
import re
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2103_04856_amd", "libfe.so")

TRACE_P = (1.0, 2.0, 1.0, -3.0, -3.0, 2.95)           # (k1 + k2 - 1.5)^2 + 0.7: k1 + k2 alone
HELFRICH_P = (1.0, 2.5, 1.0, -4.0, -4.0, 4.0)         # (k1 + k2 - 2)^2 + 0.5 k1 k2: symmetric
ASYM_P = (1.0, 0.3, 2.0, -3.0, 5.0, 0.7)              # every term
NO_S, FULL, TRACE = 1, 2, 3                           # per-voxel bodies of the sweeps
F32, F64 = 0, 1
EINVAL, ENOMEM = -1, -3


@functools.lru_cache(maxsize=None)
def _stub():
    out = os.path.join(tempfile.mkdtemp(prefix="hipstub"), "libhipstub.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-o", out, os.path.join(HERE, "hip_stub.cpp")], check=True)
    return out


def run(fn, timeout=60):
    """fn(api) in a fresh process; an assertion or a time-out there fails the caller."""
    code = (f"import sys; sys.path.insert(0, {HERE!r}); import importlib.util as u; "
            f"s = u.spec_from_file_location('cases', {fn.__code__.co_filename!r}); m = u.module_from_spec(s); "
            f"s.loader.exec_module(m); import host_stub; m.{fn.__name__}(host_stub.Api({_stub()!r}))")
    res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=timeout)
    assert res.returncode == 0, f"exit {res.returncode}: {res.stdout}{res.stderr}"


class Grid(ctypes.Structure):
    _fields_ = [("nx", ctypes.c_int), ("ny", ctypes.c_int), ("nz", ctypes.c_int), ("batch", ctypes.c_int),
                ("h", ctypes.c_double), ("dtype", ctypes.c_int)]


def dbl(v):
    return (ctypes.c_double * len(v))(*v)


class Api:
    """libfe.so on the stub runtime. Fields are host memory that no kernel reads."""

    def __init__(self, stub):
        self.stub = ctypes.CDLL(stub, mode=ctypes.RTLD_GLOBAL)
        self.lib = ctypes.CDLL(LIB)
        self.stub.stub_log_name.restype = ctypes.c_char_p
        self.stub.stub_energy.restype = ctypes.c_void_p
        self.stub.stub_next.argtypes = [ctypes.c_double]
        self.lib.fe_last_error.restype = ctypes.c_char_p

    def grid(self, shape, dtype=F32, batch=1):
        nz, ny, nx = shape
        return Grid(nx, ny, nz, batch, 1.0 / nx, dtype)

    def context(self, shape, p=HELFRICH_P, dtype=F32, batch=1):
        out = ctypes.c_void_p()
        rc = self.lib.fe_create(ctypes.byref(self.grid(shape, dtype, batch)), dbl([2.0 / shape[2]] * batch),
                                dbl(list(p) * batch), None, ctypes.byref(out))
        assert rc == 0, self.error()
        return out

    def set_params(self, ctx, shape, p, batch=1):
        assert self.lib.fe_set_params(ctx, dbl([2.0 / shape[2]] * batch), dbl(list(p) * batch)) == 0, self.error()

    def field(self, shape, values=1):
        return (ctypes.c_double * (shape[0] * shape[1] * shape[2] * values))()

    def error(self):
        return self.lib.fe_last_error().decode()

    def log(self):
        """Kernels launched since the last call, (name, blocks) in order."""
        out = [(self.stub.stub_log_name(ctypes.c_long(i)).decode(), self.stub.stub_log_blocks(ctypes.c_long(i)))
               for i in range(self.stub.stub_log_size())]
        self.stub.stub_log_clear()
        return out

    def sweeps(self):
        """The gradient and step sweeps among them: (mode, body, forms the energy)."""
        pat = re.compile(r"grad_sweepI[fd]Li\d+ELi\d+ELi\d+ELi(\d)ELb[01]ELb[01]ELi(\d)ELb([01])E")
        return [(int(m[1]), int(m[2]), m[3] == "1") for m in (pat.search(n) for n, _ in self.log()) if m]
