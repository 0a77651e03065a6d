"""The library's launch rules, as the host build tests/host/host_plan.cpp exports them."""
import ctypes
import os
from collections import namedtuple

from paper_1202_6081_amd import build as _b

Step2 = namedtuple("Step2", "pays main tail tail_rows zlen")
Adjoint = namedtuple("Adjoint", "blocks segment split")
_lib = None


def lib():
    global _lib
    if _lib is None:
        srcs = [_b.PLAN_SRC] + [os.path.join(_b.CSRC, n) for n in os.listdir(_b.CSRC) if n.endswith(".hpp")]
        if not os.path.exists(_b.PLAN_LIB) or os.path.getmtime(_b.PLAN_LIB) < max(map(os.path.getmtime, srcs)):
            _b.build_host_plan()
        _lib = ctypes.CDLL(_b.PLAN_LIB)
        _lib.hp_run_length.argtypes = [ctypes.c_uint32] * 2
        _lib.hp_run_length.restype = ctypes.c_uint32
    return _lib


def step2_plan(q, prec, shape, walls):
    """shape: (nz, ny, nx)."""
    nz, ny, nx = shape
    out = (ctypes.c_uint32 * 4)()
    return Step2(bool(lib().hp_step2_plan(q, prec, nx, ny, nz, int(walls), out)), *out)


def adjoint_launch(q, prec, shape):
    nz, ny, nx = shape
    out = (ctypes.c_int * 3)()
    lib().hp_adjoint(q, prec, nx, ny, nz, out)
    return Adjoint(out[0], out[1], bool(out[2]))


def thin_pays(q, prec, shape, walls):
    nz, ny, nx = shape
    return bool(lib().hp_thin(q, (8, 4, 2, 2)[prec], nx, ny, nz, int(walls)))
