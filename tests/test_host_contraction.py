"""The multiply-adds of the collision and of its adjoint are those written.

The kernels' compiler may fuse any multiply with an add that uses it, and where a sum
has two products its choice depends on the code around it.  The kernels agree bit for
bit (a step with totals, in place, two steps in one pass; both forms of the adjoint)
only if it has no choice: here the headers are compiled for the CPU with that freedom,
as for the GPU, and without it, and every bit has to be the same.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_1202_6081_amd import build as _b

SRC = os.path.join(_b.HOST_DIR, "host_contraction.cpp")


def _has_fma():
    try:
        with open("/proc/cpuinfo") as fh:
            return " fma " in fh.read()
    except OSError:
        return False


@pytest.fixture(scope="module")
def libs(tmp_path_factory):
    if not _has_fma():
        pytest.skip("the CPU has no fused multiply-add instruction")
    clang = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(_b.hipcc()))), "llvm", "bin", "clang++")
    out = []
    for mode in ("fast-honor-pragmas", "off"):
        lib = str(tmp_path_factory.mktemp("contract") / f"{mode}.so")
        subprocess.run([clang, *_b.HOST_FLAGS, "-O2", "-mfma", f"-ffp-contract={mode}", "-fPIC", "-shared", SRC, "-o", lib],
                       check=True)
        out.append(ctypes.CDLL(lib))
    return out


@pytest.mark.parametrize("per_mass", [0, 1])
@pytest.mark.parametrize("real", ["f32", "f64"])
@pytest.mark.parametrize("q", [27, 15])
def test_no_bit_is_the_compilers_choice(libs, q, real, per_mass):
    dtype = np.float32 if real == "f32" else np.float64
    rng = np.random.default_rng(q + per_mass)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    for _ in range(200):
        w = np.array([8 / 27] + [2 / 27] * 6 + [1 / 54] * 12 + [1 / 216] * 8 if q == 27 else [2 / 9] + [1 / 9] * 6 + [1 / 72] * 8)
        f = (w * (1 + 0.1 * rng.standard_normal(q))).astype(dtype)
        F = (1e-2 * rng.standard_normal(3)).astype(dtype)
        g = rng.standard_normal(q).astype(dtype)
        omega = rng.uniform(0.5, 1.9, q - 4)
        step, adj = [np.zeros(q, dtype) for _ in libs], [np.zeros(q + 26, dtype) for _ in libs]
        for lib, s, a in zip(libs, step, adj):
            getattr(lib, f"hc_collide_{real}")(q, p(f), p(F), p(omega), per_mass, p(s))
            getattr(lib, f"hc_adjoint_bits_{real}")(q, p(f), p(F), p(omega), per_mass, p(g), p(a))
        assert np.array_equal(step[0], step[1])
        assert np.array_equal(adj[0], adj[1])
