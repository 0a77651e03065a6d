"""The multiply-adds of the collision and of its adjoint are those written.

The kernels' compiler may fuse any multiply with an add that uses it, and where a sum
has two products its choice depends on the code around it.  The kernels agree bit for
bit (a step with totals, in place, two steps in one pass; both forms of the adjoint)
only if it has no choice: here the headers are compiled for the CPU with that freedom,
as for the GPU, and without it, and every bit has to be the same.
"""
import ctypes
import hashlib
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
@pytest.mark.parametrize("real", ["f32", "f64", "16"])
@pytest.mark.parametrize("q", [27, 15])
def test_no_bit_is_the_compilers_choice(libs, q, real, per_mass):
    dtype = np.float64 if real == "f64" else np.float32
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
            getattr(lib, f"hc_collide_{'f64' if real == 'f64' else 'f32'}")(q, p(f), p(F), p(omega), per_mass, p(s))
            getattr(lib, f"hc_adjoint_bits_{real}")(q, p(f), p(F), p(omega), per_mass, p(g), p(a))
        assert np.array_equal(step[0], step[1])
        assert np.array_equal(adj[0], adj[1])


# Gradients are FP64 numbers also where the arithmetic is FP32, so a program may hold them to
# more digits than FP32 has: their bits stay.  Digests (SHA-256, first 16 digits) of the
# adjoints of populations, force and rates at 500 nodes.
BITS_F32 = {(27, 0): "f387e6cf1ded7a3d", (27, 1): "ef57780b531938a8",
            (15, 0): "d27cb8674505ad5b", (15, 1): "2a046a07a20218fe"}
BITS_16 = {(27, 0): BITS_F32[27, 0], (27, 1): BITS_F32[27, 1],
           (15, 0): "87cc010b0199585a", (15, 1): "ab1e2373c6fb0c64"}


def _node(q, n):
    """Populations, force, their adjoint and rates of node n, from integers alone."""
    x = np.empty(2 * q + 3 + q - 4)
    state = 2 * n + 1
    for i in range(x.size):
        state = state * 6364136223846793005 + 1442695040888963407 & (1 << 64) - 1
        x[i] = (state >> 40) / (1 << 23) - 1        # [-1, 1), exact in FP32
    w = np.array([8 / 27] + [2 / 27] * 6 + [1 / 54] * 12 + [1 / 216] * 8 if q == 27 else [2 / 9] + [1 / 9] * 6 + [1 / 72] * 8)
    f = (w * (1 + 0.1 * x[:q])).astype(np.float32)
    return f, (0.01 * x[q:q + 3]).astype(np.float32), x[q + 3:2 * q + 3].astype(np.float32), 1.2 + 0.7 * x[2 * q + 3:]


@pytest.mark.parametrize("q, per_mass", list(BITS_F32))
@pytest.mark.parametrize("real, bits", [("f32", BITS_F32), ("16", BITS_16)], ids=["f32", "16"])
def test_gradients_keep_their_bits(libs, real, bits, q, per_mass):
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    out, h = np.zeros(q + 26, np.float32), hashlib.sha256()
    for n in range(500):
        f, F, g, omega = _node(q, n)
        getattr(libs[1], f"hc_adjoint_bits_{real}")(q, p(f), p(F), p(omega), per_mass, p(g), p(out))
        assert np.isfinite(out).all()
        h.update(out.tobytes())
    assert h.hexdigest()[:16] == bits[q, per_mass]
