"""Device code of the library compiled for the host (host_core.cpp): coordinates
and pull offsets against integer division and the plain wrap, and the rounding
of half-storage initial values against numpy's correctly rounded conversion and
division."""
import ctypes
import itertools
import os
import subprocess

import numpy as np
import pytest

from paper_1608_06345_amd import lbm

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def core(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("core") / "libhostcore.so")
    subprocess.check_call(
        ["/opt/rocm/llvm/bin/clang++", "-x", "c++", "-std=c++20", "-O1", "-w",
         "-ffp-contract=off", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
         "-I" + os.path.join(ROOT, "include"),
         "-I" + os.path.join(ROOT, "paper_1608_06345_amd", "csrc"),
         os.path.join(ROOT, "tests", "host_core.cpp"), "-o", so])
    lib = ctypes.CDLL(so)
    lib.host_divide.argtypes = [ctypes.c_int, ctypes.c_int64]
    lib.host_offsets_wrong.restype = ctypes.c_int64
    return lib


def _ptr(a):
    return ctypes.c_void_p(a.ctypes.data)


def test_division_by_multiplication(core):
    rng = np.random.default_rng(1)
    top = 2 ** 31 - 1
    ds = [1, 2, 3, 5, 7, 64, 65, 255, 256, 257, 641, 2 ** 16 - 1, 2 ** 16, 2 ** 16 + 1, 2 ** 30,
          2 ** 30 - 1, 2 ** 30 + 1, top - 1, top, 2 ** 31]
    ds += [int(2 ** e) for e in rng.uniform(0, 31, 200)]
    for d in ds:
        ns = {0, 1, top, top - 1, d - 1, d, d + 1, top // d * d, top // d * d - 1}
        ns |= {int(2 ** e) for e in rng.uniform(0, 31, 50)}
        ns |= {int(k) * d + s for k in rng.integers(0, top // d + 1, 20) for s in (-1, 0)}
        for n in ns:
            if 0 <= n <= top:
                assert core.host_divide(n, d) == n // d, (n, d)


@pytest.mark.parametrize("dim", [2, 3])
def test_pull_offsets(core, dim):
    sides = (1, 2, 3, 4, 7, 11)
    for shape in itertools.product(sides, sides, (1,) if dim == 2 else sides):
        for open_end in range(4 if dim == 2 else 8):
            assert core.host_offsets_wrong(dim, *shape, open_end) == 0, (shape, open_end)


def _half_edges():
    """Every half, the ties between neighbours, and the doubles around both."""
    h = np.arange(0x7C00, dtype=np.uint16).view(np.float16).astype(np.float64)
    ties = (h[:-1] + h[1:]) / 2
    x = np.concatenate([h, ties, [65519.999, 65520.0, 65536.0, 1e300, 5e-324, 1e-40, 0.0]])
    x = np.concatenate([x, np.nextafter(x, np.inf), np.nextafter(x, -np.inf)])
    x = np.concatenate([x, x * (1 + 2.0 ** -30), x * (1 - 2.0 ** -30)])
    return np.concatenate([x, -x])


def test_rounding_to_half(core):
    x = np.concatenate([_half_edges(), [np.inf, -np.inf]])
    x = np.ascontiguousarray(x)
    out = np.empty(x.size, np.uint16)
    core.host_stored_half(_ptr(x), _ptr(out), ctypes.c_int64(x.size))
    with np.errstate(over="ignore"):
        want = x.astype(np.float16).view(np.uint16)
    bad = np.flatnonzero(out != want)
    assert bad.size == 0, (x[bad[:5]], out[bad[:5]], want[bad[:5]])
    nan = np.full(1, np.nan)
    core.host_stored_half(_ptr(nan), _ptr(out), ctypes.c_int64(1))
    assert np.isnan(out[:1].view(np.float16))[0]


@pytest.mark.parametrize("vset", [37, 107])
def test_division_by_a_weight(core, vset):
    """x / w for every group weight, of values over the range of populations and
    those whose quotients round at the ties of halves."""
    rng = np.random.default_rng(2)
    x0 = rng.uniform(-1, 1, 20000) * 10.0 ** rng.uniform(-30, 6, 20000)
    for w in sorted(set(lbm.lbm_lattice(vset)[1])):
        x = np.concatenate([x0, _half_edges() * w, [np.inf, -np.inf, np.nan]])
        out = np.empty_like(x)
        core.host_quotient(_ptr(x), ctypes.c_double(w), _ptr(out), ctypes.c_int64(x.size))
        want = x / w
        # a remainder below the smallest double is lost: far below the smallest half
        tiny = np.abs(want) < 1e-280
        assert np.all(np.abs(out[tiny]) < 1e-279)
        np.testing.assert_array_equal(out[~tiny], want[~tiny])
