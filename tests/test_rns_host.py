"""The RNS engine's host-made tables on the CPU: tests/rns_host_sim.cpp compiles
csrc/rns_host.hpp with the host compiler and walks one element through the steps
of the output conversion."""
from __future__ import annotations

import ctypes
import os
import random
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if not cxx or not os.path.isdir(os.path.join(rocm, "include", "hip")):
        pytest.skip("no host C++ compiler or HIP headers")
    out = tmp_path_factory.mktemp("rnshost") / "librnshost.so"
    subprocess.run([cxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-pthread",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    "-o", str(out), os.path.join(HERE, "rns_host_sim.cpp")], check=True)
    return ctypes.CDLL(str(out))


def _words(v: int, n: int) -> np.ndarray:
    return np.frombuffer(v.to_bytes(4 * n, "little"), dtype="<u4").copy()


def _ptr(a: np.ndarray):
    return a.ctypes.data_as(ctypes.POINTER(ctypes.c_uint32))


# (declared bits of the result, bits of the modulus): as long as declared, just
# where the limbs (28 bits, in blocks of eight) end below the last word, and
# far below it.  Whatever stands behind the limbs must not show.
@pytest.mark.parametrize("declared,bits", [
    (4096, 4096), (4096, 4020), (4096, 4004), (4096, 3980), (4096, 3600), (4096, 1200),
    (2048, 2048), (2048, 1980), (2048, 1900), (2048, 1200), (2048, 512),
    (1024, 1020), (1024, 868), (1024, 512), (6144, 6000), (8192, 8000)])
def test_output_conversion_of_short_moduli(lib, declared, bits):
    rng = random.Random(declared + bits)
    T = lib.sim_tiles(bits)
    assert T > 0
    buf = np.zeros(1024, dtype=np.uint32)
    ma = int.from_bytes(buf[:lib.sim_ma(T, _ptr(buf))].tobytes(), "little")
    nw = declared // 32
    for mont in (0, 1):
        N = 0
        for x in (0, 1, -1, rng.getrandbits(bits - 2)):
            out = np.zeros(nw, dtype=np.uint32)
            while True:
                N = N or rng.getrandbits(bits) | 1 | (3 << (bits - 2))
                x %= N
                a, b = _words(N, nw), _words(x, nw)
                if lib.sim_from(_ptr(a), nw, _ptr(b), nw, T, mont, nw, 0xA5A5A5A5,
                                _ptr(out)) == 0:
                    break
                N = 0  # shares a factor with a channel
            want = x * pow(ma, -1, N) % N if mont else x
            assert int.from_bytes(out.tobytes(), "little") == want


# every split of every length that a mat-vec plan can take: the blocks cover the
# constant's bits, the digits a block's bits once, and their entries a column's table
# behind entry 0
@pytest.mark.parametrize("ebits", range(1, 65))
def test_matvec_digits(lib, ebits):
    for nblk in range(1, ebits + 1):
        bits = -(-ebits // nblk)
        for n in range(-(-bits // 12), bits + 1):
            out = np.zeros((n, 4), dtype=np.int32)
            entries = lib.sim_digits(ebits, n, nblk,
                                     out.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)))
            shift, at = 0, 1
            for s, w, first, last in out.tolist():
                assert s == shift and 1 <= w <= 12
                assert first == at and last == at + (1 << w) - 2
                shift, at = shift + w, last + 1
            assert shift == bits and at == entries
            assert max(out[:, 1]) - min(out[:, 1]) <= 1


# the compiled splits keep every 32-bit sum in range, and splits that would not are
# refused (the sums of beta at T = 34 reach 0.78 of 2^31 with four tiles a wavefront)
@pytest.mark.parametrize("T,mt,ok", [
    (5, 0, 1), (9, 0, 1), (13, 0, 1), (17, 0, 1), (26, 0, 1), (34, 0, 1),
    (34, 4, 1), (34, 6, 0), (34, 8, 0), (17, 4, 1), (17, 8, 0)])
def test_bounds_of_the_splits(lib, T, mt, ok):
    assert lib.sim_bounds(T, mt) == ok
