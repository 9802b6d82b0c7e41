"""The blob's CRC-32 against zlib's: every length around the 8-, 16- and 64-byte steps of its table and carry-less
multiply forms, offsets off their alignment, and a running value carried over pieces (host code, built with g++)."""
import ctypes as C
import os
import shutil
import subprocess
import zlib

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2312_05492_amd", "csrc")


@pytest.fixture(scope="module")
def crc(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    so = str(tmp_path_factory.mktemp("crc") / "blob.so")
    subprocess.check_call([cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                           os.path.join(CSRC, "blob.cpp"), "-o", so])
    f = getattr(C.CDLL(so), "_ZN3szi12crc32_updateEjPKhm")
    f.restype = C.c_uint32
    f.argtypes = [C.c_uint32, C.c_void_p, C.c_size_t]
    return f


def test_crc32_equals_zlib(crc):
    data = np.random.default_rng(1).integers(0, 256, 5000, dtype=np.uint8)
    for n in list(range(0, 330)) + [1000, 4096, 4979]:
        for off in (0, 1, 7, 16):
            piece = data[off:off + n].tobytes()
            assert crc(0, data.ctypes.data + off, n) == zlib.crc32(piece)
            assert crc(zlib.crc32(b"before"), data.ctypes.data + off, n) == zlib.crc32(piece, zlib.crc32(b"before"))


@pytest.fixture(scope="module")
def crc_tables(tmp_path_factory):
    """The library's CRC as a CPU without carry-less multiplies runs it: tables alone, at every length."""
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("crc_tables")
    (d / "t.cpp").write_text("#include <cmath>\n#include <cstdarg>\n#include <cstdio>\n#include <cstring>\n"
                             "#include <string>\n#include <vector>\n#include <algorithm>\n"
                             "#undef __x86_64__\n#include \"blob.cpp\"\n")
    subprocess.check_call([cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                           str(d / "t.cpp"), "-o", str(d / "t.so")])
    f = getattr(C.CDLL(str(d / "t.so")), "_ZN3szi12crc32_updateEjPKhm")
    f.restype = C.c_uint32
    f.argtypes = [C.c_uint32, C.c_void_p, C.c_size_t]
    return f


def test_crc32_by_tables_equals_zlib(crc_tables):
    test_crc32_equals_zlib(crc_tables)
