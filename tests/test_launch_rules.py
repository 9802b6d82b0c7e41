"""The rules that size the Huffman launches, from the library's own header built with g++ (no GPU): workgroups per
compute unit of the device at hand, entries of a result's record, and the long sums that a block adds up."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2312_05492_amd", "csrc")
SOURCE = """
#include "szi_internal.h"
extern "C" int block_chunks(uint64_t chunks, int cus) { return szi::enc_block_chunks(chunks, cus); }
extern "C" uint64_t entries(uint64_t chunks) { return szi::sub_entries(chunks); }
extern "C" int super_shift(uint64_t blocks) { return szi::enc_super_shift(blocks); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    cxx, rocm = shutil.which("g++"), "/opt/rocm/include"
    if cxx is None or not os.path.exists(rocm + "/hip/hip_runtime.h"):
        pytest.skip("no g++ or no HIP headers")
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(SOURCE)
    subprocess.check_call([cxx, "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I", rocm, "-I",
                           os.path.join(ROOT, "include"), "-I", CSRC, str(d / "rules.cpp"), "-o", str(d / "rules.so")])
    lib = C.CDLL(str(d / "rules.so"))
    lib.block_chunks.argtypes = [C.c_uint64, C.c_int]
    lib.entries.restype = C.c_uint64
    lib.entries.argtypes = [C.c_uint64]
    lib.super_shift.argtypes = [C.c_uint64]
    return lib


@pytest.mark.parametrize("cus", [32, 64, 228, 256, 304])
def test_encode_blocks_per_cu(rules, cus):
    # the largest of 4, 8, 16 and 32 chunks a workgroup that leaves eight workgroups a CU
    for ec in (4, 8, 16, 32):
        for chunks in (8 * cus * ec - 1, 8 * cus * ec, 16 * cus * ec - 1):
            want = max([4] + [e for e in (8, 16, 32) if chunks >= 8 * cus * e])
            assert rules.block_chunks(chunks, cus) == want
    assert rules.block_chunks(1, cus) == 4 and rules.block_chunks(1 << 24, cus) == 32


def test_record_stays_within_its_blocks(rules):
    # a place for each chunk costs nothing beside its eight offsets in device blocks of 512 bytes
    for chunks in list(range(1, 200)) + [131072, 131073, 4194304]:
        n = rules.entries(chunks)
        assert n >= 8 * chunks and -(-2 * n // 512) == -(-16 * chunks // 512)
        assert n > 8 * (32 * ((chunks - 1) // 32) + 1)   # the high half of the last unit's first word


def test_long_sums_added_up(rules):
    # at most 256 of them, more are scanned
    for blocks in (1, 64, 16383, 16384, 16385, 524288):
        shift = rules.super_shift(blocks)
        assert shift == 8 or blocks >> shift <= 256
        assert (shift == 8) == (blocks > 16384)
