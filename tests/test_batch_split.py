"""The plain arithmetic of the batch kernel (csrc/sqllm_batch_split.h), compiled for the CPU with signed overflow made fatal: windows of
nonzeros up to the largest position the interface accepts (nnz < 2^31), against the definition in Python's integers."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2306_07629_amd", "csrc")
TOP = 2 ** 31 - 1

SOURCE = r"""
#include "sqllm_batch_split.h"
using namespace sqllm;
extern "C" {
int count(int first, int end) { return window_count(first, end); }
int rest(int p0, int end) { return window_rest(p0, end); }
uint32_t row_bits(int lo, int hi, int p0, int q) { return window_row_bits(lo, hi, p0, q); }
}
"""


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    d = tmp_path_factory.mktemp("split")
    src, so = d / "split.cpp", d / "split.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-ftrapv", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    lib.row_bits.restype = ctypes.c_uint32
    return lib


@pytest.mark.parametrize("first,end", [(0, 1), (0, 128), (3, 132), (7, 7), (0, TOP), (TOP - 1, TOP), (TOP - 127, TOP), (TOP - 200, TOP),
                                       (TOP - 128 * 40, TOP), (TOP - 5000, TOP - 90)])
def test_windows_cover_a_row_group_and_read_nothing_else(split, first, end):
    n = split.count(first, end)
    assert n == -(-(end - first) // 128)
    for f in sorted({0, 1, n // 2, n - 2, n - 1} & set(range(n))) if n > 64 else range(n):
        p0 = first + 128 * f
        last = p0 + split.rest(p0, end)
        assert p0 <= last == end - 1                                 # the kernel reads positions p0 + min(k, rest), k < 128
        reads = [p0 + min(k, split.rest(p0, end)) for k in range(128)]
        assert first <= min(reads) and max(reads) < end


@pytest.mark.parametrize("base", [0, 1000, TOP - 700])
def test_row_bits_name_the_positions_of_the_row(split, base):
    ptr = [base + o for o in (0, 0, 5, 37, 37, 160, 161, 500, 700)]  # eight rows, empty ones among them
    for p0 in [base + 128 * f for f in range(split.count(ptr[0], ptr[-1]))]:
        for q in range(4):
            owner = [next((r for r in range(8) if ptr[r] <= p0 + 32 * q + k < ptr[r + 1]), None) for k in range(32)]
            for r in range(8):
                assert split.row_bits(ptr[r], ptr[r + 1], p0, q) == sum(1 << k for k in range(32) if owner[k] == r), (p0, q, r)
    assert split.row_bits(0, base, base, 0) == 0                     # rows far in front of and far behind the window
    assert split.row_bits(TOP, TOP, 0, 3) == 0
