"""csrc/sqllm_batch_split.h, csrc/sqllm_csr.h and csrc/sqllm_buckets.h compiled for the CPU, with signed overflow made fatal."""
import ctypes
import functools
import os
import subprocess
import tempfile

import numpy as np

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2306_07629_amd", "csrc")

SOURCE = r"""
#include "sqllm_batch_split.h"
#include "sqllm_buckets.h"
#include "sqllm_csr.h"
using namespace sqllm;
extern "C" {
int count(int first, int end) { return window_count(first, end); }
int rest(int p0, int end) { return window_rest(p0, end); }
uint32_t row_bits(int lo, int hi, int p0, int q) { return window_row_bits(lo, hi, p0, q); }
void split(int M, int N, int bits, int B, int dense, int sparse, int* out) {
    const BatchSplit s = batch_split(M, N, bits, B, dense != 0, sparse != 0);
    out[0] = s.row_groups; out[1] = s.blocks; out[2] = s.dense_waves; out[3] = s.sparse_waves; out[4] = (int)s.lds;
}
int waves_per_simd(int row_groups, int B) { return batch_waves_per_simd(row_groups, B); }
int batches(int first, int end) { return csr_batch_count(first, end); }
void positions(int first, int end, int b, int* out) {
    for (int lane = 0; lane < kBatchNonzeros; ++lane) out[lane] = csr_position(end, csr_nonzero(first, b, lane));
}
void rows4(const int* rp, int b, int* out) {
    for (int lane = 0; lane < kBatchNonzeros; ++lane) out[lane] = csr_row<4>(*reinterpret_cast<const int(*)[5]>(rp), csr_nonzero(rp[0], b, lane));
}
void rows8(const int* rp, int b, int* out) {
    for (int lane = 0; lane < kBatchNonzeros; ++lane) out[lane] = csr_row<8>(*reinterpret_cast<const int(*)[9]>(rp), csr_nonzero(rp[0], b, lane));
}
uint32_t counter(uint32_t v) { return spread_word(v); }
int kmeans_shape(int M, int N) { return kmeans_columns(M, N); }
int has_room(int p, int row_end, int capacity) { return csr_has_room(p, row_end, capacity); }
}
"""


@functools.lru_cache(maxsize=None)
def library():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "split.cpp"), os.path.join(d, "split.so")
        with open(src, "w") as f:
            f.write(SOURCE)
        subprocess.run(["g++", "-std=c++17", "-O1", "-ftrapv", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + CSRC, src, "-o", so], check=True)
        lib = ctypes.CDLL(so)
    lib.row_bits.restype = lib.counter.restype = ctypes.c_uint32
    return lib


def batch_split(M, N, bits, B, dense, sparse):
    """(row groups, blocks, dense waves, sparse waves, bytes of LDS) of the launch"""
    out = (ctypes.c_int * 5)()
    library().split(M, N, bits, B, int(dense), int(sparse), out)
    return tuple(out)


def csr_positions(first, end, b):
    """the positions that the 64 lanes read for batch b of the nonzeros [first, end)"""
    out = np.empty(64, dtype=np.int32)
    library().positions(int(first), int(end), int(b), out.ctypes.data_as(ctypes.POINTER(ctypes.c_int)))
    return out.astype(np.int64)


def csr_rows(rp, b):
    """the rows (0 .. R - 1; R and more: none) to which the 64 lanes add their products of batch b; rp: R + 1 row pointers, R = 4 or 8"""
    a, out = np.ascontiguousarray(rp, dtype=np.int32), np.empty(64, dtype=np.int32)
    p = ctypes.POINTER(ctypes.c_int)
    {5: library().rows4, 9: library().rows8}[a.size](a.ctypes.data_as(p), int(b), out.ctypes.data_as(p))
    return out
