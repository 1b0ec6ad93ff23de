"""Which shape of the k-means kernel a matrix takes (csrc/sqllm_buckets.h, compiled for the CPU)."""
import os
import re

import pytest

import host_split

WIDER = {1024: 1024, 2048: 4096, 4096: 4096, 6144: 11776, 8192: 11776}    # by columns: the shape with more threads


def shape(M, N):
    return host_split.library().kmeans_shape(M, N)


def test_every_row_fits_its_shape_and_every_shape_is_launched():
    seen = set()
    for N in range(128, 28673, 128):
        for M in (1, 512, 513, 768, 769, 1024, 1025, 1536, 1537, 4096, 2 ** 31 - 1):
            assert shape(M, N) >= N
            seen.add(shape(M, N))
    src = open(os.path.join(host_split.CSRC, "sqllm_quant.hip")).read()
    body = src[src.index("launch_kmeans_shape("):]
    cases = {int(a): b for a, b in re.findall(r"case (\d+): return launch_kmeans_bits<KmeansUpTo(\d+)>", body)}
    assert all(str(a) == b for a, b in cases.items()) and seen == set(cases) | {28672}


@pytest.mark.parametrize("N", [1152, 2048, 4224, 5120, 6144, 6272, 8192])
def test_few_rows_take_the_shape_with_more_threads(N):
    """as many as the wider shape has on the chip at once: six per unit up to 4096 columns, two beyond"""
    top = next(c for c in WIDER if N <= c)
    on_chip = 256 * (6 if N <= 4096 else 2)
    for M in (1, 16, 200, on_chip - 1, on_chip):
        assert shape(M, N) == WIDER[top]
    for M in (on_chip + 1, 4096, 100000):
        assert shape(M, N) == top


def test_rows_that_are_as_many_generations_either_way():
    """6145 to 8192 columns, three rows per unit against two"""
    for N in (6272, 8192):
        for M in range(1, 6000):
            narrow, wide = -(-M // 768), -(-M // 512)
            assert shape(M, N) == (8192 if narrow < wide else 11776), (M, N)


def test_short_and_long_rows_take_one_shape_whatever_their_number():
    for N, want in ((128, 1024), (1024, 1024), (2176, 4096), (4096, 4096), (8320, 11776), (11776, 11776), (11904, 12288), (12416, 16384), (16512, 28672)):
        assert {shape(M, N) for M in (1, 512, 513, 1000, 4096)} == {want}
