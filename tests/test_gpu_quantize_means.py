"""Row lengths and row counts at which the k-means kernel changes its shape, and the means of its clusters.  A mean is formed without
a division and checked against the places where that could round differently: means that are exact, that lie in the middle between two
fp32 numbers or next to it, equal weights of both signs, zeros of both signs."""
import numpy as np
import pytest

from oracle import quant_oracle as qo

pytestmark = pytest.mark.gpu


def rows(kind, M, N, rng):
    """(weights, sensitivities) of M rows"""
    if kind == "middles":
        # two neighbouring powers with sensitivities that put the mean on or next to a multiple of half an fp32 step: 1 + k / 2^24 and such
        w = np.where(rng.random((M, N)) < 0.5, 1.0, 1.0 + 2.0 ** -10)
        s = rng.choice([1, 2, 4, 8191, 8192, 8193, 16384, 16385, 32768, 65535], size=(M, N))
    elif kind == "zeros":
        w = rng.choice([0.0, -0.0, 2.0 ** -24, -(2.0 ** -24), 0.5, -0.5], size=(M, N))
        s = rng.integers(0, 3, size=(M, N))
    elif kind == "levels":
        w = np.round(rng.standard_normal((M, N)) * 8) / 8
        s = np.full((M, N), 4096)
    else:                                                                 # wide rows: beyond the range of 32-bit products
        w = rng.standard_normal((M, N)) * 9000
        s = rng.integers(1, 65536, size=(M, N))
    return w.astype(np.float16).view(np.uint16), s.astype(np.uint16)


def check(M, N, bits, w, s):
    import torch
    import paper_2306_07629_amd as sq
    import oracle
    counts = (M * N // 300, M * N // 300, M * N // 500)
    q = sq.quantize_layer(torch.from_numpy(w.view(np.int16)).cuda(), torch.from_numpy(s.view(np.int16)).cuda(), bits, *counts, max_iter=32)
    ref = qo.quantize_layer(w, s, bits, *counts, 32)
    nnz = q.nnz()
    assert np.array_equal(q.rowptr.cpu().numpy(), ref["rowptr"])
    assert np.array_equal(q.cols.cpu().numpy()[:nnz], ref["cols"]) and np.array_equal(q.vals.cpu().numpy().view(np.uint16)[:nnz], ref["vals"])
    assert np.array_equal(q.iters.cpu().numpy(), ref["iters"])
    assert np.array_equal(q.lut.cpu().numpy().view(np.uint16), ref["lut"])
    assert np.array_equal(oracle.unpack(M, N, bits, q.qidx.cpu().numpy()), ref["idx"])


@pytest.mark.parametrize("kind", ["middles", "zeros", "levels", "wide"])
@pytest.mark.parametrize("N,bits", [(128, 2), (1024, 3), (1152, 4), (4096, 4), (4224, 3)])
def test_means_next_to_the_middle_of_two_numbers(kind, N, bits):
    check(6, N, bits, *rows(kind, 6, N, np.random.default_rng(N + bits)))


# last and first row length of every shape; 8192 columns: 512 rows and more than that
@pytest.mark.parametrize("M,N,bits", [(9, 896, 4), (9, 1024, 2), (9, 1152, 3), (9, 2048, 4), (9, 2176, 3), (5, 6144, 4), (5, 6272, 3),
                                      (512, 6272, 3), (513, 6272, 4), (513, 8192, 2), (5, 8320, 4), (5, 11776, 4), (5, 11904, 3), (5, 12288, 2)])
def test_shapes(M, N, bits):
    import gen
    check(M, N, bits, gen.make_weights(M, N, N + bits), gen.make_sens(M, N, N + bits))
