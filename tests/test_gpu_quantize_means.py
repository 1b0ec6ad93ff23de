"""Row lengths and row counts at which the k-means kernel changes its shape, and the means of its clusters.  A mean is formed without
a division and checked against the places where that could round differently: quotients that lie in the middle between two fp32 numbers or up
to eight units of the last fp64 place beside it, where the kernel does divide (that the rows reach it is asserted on the host), means that are
exact, equal weights of both signs, zeros of both signs."""
import numpy as np
import pytest

from oracle import quant_oracle as qo

pytestmark = pytest.mark.gpu


def rows(kind, M, N, rng):
    """(weights, sensitivities) of M rows"""
    if kind == "two values":
        # neighbouring numbers; with two bits or more each has a cluster of its own, and the means are exact
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


def check(M, N, bits, w, s, counts=None):
    import torch
    import paper_2306_07629_amd as sq
    import oracle
    counts = (M * N // 300, M * N // 300, M * N // 500) if counts is None else counts
    q = sq.quantize_layer(torch.from_numpy(w.view(np.int16)).cuda(), torch.from_numpy(s.view(np.int16)).cuda(), bits, *counts, max_iter=32)
    ref = qo.quantize_layer(w, s, bits, *counts, 32)
    nnz = q.nnz()
    assert np.array_equal(q.rowptr.cpu().numpy(), ref["rowptr"])
    assert np.array_equal(q.cols.cpu().numpy()[:nnz], ref["cols"]) and np.array_equal(q.vals.cpu().numpy().view(np.uint16)[:nnz], ref["vals"])
    assert np.array_equal(q.iters.cpu().numpy(), ref["iters"])
    assert np.array_equal(q.lut.cpu().numpy().view(np.uint16), ref["lut"])
    assert np.array_equal(oracle.unpack(M, N, bits, q.qidx.cpu().numpy()), ref["idx"])
    return ref


@pytest.mark.parametrize("kind", ["two values", "zeros", "levels", "wide"])
@pytest.mark.parametrize("N,bits", [(128, 2), (1024, 3), (1152, 4), (4096, 4), (4224, 3)])
def test_means_of_few_values_and_of_wide_rows(kind, N, bits):
    check(6, N, bits, *rows(kind, 6, N, np.random.default_rng(N + bits)))


def shared(total, n, rng):
    """n sensitivities with that sum"""
    s = np.full(n, total // n)
    s[:total % n] += 1
    a, b = np.array_split(rng.permutation(n), 2)
    d = rng.integers(0, np.minimum(s[a[:b.size]], 65535 - s[b]) + 1)
    s[a[:b.size]] -= d
    s[b] += d
    assert s.sum() == total and s.min() >= 0 and s.max() <= 65535
    return s


def row_with_a_mean_at(offset, N, bits, scale, sign, rng):
    """(weights, sensitivities, members of the cluster): 2^bits groups of equal size, which are the clusters; one holds the neighbours 1 and
    1 + 2^-10 (times scale), with sensitivities whose mean is 1 + odd / 2^24 for offset 0, and a little above or below that else: the quotient
    differs from the middle by offset / (sum of the sensitivities) / 2^24"""
    K, G = 1 << bits, N >> bits
    c = int(rng.integers(0, K))
    if offset == 0:
        t = int(rng.integers(1, G * 65535 * 7 // 10 // 2 ** 14 + 1))
        S, odd = t * 2 ** 14, int(rng.integers(0, 2 ** 13)) * 2 + 1
    else:
        S = int(rng.integers(2 ** 25, G * 65535 * 7 // 10)) | 1
        odd = -offset * pow(S, -1, 2 ** 14) % 2 ** 14
    Su = (odd * S + offset) // 2 ** 14
    assert (odd * S + offset) % 2 ** 14 == 0 and odd % 2 == 1 and 0 < Su < S
    u = min(max(round(G * Su / S), -(-Su // 65535), 1), G - 1 - (S - Su) // 65535)
    g = np.arange(N) // G
    w = np.where(g == c, 1.0, 4.0 * (g - c) + np.where(g > c, 4.0, 0.0))
    w[c * G:c * G + u] = 1.0 + 2.0 ** -10
    s = rng.integers(1, 65536, N)
    s[c * G:c * G + u], s[c * G + u:(c + 1) * G] = shared(Su, u, rng), shared(S - Su, G - u, rng)
    order = rng.permutation(N)
    return (sign * scale * w)[order].astype(np.float16).view(np.uint16), s[order].astype(np.uint16), (g == c)[order]


@pytest.mark.parametrize("N,bits", [(1024, 2), (2048, 3), (4096, 2), (4096, 4), (5120, 2), (8192, 2), (11776, 2), (11776, 3), (16384, 3), (28672, 4)])
def test_means_next_to_the_middle_of_two_numbers(N, bits):
    rng = np.random.default_rng(N + bits)
    offsets = [0, 0] + ([1, -1, 3, -3] if (N >> bits) * 65535 * 7 // 10 > 2 ** 26 else [1, -1] if (N >> bits) * 65535 * 7 // 10 > 2 ** 25 else [])
    cases = [(o, scale, sign) for o in offsets for scale in ((1.0, 64.0) if bits == 2 else (1.0,)) for sign in (1, -1)]   # 64: rows of 128 and more
    w, s, member = (np.array(a) for a in zip(*(row_with_a_mean_at(o, N, bits, scale, sign, rng) for o, scale, sign in cases)))
    near = 0
    for i, (o, scale, sign) in enumerate(cases):
        S0 = int(s[i][member[i]].astype(np.int64).sum())
        p = s[i][member[i]].astype(np.int64) * qo.half_to_fixed(w[i][member[i]])
        S1 = qo._exact_to_f64(int((p >> 32).sum()), int((p & 0xFFFFFFFF).sum()))
        q = S1 * np.float64(2.0 ** -24) / np.float64(S0)
        dropped = int(q.view(np.uint64)) & 0x1FFFFFFF                # the bits that fp32 has no place for
        assert o != 0 or dropped == 0x10000000
        near += abs(dropped - 0x10000000) <= 8
    assert near >= len(cases) * 2 // 3
    q = check(len(cases), N, bits, w, s, (0, 0, 0))
    for i in range(len(cases)):                                      # the members did share a cluster
        assert len(set(q["idx"][i][member[i]])) == 1


# last and first row length of every shape; 8192 columns: 512 rows and more than that
@pytest.mark.parametrize("M,N,bits", [(9, 896, 4), (9, 1024, 2), (9, 1152, 3), (9, 2048, 4), (9, 2176, 3), (5, 6144, 4), (5, 6272, 3),
                                      (512, 6272, 3), (513, 6272, 4), (513, 8192, 2), (5, 8320, 4), (5, 11776, 4), (5, 11904, 3), (5, 12288, 2)])
def test_shapes(M, N, bits):
    import gen
    check(M, N, bits, gen.make_weights(M, N, N + bits), gen.make_sens(M, N, N + bits))
