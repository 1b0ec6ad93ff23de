"""The k-means kernel's counting sort where it can go wrong: rows whose keys fill one bucket, all buckets or a few distinct keys only,
weights of 128 and more (sums beyond 64 bits), the widths at which the threads per row change, and rows that are extracted entirely.
Bit-exact against the quantiser oracle."""
import numpy as np
import pytest

from oracle import quant_oracle as qo
from test_gpu_quantize import compare, run_gpu

pytestmark = pytest.mark.gpu


def weights(kind, M, N, rng):
    z = rng.standard_normal((M, N))
    w = {"narrow": 1.0 + 1e-3 * z,                       # two or three buckets hold everything
         "wide": 20000.0 * np.tanh(z),                   # |w| >= 128: the two-word sums
         "edge": np.where(z > 0, 128.0, -127.9375),      # just at the limit of the one-word sums
         "tiny": 2.0 ** -24 * np.round(3 * z),           # subnormals, zeros
         "spread": np.sign(z) * 2.0 ** rng.uniform(-24, 15, (M, N))}[kind]   # every exponent: shift at its largest
    out = w.astype(np.float16).view(np.uint16).copy()
    out[0, ::3] = 0x8000                                 # -0 and +0 side by side
    out[0, 1::3] = 0
    return out


@pytest.mark.parametrize("kind", ["narrow", "wide", "edge", "tiny", "spread"])
@pytest.mark.parametrize("N,bits", [(128, 3), (4096, 4), (4224, 2), (16384, 3), (16512, 4)])
def test_bucket_layouts_and_sum_widths(kind, N, bits):
    M = 5
    print(f"buckets kind={kind} N={N} bits={bits}", flush=True)
    rng = np.random.default_rng(N + bits)
    w = weights(kind, M, N, rng)
    s = rng.integers(0, 65536, (M, N)).astype(np.uint16)
    if kind == "narrow":
        s[1, :] = 65535                                  # largest sums
    counts = (0, 0, 0) if kind == "edge" else (7, 5, 9)
    compare(M, N, bits, run_gpu(w, s, bits, *counts, 25), qo.quantize_layer(w, s, bits, *counts, 25))


def test_rows_extracted_entirely():
    M, N, bits = 4, 256, 3
    rng = np.random.default_rng(5)
    w = rng.standard_normal((M, N)).astype(np.float16)
    w[1] = np.abs(w[1]) + 100                            # every weight of the row is among the largest of the matrix
    s = rng.integers(1, 500, (M, N)).astype(np.uint16)
    got = run_gpu(w.view(np.uint16), s, bits, 0, N, 0, 10)
    ref = qo.quantize_layer(w.view(np.uint16), s, bits, 0, N, 0, 10)
    assert int(ref["rowptr"][2] - ref["rowptr"][1]) == N
    compare(M, N, bits, got, ref)


@pytest.mark.parametrize("N,bits", [(128, 2), (4096, 3), (11008, 4), (16384, 2), (28672, 3)])
def test_limit_of_the_one_word_sums(N, bits):
    """one row on each side of every limit: 127.875 is the largest weight of a row with one-word sums, 127.9375 and -128 are the first of
    the two-word sums; largest sensitivities, so the sums themselves reach their limits"""
    M = 9
    print(f"one-word limit N={N} bits={bits}", flush=True)
    rng = np.random.default_rng(N)
    top, first = 127.875, 127.9375
    sign = np.where(rng.random(N) < 0.5, -1.0, 1.0)
    w = np.array([np.full(N, top), np.full(N, first), np.full(N, 128.0), np.full(N, -first), np.full(N, -128.0), top * sign, first * sign,
                  128.0 * sign, np.where(rng.random(N) < 0.3, rng.uniform(-100, 100, N), top * sign)]).astype(np.float16)
    s = np.full((M, N), 65535, dtype=np.uint16)
    s[8] = rng.integers(0, 65536, N)
    w = w.view(np.uint16)
    compare(M, N, bits, run_gpu(w, s, bits, 0, 0, 0, 12), qo.quantize_layer(w, s, bits, 0, 0, 0, 12))


def crowded_weights(kind, M, N, rng):
    """rows with many words of few keys: some buckets hold kHeavy = 256 words and more, next to buckets of a few"""
    z = rng.standard_normal((M, N))
    if kind == "pruned":                                 # nine tenths zeros, of both signs
        w = np.where(rng.random((M, N)) < 0.9, np.where(z > 1, -0.0, 0.0), 0.02 * z)
    elif kind == "constant":
        w = np.full((M, N), 0.01)
    elif kind == "levels":                               # as from a 4-bit quantiser
        w = np.clip(np.round(3 * z), -8, 7) * 2.0 ** -6
    elif kind == "neighbours":                           # keys that share a heavy bucket: the row's range makes buckets of 2^shift keys
        w = np.float16(0.75) + np.clip(np.round(6 * z), -14, 14) * 2.0 ** -11
        w[:, ::97] = 1e-3 * z[:, ::97]
        w[:, 1::211] = -2.0
    else:                                                # "wide": the same with |w| >= 128, the two-word sums
        w = np.float16(300.0) + np.clip(np.round(6 * z), -14, 14) * 2.0 ** -2
        w[:, ::97] = 1e-3 * z[:, ::97]
        w[:, 1::211] = -20000.0
    return w.astype(np.float16).view(np.uint16)


@pytest.mark.parametrize("kind", ["pruned", "constant", "levels", "neighbours", "wide"])
@pytest.mark.parametrize("N,bits", [(128, 2), (256, 4), (4096, 3), (4224, 4), (16384, 2), (16512, 3), (28672, 4)])
def test_buckets_that_hold_much_of_a_row(kind, N, bits):
    M = 4
    print(f"crowded kind={kind} N={N} bits={bits}", flush=True)
    rng = np.random.default_rng(N * bits)
    w = crowded_weights(kind, M, N, rng)
    s = rng.integers(0, 65536, (M, N)).astype(np.uint16)
    s[1] = 65535
    s[2, ::2] = 0
    counts = (3, 2, 7)
    compare(M, N, bits, run_gpu(w, s, bits, *counts, 32), qo.quantize_layer(w, s, bits, *counts, 32))


@pytest.mark.parametrize("M,N,bits", [(2048, 11008, 4), (512, 28672, 4)])
def test_pruned_rows_take_no_longer_than_a_few_ordinary_ones(M, N, bits):
    """An update looks at a handful of words of a bucket, however many it holds: read through, the bucket of the zeros made a pruned matrix
    37 and 58 times as slow as an ordinary one; bisected it takes twice as long.  Bound: 6."""
    import torch
    import paper_2306_07629_amd as sq
    print(f"pruned time M={M} N={N}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    z = torch.randn((M, N), generator=g, device="cuda") * 0.02
    s = torch.randint(0, 30000, (M, N), generator=g, device="cuda", dtype=torch.int16)
    times = []
    for w in (z, torch.where(torch.rand((M, N), generator=g, device="cuda") < 0.9, torch.zeros_like(z), z)):
        w = w.half()
        sq.quantize_layer(w, s, bits, 10, 10, 10)
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        best = float("inf")
        for _ in range(5):
            t0.record()
            sq.quantize_layer(w, s, bits, 10, 10, 10)
            t1.record()
            t1.synchronize()
            best = min(best, t0.elapsed_time(t1))
        times.append(best)
    assert times[1] <= 6 * times[0], times
