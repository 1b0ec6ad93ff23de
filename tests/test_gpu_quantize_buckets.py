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
