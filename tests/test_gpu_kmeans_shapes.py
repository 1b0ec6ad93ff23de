"""All shapes of the k-means kernel with every form of its rows: the shapes that only matrices of many rows take, with rows that fill one
bucket, many buckets or a few keys only, and with weights of 128 and more.  A few distinct rows are repeated until the matrix has as many as
the shape asks for; the distinct ones are checked bit for bit against the quantiser oracle and the others against them."""
import numpy as np
import pytest

import host_split
import oracle
from oracle import quant_oracle as qo
from test_gpu_quantize import run_gpu
from test_gpu_quantize_buckets import crowded_weights, weights

pytestmark = pytest.mark.gpu

# (M, N, bits, shape): both sides of every limit of the rule, last and first row length of the shapes
SHAPES = [(1536, 1152, 3, 4096), (1537, 1152, 4, 2048), (1537, 2048, 2, 2048), (512, 4224, 2, 11776), (513, 4224, 4, 6144), (513, 6144, 3, 6144),
          (512, 6272, 4, 11776), (513, 6272, 2, 8192), (768, 8192, 3, 8192), (769, 8192, 4, 11776), (1025, 6272, 4, 8192), (4, 11776, 3, 11776),
          (4, 11904, 4, 12288), (4, 12288, 2, 12288)]
KINDS = ["ordinary", "pruned", "constant", "levels", "neighbours", "wide rows", "one bucket", "every exponent", "edge"]


def distinct_rows(kind, D, N, rng):
    if kind == "ordinary":
        return (0.02 * rng.standard_t(4, (D, N))).astype(np.float16).view(np.uint16)
    old = {"one bucket": "narrow", "every exponent": "spread", "edge": "edge"}
    return weights(old[kind], D, N, rng) if kind in old else crowded_weights(kind.split()[0], D, N, rng)


@pytest.mark.parametrize("M,N,bits,shape", SHAPES)
@pytest.mark.parametrize("kind", KINDS)
def test_every_form_of_a_row(kind, M, N, bits, shape):
    assert host_split.library().kmeans_shape(M, N) == shape
    print(f"shape kind={kind} M={M} N={N} bits={bits}", flush=True)
    rng = np.random.default_rng(M + N + bits)
    D = 4
    w = distinct_rows(kind, D, N, rng)
    s = rng.integers(0, 65536, (D, N)).astype(np.uint16)
    s[1] = 65535
    s[2, ::2] = 0
    row = np.arange(M) % D
    copies = -(-M // D)
    counts = (0, 0, 0) if kind == "edge" else (3 * copies, 2 * copies, 7 * copies)
    w, s = np.ascontiguousarray(w[row]), np.ascontiguousarray(s[row])
    got = run_gpu(w, s, bits, *counts, 20)
    ref = qo.quantize_layer(w, s, bits, *counts, 20, rows=range(D))
    assert np.array_equal(got["rowptr"], ref["rowptr"]) and np.array_equal(got["cols"], ref["cols"]) and np.array_equal(got["vals"], ref["vals"])
    idx = oracle.unpack(M, N, bits, got["qidx"])
    for mine, theirs in ((got["iters"], ref["iters"]), (got["lut"], ref["lut"]), (idx, ref["idx"])):
        assert np.array_equal(mine[:D], theirs[:D])
        assert np.array_equal(mine, mine[:D][row])
