"""The sparse term of a planned one-column call is added lane by lane to the partial sums of the dense term.  Row counts around the 16
entries of a group, the batches of a slot and the rounds of the overflow, with sums that are whole numbers: every entry counts once, in
its own row.  And an infinite activation in column 0, the column that the padding of the groups names."""
import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu


def hand(N, bits, counts, weight, seed):
    rng = np.random.default_rng(seed)
    M, K = len(counts), 1 << bits
    idx = rng.integers(0, K, size=(M, N), dtype=np.uint8)
    lut = np.full((M, K), weight, dtype=np.float16)
    rowptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    cols = np.concatenate([1 + np.sort(rng.choice(N - 1, c, replace=False)) for c in counts if c]).astype(np.int32)   # never column 0
    vals = rng.integers(1, 4, size=cols.size).astype(np.float16)
    x = rng.integers(1, 3, size=(N, 1)).astype(np.float16)
    return idx, lut, rowptr, cols, vals, x


@pytest.mark.parametrize("N", [256, 4096, 8192, 16384, 22528])           # 1, 2, 4, 8 and 11 waves; from 8 on eight rows to a workgroup
@pytest.mark.parametrize("bits", [2, 3, 4])
def test_every_entry_counts_once_in_its_own_row(N, bits):
    import paper_2306_07629_amd as sq
    top = min(N - 1, 12000)
    counts = [0, 1, 15, 16, 17, 31, 32, 33, 0, 0, 63, 64, 65, min(top, 700), 0, 2, top, 1, 5, 16, 240, min(top, 255)]   # 22 rows: the last quad is half
    idx, lut, rowptr, cols, vals, x = hand(N, bits, counts, 0.0, seed=N + bits)
    L = gen.hand_layer(idx, lut, bits, rowptr, cols, vals, x)
    D = sq.DeviceLayer(L).build_plan()
    y = D.matvec().cpu().numpy().view(np.float16).astype(np.float64)[:, 0]
    prod = vals.astype(np.float64) * x[cols, 0].astype(np.float64)
    want = np.array([prod[rowptr[i]:rowptr[i + 1]].sum() for i in range(len(counts))])
    # whole numbers below 2^24: fp32 sums are exact in any order, and y is their rounding to fp16
    assert np.array_equal(y, want.astype(np.float16).astype(np.float64))
    alone = D.y.clone()
    D.y.zero_()
    sq.sqllm_dense_sparse_matvec_multi([D.descriptor(), sq.DeviceLayer(L).build_plan().descriptor()])
    assert np.array_equal(D.y.cpu().numpy(), alone.cpu().numpy())


@pytest.mark.parametrize("N", [256, 8192, 22528])
def test_padding_of_the_groups_does_not_meet_an_infinite_activation(N):
    import paper_2306_07629_amd as sq
    counts = [3, 0, 17, 1, 5, 200, 0, 9, 33]
    idx, lut, rowptr, cols, vals, x = hand(N, 3, counts, 0.5, seed=N)
    x[0, 0] = np.inf
    D = sq.DeviceLayer(gen.hand_layer(idx, lut, 3, rowptr, cols, vals, x)).build_plan()
    y = D.matvec().cpu().numpy().view(np.float16).astype(np.float64)[:, 0]
    assert (y == np.inf).all()                                            # 0.5 * inf plus finite terms; 0 * inf would be NaN
