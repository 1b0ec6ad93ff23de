"""The sparse term straight from the CSR arrays, one activation column: every lane adds to its own partial sums of the workgroup's rows.
Row ends at every place of a 64-entry batch, batches in one row and in several, rounds that all waves share, with sums that are whole
numbers: every entry counts once, in its own row."""
import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [256, 4096, 16384, 22528])                 # four rows to a workgroup; from 16384 columns on eight
@pytest.mark.parametrize("first", [0, 1, 63, 64, 65, 600])               # nonzeros of row 0: where the other rows end in their batches
def test_every_entry_counts_once_in_its_own_row(N, first):
    import paper_2306_07629_amd as sq
    rng = np.random.default_rng(N + first)
    top = min(N, 9000)
    counts = [min(first, N), 0, 1, 62, 2, 64, 0, 63, 0, 0, 0, 128, min(top, 129), 3, top, 1, 5]
    M = len(counts)
    idx = rng.integers(0, 8, size=(M, N), dtype=np.uint8)
    lut = np.zeros((M, 8), dtype=np.float16)
    rowptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    cols = np.concatenate([np.sort(rng.choice(N, c, replace=False)) for c in counts if c]).astype(np.int32)
    vals = rng.integers(1, 4, size=cols.size).astype(np.float16)
    x = rng.integers(1, 3, size=(N, 1)).astype(np.float16)
    D = sq.DeviceLayer(gen.hand_layer(idx, lut, 3, rowptr, cols, vals, x))
    prod = vals.astype(np.float64) * x[cols, 0].astype(np.float64)
    want = np.array([prod[rowptr[i]:rowptr[i + 1]].sum() for i in range(M)]).astype(np.float16)   # exact in fp32, whatever the order
    fused = D.matvec().cpu().numpy().view(np.float16)[:, 0]
    assert np.array_equal(fused, want)
    alone = D.csr_spmv().cpu().numpy().view(np.float16)[:, 0]
    assert np.array_equal(alone, want)
    D.y.zero_()
    sq.sqllm_dense_sparse_matvec_multi([D.descriptor(), sq.DeviceLayer(gen.hand_layer(idx, lut, 3, rowptr, cols, vals, x)).descriptor()])
    assert np.array_equal(D.y.cpu().numpy().view(np.float16)[:, 0], want)
