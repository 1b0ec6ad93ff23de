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


@pytest.mark.parametrize("N", [128, 16384])                              # four and eight rows to a workgroup
@pytest.mark.parametrize("fused", [False, True])
def test_nonzeros_up_to_the_largest_position(N, fused):
    """2^31 - 1 nonzeros (13 GB; entries of one row and column add up): the last workgroup's batches begin less than a round before the end
    of the 32-bit range, and its last rows end inside a batch.  Small integers, so every sum is exact."""
    import torch
    import paper_2306_07629_amd as sq
    M, nnz = 4096, 2 ** 31 - 1
    print(f"largest nnz N={N} fused={fused}", flush=True)
    rowptr = torch.minimum(torch.arange(M + 1, dtype=torch.int64) * 2 ** 19, torch.tensor(nnz))
    rowptr[M - 8:M] = nnz - torch.tensor([3000, 700, 131, 130, 70, 69, 2, 1])   # the last eight rows hold 2300, 569, 1, 60, 1, 67, 1 and 1
    cols = torch.full((nnz,), 3, dtype=torch.int32, device="cuda")
    vals = torch.zeros(nnz, dtype=torch.int16, device="cuda")
    vals[:2] = 0x3C00
    vals[nnz - 2900:] = 0x3C00
    x = torch.zeros((N, 1), dtype=torch.float16, device="cuda")
    x[3] = 1
    y = torch.zeros((M, 1), dtype=torch.float16, device="cuda")
    if fused:
        qidx = torch.zeros(M * N * 2 // 8, dtype=torch.uint8, device="cuda")
        lut = torch.zeros((M, 4), dtype=torch.float16, device="cuda")
        sq.sqllm_dense_sparse_matvec(M, N, 2, nnz, 1, qidx, lut, rowptr.int().cuda(), cols, vals, x, y)
    else:
        sq.sqllm_csr_spmv(M, N, nnz, 1, rowptr.int().cuda(), cols, vals, x, y)
    want = torch.zeros((M, 1))
    want[0] = 2
    want[M - 8:, 0] = torch.tensor([2200., 569, 1, 60, 1, 67, 1, 1])
    got = y.cpu()
    del cols, vals
    torch.cuda.empty_cache()
    assert torch.equal(got, want.half())
