"""The batch kernel where its split can go wrong: the row counts at which the rows and waves per workgroup change, a last row group of one
row, fewer windows than dense waves, rows whose nonzeros fill many windows (what the sparse waves leave over is shared by all waves), every
batch size with and without a dense term, and an infinite activation, which must stay with the rows that share a 16-row tile with its
nonzero.  Bounds: 2e-3 sum |W||x| against the fp64 oracle, plus half the spacing of subnormal results."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
TOL = 2e-3


def check(y, ref, absdot, what):
    err = np.abs(y.cpu().numpy().view(np.float16).astype(np.float64) - ref)
    assert (err <= TOL * absdot + 2.0 ** -25).all(), (what, float(np.max(err / (TOL * absdot + 2.0 ** -25))))


@pytest.mark.parametrize("M,N,bits,B", [(4096, 128, 3, 16), (4097, 256, 4, 5), (8192, 384, 2, 7), (8193, 1024, 3, 13), (17, 5120, 4, 8),
                                        (33, 640, 2, 3), (1, 28672, 3, 16)])
def test_row_counts_where_the_split_changes(M, N, bits, B):
    import paper_2306_07629_amd as sq
    print(f"batch M={M} N={N} bits={bits} B={B}", flush=True)
    for frac, skew in ((0.0, None), (0.01, (0.1, 0.5))):
        L = gen.make_layer(M, N, bits, frac=frac, skew=skew, B=B, seed=M + N + B)
        D = sq.DeviceLayer(L)
        ref, absdot = oracle.layer_matvec(L)
        check(D.matvec(), ref, absdot, ("fused", frac))


@pytest.mark.parametrize("M,N,bits,B", [(8209, 384, 4, 5), (8209, 640, 4, 6), (8209, 1152, 4, 7), (8225, 896, 4, 8), (8209, 768, 4, 13), (8225, 1152, 4, 16),
                                        (8209, 384, 3, 13), (8209, 640, 3, 14), (8225, 1152, 2, 15), (8209, 1024, 3, 16)])
def test_more_workgroups_than_units(M, N, bits, B):
    """workgroups that share a unit and workgroups that cannot (4 bits from 6 columns on, from 8 without a sparse term); 13 columns and
    more request activations one window ahead"""
    import paper_2306_07629_amd as sq
    print(f"beyond the units M={M} N={N} bits={bits} B={B}", flush=True)
    for frac in (0.0, 0.02):
        L = gen.make_layer(M, N, bits, frac=frac, skew=(0.1, 0.5) if frac else None, B=B, seed=M + N + B)
        ref, absdot = oracle.layer_matvec(L)
        check(sq.DeviceLayer(L).matvec(), ref, absdot, ("fused", frac))


@pytest.mark.parametrize("B", list(range(2, 17)))
def test_heavy_rows_fill_many_windows(B):
    """two full rows of 6144 columns (48 windows each) in one workgroup, neighbours empty or with a few nonzeros"""
    import torch
    import paper_2306_07629_amd as sq
    M, N, bits = 50, 6144, 3
    print(f"heavy B={B}", flush=True)
    L = gen.make_layer(M, N, bits, frac=0.0, skew=None, B=B, seed=B)
    rng = np.random.default_rng(B)
    counts = rng.integers(0, 40, M)
    counts[[3, 20]] = N
    counts[[4, 15, 16, 49]] = 0
    rowptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    cols = np.concatenate([np.sort(rng.choice(N, c, replace=False)) for c in counts]).astype(np.int32)
    vals = (rng.standard_normal(cols.size) * 0.1).astype(np.float16).view(np.uint16)
    L.rowptr, L.cols, L.vals, L.nnz = rowptr, cols, vals, int(cols.size)
    D = sq.DeviceLayer(L)
    ref, absdot = oracle.matvec(M, N, bits, B, L.qidx, L.lut, rowptr, cols, vals, L.x)
    y = D.matvec().clone()
    check(y, ref, absdot, "fused")
    assert torch.equal(D.matvec(), y)                                # a fixed order of additions
    zero = np.zeros_like(L.lut)
    ref, absdot = oracle.matvec(M, N, bits, B, L.qidx, zero, rowptr, cols, vals, L.x)
    check(D.csr_spmv(), ref, absdot, "sparse alone")


# (M, N, bits, windows the sparse waves take alone): two, two, four and three sparse waves of six windows each
SHARED = [(50, 6144, 3, 12), (4113, 2048, 3, 12), (8209, 2048, 3, 24), (8209, 2048, 4, 18)]


@pytest.mark.parametrize("M,N,bits,alone", SHARED)
@pytest.mark.parametrize("B", [6, 13, 16])
@pytest.mark.parametrize("group", [0, 1])                            # the row group that holds the heavy rows
def test_every_shared_window_counts_once(M, N, bits, alone, B, group):
    """fused calls whose workgroups hold as many windows as the sparse waves take alone, one more, and many more, which all waves share.
    Tables of zeros, and values and activations of +1 and -1: every sum is a whole number that fp16 holds, and a nonzero lost or counted
    twice changes it"""
    import torch
    import host_split
    import paper_2306_07629_amd as sq
    print(f"shared windows M={M} N={N} bits={bits} B={B} group={group}", flush=True)
    RG, _, ND, NS, _ = host_split.batch_split(M, N, bits, B, True, True)
    assert ND > 0 and NS * 6 == alone
    rng = np.random.default_rng(M + B + group)
    for windows in (alone, alone + 1, alone + 27):
        block = 16 * RG * (M // (16 * RG) // 2)                      # a workgroup in the middle, and the last one, which may be short
        counts = rng.integers(0, 4, M)
        for r0 in (block, M - 1 - (M - 1) % (16 * RG)):
            heavy, other = (r0 + 16 * group, r0) if r0 + 16 * group < M and group < RG else (r0, r0)
            counts[r0:min(r0 + 16 * RG, M)] = 0
            # one window in the other row group (if there is one); in the heavy one rows whose sum is no multiple of 128 columns
            if other != heavy:
                counts[other] = 1
            total = 128 * (windows - (1 if other != heavy else 0)) - 37
            for k in range(min(16, M - heavy)):
                counts[heavy + k] = min(total, N)
                total -= counts[heavy + k]
        rowptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
        cols = np.concatenate([np.sort(rng.choice(N, c, replace=False)) for c in counts]).astype(np.int32)
        sign = lambda shape: (2 * rng.integers(0, 2, shape) - 1)
        vals, x = sign(cols.size), sign((N, B))
        want = np.zeros((M, B), dtype=np.int64)
        np.add.at(want, np.repeat(np.arange(M), counts), vals[:, None] * x[cols])
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
        y = torch.zeros((M, B), dtype=torch.float16, device="cuda")
        sq.sqllm_dense_sparse_matvec(M, N, bits, cols.size, B, dev(rng.integers(0, 256, M * N * bits // 8).astype(np.uint8)),
                                     torch.zeros((M, 1 << bits), dtype=torch.float16, device="cuda"), dev(rowptr), dev(cols),
                                     dev(vals.astype(np.float16)), dev(x.astype(np.float16)), y)
        assert np.abs(want).max() <= 2048
        assert np.array_equal(y.cpu().numpy().astype(np.int64), want), windows


@pytest.mark.parametrize("B", [2, 5, 8, 16])
@pytest.mark.parametrize("M", [64, 5000])                            # 16 and 32 rows per workgroup
def test_infinite_activation_stays_in_its_tile(M, B):
    import torch
    import paper_2306_07629_amd as sq
    N = 256
    print(f"inf M={M} B={B}", flush=True)
    rowptr = np.arange(M + 1, dtype=np.int32)
    cols = np.full(M, 7, dtype=np.int32)
    cols[20] = 9                                                     # the only nonzero of the column whose activations are infinite
    x = np.ones((N, B), dtype=np.float16)
    x[9] = np.inf
    x[11] = np.nan                                                   # no nonzero reads it
    y = torch.zeros((M, B), dtype=torch.int16, device="cuda")
    dev = lambda a: torch.from_numpy(a).cuda()
    sq.sqllm_csr_spmv(M, N, M, B, dev(rowptr), dev(cols), dev(np.full(M, 0x3C00, np.int16)), dev(x.view(np.int16)), y)
    got = y.cpu().numpy().view(np.float16)
    other = np.r_[0:16, 32:M]
    assert np.array_equal(got[other], np.ones((M - 16, B), np.float16))
    assert np.isinf(got[20]).all()


@pytest.mark.parametrize("M,B", [(4096, 16), (65536, 5)])            # 16 and 32 rows per workgroup
def test_nonzeros_up_to_the_largest_position(M, B):
    """2^31 - 1 nonzeros (13 GB; entries of one row and column add up): the last windows begin less than 128 positions before the end of
    the 32-bit range.  Small integers, so every sum is exact."""
    import torch
    import paper_2306_07629_amd as sq
    N, nnz = 128, 2 ** 31 - 1
    print(f"largest nnz M={M} B={B}", flush=True)
    rowptr = torch.minimum(torch.arange(M + 1, dtype=torch.int64) * (2 ** 31 // M), torch.tensor(nnz)).to(torch.int32)
    cols = torch.full((nnz,), 3, dtype=torch.int32, device="cuda")
    vals = torch.zeros(nnz, dtype=torch.int16, device="cuda")
    first = int(rowptr[M - 1])
    for lo, hi in ((0, 2), (first - 3, first + 5), (nnz - 130, nnz)):
        vals[lo:hi] = 0x3C00
    x = torch.zeros((N, B), dtype=torch.float16, device="cuda")
    x[3] = torch.arange(1, B + 1, dtype=torch.float16)
    x[0] = x[127] = float("inf")                                     # columns that no nonzero names
    y = torch.zeros((M, B), dtype=torch.float16, device="cuda")
    sq.sqllm_csr_spmv(M, N, nnz, B, rowptr.cuda(), cols, vals, x, y)
    want = torch.zeros((M, B), dtype=torch.float16)
    want[0], want[M - 2], want[M - 1] = 2 * x[3].cpu(), 3 * x[3].cpu(), 135 * x[3].cpu().float()
    got = y.cpu()
    del cols, vals
    torch.cuda.empty_cache()
    assert torch.equal(got, want)
