"""Host-side check that the batch kernel never reads past the end of an input array: every address range it touches, re-computed from the
clamping formulas it uses (rows past M, windows past a wave's last one, surplus lanes of an index load, nonzeros past a row group, the
dwords that hold a gathered row of x), lies inside the array."""
import numpy as np
import pytest

import host_split
from test_read_bounds import SHAPES, rowptr_for

LANES = np.arange(64)


def row_reads(col, B):
    """(first byte, bytes) of the loads that fetch the row of x of a column: whole rows of 8 and 16 columns in pieces of 16 bytes, else from
    the dword on in which the row begins, in dwords"""
    first = col * 2 * B & ~3
    return first, 2 * B if B in (8, 16) else 4 * ((B + 1) // 2)


def batch_kernel_reads(M, N, bits, B, rowptr, cols):
    nwin, nnz = N // 128, int(rowptr[-1])
    RG, groups, ND, _, _ = host_split.batch_split(M, N, bits, B, True, nnz > 0)   # the launcher's own rule
    R, K = 16 * RG, 1 << bits
    heavy = int(np.argmax(np.diff(rowptr))) // R
    for block in sorted({0, groups - 1, groups // 2, heavy}):
        r0 = block * R
        rows = np.minimum(r0 + np.arange(R), M - 1)
        yield "lut", int(rows.min()) * 2 * K, (int(rows.max()) + 1) * 2 * K
        gp, ge = [], []
        for rg in range(RG):
            lo = np.minimum(r0 + 16 * rg + np.arange(16), M)
            hi = np.minimum(r0 + 16 * rg + np.arange(16) + 1, M)
            if nnz:
                yield "rowptr", 4 * int(lo.min()), 4 * int(hi.max()) + 4
            gp.append(int(rowptr[lo[0]]))
            ge.append(int(rowptr[hi[15]]))
        p = np.minimum(LANES, 16 * bits - 1)
        for wave in range(ND):
            last_t = wave + (nwin - 1 - wave) // ND * ND
            t = wave
            while t < nwin + 3 * ND:
                tt = min(t, last_t)
                for rg in range(RG):
                    row = np.minimum(r0 + 16 * rg + p // bits, M - 1).astype(np.int64)
                    off = row * (N * bits // 8) + (p % bits) * 16 + tt * bits * 16
                    yield "qidx", int(off.min()), int(off.max()) + 16
                yield "x", tt * 256 * B, (tt + 1) * 256 * B          # 64 lanes times 4 B bytes
                t += ND
        for rg in range(RG):
            for f in range((ge[rg] - gp[rg] + 127) // 128):
                q = np.minimum(gp[rg] + 128 * f + np.arange(128), ge[rg] - 1)
                yield "cols", 4 * int(q.min()), 4 * int(q.max()) + 4
                yield "vals", 2 * int(q.min()), 2 * int(q.max()) + 2
                first, n = row_reads(cols[q].astype(np.int64), B)
                yield "x", int(first.min()), int(first.max()) + n


@pytest.mark.parametrize("B", range(2, 17))
def test_a_gathered_row_is_read_whole_and_inside_the_array(B):
    N = 128
    for col in range(N):
        first, n = row_reads(col, B)
        assert first % 4 == 0 and 0 <= first <= col * 2 * B          # whole row
        assert col * 2 * B + 2 * B <= first + n <= 2 * N * B         # and no byte past the last row
        assert n - 2 * B == 2 * (B % 2)                              # at most one foreign half


@pytest.mark.parametrize("M,N,bits,B", [s for s in SHAPES if s[3] > 1] + [(4096, 128, 3, 16), (4097, 256, 4, 5), (8193, 384, 3, 13), (8209, 768, 4, 16)])
def test_every_load_of_the_batch_kernel_stays_inside_its_array(M, N, bits, B):
    rowptr = rowptr_for(M, N, M + N + bits)
    nnz = int(rowptr[-1])
    cols = np.random.default_rng(M).integers(0, N, nnz)
    cols[:2] = (0, N - 1)
    for name, lo, hi in batch_kernel_reads(M, N, bits, B, rowptr, cols):
        size = {"x": 2 * N * B, "qidx": M * N * bits // 8, "lut": M * 2 * (1 << bits), "rowptr": 4 * (M + 1), "cols": 4 * nnz, "vals": 2 * nnz}[name]
        assert 0 <= lo and hi <= size, (name, lo, hi, size)
