"""The plain arithmetic of the batch kernel (csrc/sqllm_batch_split.h), compiled for the CPU with signed overflow made fatal: windows of
nonzeros up to the largest position the interface accepts (nnz < 2^31), against the definition in Python's integers, and the split of
rows and waves over the workgroups."""
import pytest

import host_split

TOP = 2 ** 31 - 1


@pytest.fixture(scope="module")
def split():
    return host_split.library()


@pytest.mark.parametrize("first,end", [(0, 1), (0, 128), (3, 132), (7, 7), (0, TOP), (TOP - 1, TOP), (TOP - 127, TOP), (TOP - 200, TOP),
                                       (TOP - 128 * 40, TOP), (TOP - 5000, TOP - 90)])
def test_windows_cover_a_row_group_and_read_nothing_else(split, first, end):
    n = split.count(first, end)
    assert n == -(-(end - first) // 128)
    for f in sorted({0, 1, n // 2, n - 2, n - 1} & set(range(n))) if n > 64 else range(n):
        p0 = first + 128 * f
        last = p0 + split.rest(p0, end)
        assert p0 <= last == end - 1                                 # the kernel reads positions p0 + min(k, rest), k < 128
        reads = [p0 + min(k, split.rest(p0, end)) for k in range(128)]
        assert first <= min(reads) and max(reads) < end


@pytest.mark.parametrize("base", [0, 1000, TOP - 700])
def test_row_bits_name_the_positions_of_the_row(split, base):
    ptr = [base + o for o in (0, 0, 5, 37, 37, 160, 161, 500, 700)]  # eight rows, empty ones among them
    for p0 in [base + 128 * f for f in range(split.count(ptr[0], ptr[-1]))]:
        for q in range(4):
            owner = [next((r for r in range(8) if ptr[r] <= p0 + 32 * q + k < ptr[r + 1]), None) for k in range(32)]
            for r in range(8):
                assert split.row_bits(ptr[r], ptr[r + 1], p0, q) == sum(1 << k for k in range(32) if owner[k] == r), (p0, q, r)
    assert split.row_bits(0, base, base, 0) == 0                     # rows far in front of and far behind the window
    assert split.row_bits(TOP, TOP, 0, 3) == 0


UNIT_LDS, UNITS = 160 * 1024, 256


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("B", range(2, 17))
def test_split_fills_the_units_it_says_it_fills(split, bits, B):
    for M in (1, 16, 200, 4096, 4097, 8192, 8193, 22016, 10 ** 6, TOP):
        for N in (128, 384, 640, 1024, 8192, 28672):
            for dense, sparse in ((1, 1), (1, 0), (0, 1)):
                rg, blocks, nd, ns, lds = host_split.batch_split(M, N, bits, B, dense, sparse)
                assert blocks * 16 * rg >= M > (blocks - 1) * 16 * rg
                assert (nd > 0) == bool(dense) and nd <= N // 128    # a dense wave without a window would read one that is not its own
                assert (ns > 0) == bool(sparse) and 1 <= nd + ns <= 8
                assert lds <= UNIT_LDS
                # four waves per SIMD of 512 registers: two workgroups of eight waves fit a unit's four
                if rg == 2 and B >= 13:
                    assert split.waves_per_simd(rg, B) == 4
                if dense and blocks > UNITS and N >= 1024:
                    shared = nd == 4
                    assert not shared or 2 * lds <= UNIT_LDS
                    assert shared == (bits < 4 or (B <= 5 if sparse else B <= 11 and B != 8)), (bits, B, sparse)
                    if not shared:                                   # one workgroup keeps the unit busy
                        assert nd + ns == 8 and nd >= 5
