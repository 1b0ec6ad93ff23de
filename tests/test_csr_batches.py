"""The plain arithmetic of the one-column kernel over the CSR arrays (csrc/sqllm_csr.h), compiled for the CPU with signed overflow made
fatal: what the lanes read and the rows they add to, for nonzeros up to the largest position the interface accepts (nnz < 2^31), against
the definition in Python's integers."""
import pytest

import host_split

TOP = 2 ** 31 - 1


@pytest.mark.parametrize("R", [4, 8])
@pytest.mark.parametrize("base", [0, 1000, TOP - 700, TOP - 6000])
@pytest.mark.parametrize("ends", [(0, 0, 5, 37, 37, 160, 161, 500, 700), (0, 1, 64, 65, 128, 128, 129, 640, 641), (0, 0, 0, 0, 0, 0, 0, 0, 1),
                                  (0, 63, 63, 64, 600, 610, 611, 612, 700)])
def test_every_nonzero_is_read_once_and_added_to_its_own_row(R, base, ends):
    rp = [base + e for e in ends[:R + 1]]
    first, end = rp[0], rp[R]
    n = host_split.library().batches(first, end)
    assert n == -(-(end - first) // 64)
    if n == 0:
        return                                                       # nothing is read
    seen = []
    for b in range(n + 8 * 17):                                      # a round asks for up to eight batches of each of 16 waves, surplus ones included
        at, row = host_split.csr_positions(first, end, b), host_split.csr_rows(rp, b)
        for lane in range(64):
            p = first + 64 * b + lane
            assert at[lane] == min(p, end - 1)
            if p < end:
                assert rp[row[lane]] <= p < rp[row[lane] + 1]
                seen.append(p)
            else:
                assert row[lane] >= R
    assert seen == list(range(first, end))


def test_all_nonzeros_in_one_row():
    """the largest row that the interface accepts, and its last batches"""
    n = host_split.library().batches(0, TOP)
    assert n == 2 ** 25
    for rp in ([0, 0, TOP, TOP, TOP], [0] * 8 + [TOP]):
        R = len(rp) - 1
        own = next(i for i in range(R) if rp[i + 1] == TOP)
        assert (host_split.csr_rows(rp, n - 1)[:63] == own).all() and host_split.csr_rows(rp, n - 1)[63] >= R
        assert (host_split.csr_rows(rp, n + 135) >= R).all()
    assert host_split.csr_positions(0, TOP, n - 1).max() == TOP - 1 == host_split.csr_positions(0, TOP, n + 135).min()
