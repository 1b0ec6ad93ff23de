"""Where the offline pass may write the CSR entries of a row (csrc/sqllm_csr.h, compiled for the CPU with signed overflow made fatal).  They
are counted by one kernel and written by another; should the weights change in between -- a caller that does not order its streams -- the
second may find more of them than the first did, and none of those may be written past the row or past the arrays."""
import os

import pytest

import host_split

TOP = 2 ** 31 - 1


@pytest.mark.parametrize("first,row_end,capacity", [(0, 5, 5), (0, 5, 100), (7, 7, 100), (700, 732, 1000), (TOP - 40, TOP - 1, TOP - 1), (TOP - 8, TOP, TOP)])
def test_all_counted_entries_have_room_and_no_others(first, row_end, capacity):
    room = host_split.library().has_room
    assert all(room(p, row_end, capacity) for p in range(first, row_end))
    assert not any(room(p, row_end, capacity) for p in range(row_end, min(row_end + 40, TOP + 1)))


@pytest.mark.parametrize("p,row_end,capacity", [(5, 9, 5), (5, 9, 0), (0, 9, 0), (-1, 9, 9), (-TOP - 1, 9, 9), (3, -1, 9), (TOP, TOP, TOP), (-3, -1, 9)])
def test_none_is_written_outside_the_arrays(p, row_end, capacity):
    assert not host_split.library().has_room(p, row_end, capacity)


def test_the_kernel_asks_before_it_writes():
    src = open(os.path.join(host_split.CSRC, "sqllm_quant.hip")).read()
    body = src[src.index("auto write_entries"):]
    body = body[:body.index("};")]
    ask = body.index("if (csr_has_room(entry, end, capacity)) {")
    assert src.count("cols[") == 1 and src.count("vals[") == 1       # the only place that writes them
    assert ask < body.index("cols[entry] = j;") < body.index("vals[entry] = wrow[j];") < body.index("}", ask)
