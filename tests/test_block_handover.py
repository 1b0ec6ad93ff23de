"""The hand-over between the blocks of the offline pass's three passes over the matrix, in the code the compiler emits: a block's atomics and
agent-scope stores, then every wave's wait for them, the barrier, and only then the count; the last block invalidates its caches before it
reads what the others left.  (The language does not promise that order without a release that would cost 4 % of a call, so a compiler that
changes it must be noticed here.)"""
import re

import pytest

KERNELS = ["quant_hist1_kernel", "quant_hist2_kernel", "quant_count_kernel"]


def instructions(assembly, kernel):
    body = re.search(r"^_ZN5sqllm\d+%s\S*:\s.*?\n(.*?)\.Lfunc_end" % kernel, assembly, re.S | re.M)[1]
    lines = (re.sub(r"\s*;.*", "", l).strip() for l in body.split("\n"))
    return [l for l in lines if l and not l.endswith(":") and not l.startswith(".")]


def handover_is_ordered(ins):
    memory = [i for i, l in enumerate(ins) if l.startswith(("global_", "flat_", "buffer_atomic", "buffer_store"))]
    counts = [i for i in memory if ins[i].startswith("global_atomic_add") and " sc0" in ins[i]]
    if len(counts) != 1:                                             # the only atomic whose old value is asked for
        return False
    c = counts[0]
    writes = [i for i in memory if i < c and ("atomic" in ins[i] or "store" in ins[i])]
    if not writes:
        return False
    waits = [i for i in range(writes[-1], c) if ins[i].startswith("s_waitcnt") and "vmcnt(0)" in ins[i]]
    barriers = [i for i in range(writes[-1], c) if ins[i] == "s_barrier"]
    if not waits or not barriers or waits[0] > barriers[0]:
        return False
    invalidate = next((i for i in range(c, len(ins)) if ins[i].startswith("buffer_inv") and "sc1" in ins[i]), len(ins))
    return all(i < waits[0] or i == c or i > invalidate for i in memory) and invalidate < len(ins)


@pytest.mark.parametrize("kernel", KERNELS)
def test_blocks_are_counted_after_what_they_hand_over(assembly, kernel):
    assert handover_is_ordered(instructions(assembly, kernel))


@pytest.mark.parametrize("kernel", KERNELS)
def test_the_check_sees_a_missing_wait_barrier_or_invalidate(assembly, kernel):
    ins = instructions(assembly, kernel)
    c = next(i for i, l in enumerate(ins) if l.startswith("global_atomic_add") and " sc0" in l)
    last = lambda p: max(i for i in range(c) if p(ins[i]))
    wait, barrier = last(lambda l: l.startswith("s_waitcnt") and "vmcnt(0)" in l), last(lambda l: l == "s_barrier")
    write = last(lambda l: l.startswith("global_atomic") or l.startswith("global_store"))
    inv = next(i for i in range(c, len(ins)) if ins[i].startswith("buffer_inv"))
    for drop in (wait, barrier, inv):
        assert not handover_is_ordered(ins[:drop] + ins[drop + 1:])
    moved = ins[:write] + ins[write + 1:barrier + 1] + [ins[write]] + ins[barrier + 1:]
    assert not handover_is_ordered(moved)
