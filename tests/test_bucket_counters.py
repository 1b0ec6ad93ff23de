"""Where the k-means kernel counts its buckets (csrc/sqllm_buckets.h, compiled for the CPU): 4096 words of two counters each, of which a thread
of the scan owns eight neighbours."""
import numpy as np
import pytest

import host_split

BUCKETS, BANKS = 8192, 64


@pytest.fixture(scope="module")
def words():
    return np.array([host_split.library().counter(v) for v in range(BUCKETS // 2)])


def test_every_pair_of_buckets_has_a_word_of_its_own(words):
    assert np.array_equal(np.sort(words), np.arange(BUCKETS // 2))


def test_the_words_of_a_thread_stay_together(words):
    block = words.reshape(-1, 8)
    assert (block[:, :1] % 8 == 0).all() and np.array_equal(block, block[:, :1] + np.arange(8))


@pytest.mark.parametrize("levels", [np.arange(-8, 8), np.concatenate([np.arange(-8, 0), np.arange(1, 9)]), np.arange(-4, 4)])
@pytest.mark.parametrize("scale", [2.0 ** -9, 2.0 ** -6, 1.0, 3.0])
def test_levels_of_a_quantiser_are_counted_in_many_banks(words, levels, scale):
    bits = (levels * scale).astype(np.float16).view(np.uint16)
    key = np.where(bits & 0x8000, ~bits, bits | 0x8000).astype(np.uint16).astype(int)
    key -= key.min()
    shift = max(0, int(key.max() | 1).bit_length() - 13)
    v = key >> shift >> 1
    plain, spread = np.unique(v % BANKS).size, np.unique(words[v] % BANKS).size
    assert spread >= 2 * min(plain, 3), (plain, spread)              # levels at powers of two: one or two banks as they lie
