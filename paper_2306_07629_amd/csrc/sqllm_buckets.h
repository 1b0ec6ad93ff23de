// Plain arithmetic of the k-means kernel's counting sort.  No HIP in here: the kernel and the tests that run without a GPU use it.
#pragma once
#include <stdint.h>

namespace sqllm {

// Word of LDS in which the counters of the buckets 2 v and 2 v + 1 lie while they are counted.  Weights that come from another quantiser have a
// few levels whose keys lie powers of two apart: with 8192 buckets all of them are counted in the same one or two banks, and the lanes of a
// wave wait for each other.  Bits 3 to 5 of v, which choose the bank, are mixed with bits 5 to 7; the eight words of a thread of the scan stay
// together.
constexpr uint32_t spread_word(uint32_t v) { return v ^ ((v >> 2) & 56u); }

}  // namespace sqllm
