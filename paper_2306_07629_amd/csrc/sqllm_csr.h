// Plain arithmetic over the CSR arrays, of the one-column kernel -- which nonzeros a workgroup's batches hold and whose rows they are -- and of
// the offline pass, which writes them.  No HIP in here: the kernels and the tests that run without a GPU use these functions.
// Positions of nonzeros go up to 2^31 - 2 (nnz < 2^31), and a workgroup may begin so close to that end that its first position plus a few
// batches exceeds an int.  The batches that a round asks for beyond the last nonzero are a few thousand positions, so an unsigned sum holds all
// of them; it is clamped and compared as such.
#pragma once
#include <stdint.h>

namespace sqllm {

constexpr int kBatchNonzeros = 64;                                   // one per lane
constexpr int csr_batch_count(int first, int end) { return (int)(((uint32_t)(end - first) + (kBatchNonzeros - 1)) / kBatchNonzeros); }
// the lane's nonzero in batch b of those from `first` on; batches and lanes behind the last nonzero are asked for as well
constexpr uint32_t csr_nonzero(int first, int b, int lane) { return (uint32_t)first + (uint32_t)b * kBatchNonzeros + (uint32_t)lane; }
// what is read for it: behind the last nonzero, that one again (there is one)
constexpr int csr_position(int end, uint32_t p) { return (int)(p < (uint32_t)end - 1 ? p : (uint32_t)end - 1); }
// its row among the R rows that begin at rp[0] .. rp[R - 1] and end at rp[R]; R or more: no row
template <int R>
constexpr int csr_row(const int (&rp)[R + 1], uint32_t p) {
    int row = p < (uint32_t)rp[R] ? 0 : R;
    for (int i = 1; i < R; ++i) row += p >= (uint32_t)rp[i] ? 1 : 0;
    return row;
}

// May an entry be written at position p?  In front of the end of its row and of the arrays: always, unless the weights have changed since the
// row's entries were counted.
constexpr bool csr_has_room(int p, int row_end, int capacity) { return p >= 0 && p < (row_end < capacity ? row_end : capacity); }

}  // namespace sqllm
