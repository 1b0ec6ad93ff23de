// Plain arithmetic of the batch kernel: where the 128-nonzero windows of its sparse term lie, and how rows and waves are split over the
// workgroups.  No HIP in here: the kernel, its launcher and the tests that run without a GPU all use these functions.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace sqllm {

// ---------------------------------------------------------------------------------------------- windows of the sparse term
// Positions of nonzeros go up to 2^31 - 2 (nnz < 2^31): a window may begin so close to that end that its first position plus 127 does
// not fit 32 bits.  So only differences of positions are formed, and offsets are clamped before they are added.
constexpr int kWindowNonzeros = 128;
constexpr int window_count(int first, int end) { return (int)(((uint32_t)(end - first) + (kWindowNonzeros - 1)) / kWindowNonzeros); }
// largest offset from p0 that the window beginning there may read: offsets past the row group repeat its last nonzero
constexpr int window_rest(int p0, int end) { return end - 1 - p0; }
constexpr int clamped(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }
// bit k: nonzero p0 + 32 q + k belongs to the row [lo, hi); positions past the row group belong to no row
constexpr uint32_t window_row_bits(int lo, int hi, int p0, int q) {
    const int b0 = clamped(clamped(lo - p0, 0, kWindowNonzeros) - 32 * q, 0, 32), b1 = clamped(clamped(hi - p0, 0, kWindowNonzeros) - 32 * q, 0, 32);
    return (uint32_t)((1ull << b1) - (1ull << b0));
}

}  // namespace sqllm
