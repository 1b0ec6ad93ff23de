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

// ---------------------------------------------------------------------------------------------- LDS of a workgroup
// Pair tables of a row group: entry e of row r lies at byte e * kEntryStride + r * 4, a second copy 64 bytes further.
constexpr uint32_t kEntryStride = 128;
constexpr size_t batch_table_bytes(int bits, int row_groups) { return (size_t)row_groups * (1u << (2 * bits)) * kEntryStride; }
// A wave's activations: one plane of 64 row pairs per column.  With 8 and 16 columns the planes are rotated by up to 24 dwords each and lie
// 400 bytes apart, else 272.
constexpr bool batch_rotated(int B) { return B == 8 || B == 16; }
constexpr int batch_pitch(int B) { return batch_rotated(B) ? 400 : 272; }
// ... behind the indices of a dense wave's window, row by row: 48 bytes per row, or 64 with the four chunks rotated by row (eight
// neighbouring lanes then read chunks of eight different bank groups); or behind the values of a sparse wave's 128 nonzeros
constexpr int batch_index_bytes(int bits) { return bits == 4 ? 1024 : 768; }
constexpr int batch_dense_bytes(int bits, int B) { return batch_index_bytes(bits) + B * batch_pitch(B); }
constexpr int batch_sparse_bytes(int B) { return 256 + B * batch_pitch(B); }
constexpr size_t batch_lds_bytes(int bits, int B, int row_groups, int dense_waves, int sparse_waves) {
    const size_t stage = (dense_waves ? batch_table_bytes(bits, row_groups) : 0) + (size_t)dense_waves * batch_dense_bytes(bits, B) + (size_t)sparse_waves * batch_sparse_bytes(B);
    const size_t part = (size_t)(dense_waves + sparse_waves) * row_groups * 16 * 64;   // the partial sums at the end
    return stage > part ? stage : part;
}

// ---------------------------------------------------------------------------------------------- rows and waves per workgroup
constexpr int kUnits = 256, kUnitLds = 160 * 1024;
constexpr int kMaxBatchWaves = 8;
// Waves per SIMD the registers of an instantiation are held down for.  Workgroups of 32 rows share a unit in twos (below), 16 waves in all,
// so they may not take more than 128 registers; up to 12 columns they need at most that many by themselves, and a bound made the compiler
// order their loads worse (22016x8192, 3 bits, 8 columns 37.6 against 35.9 us).
constexpr int batch_waves_per_simd(int row_groups, int B) { return row_groups == 2 && B >= 13 ? 4 : 3; }
struct BatchSplit {
    int row_groups, blocks, dense_waves, sparse_waves;
    size_t lds;
};
// 16 rows per workgroup while that gives every compute unit at most one workgroup, else 32: the activations that a workgroup reads and
// transposes serve twice the rows (weights from HBM, 0.45 % nonzeros, six and two waves: 5120x5120 at 16 columns 9.3 against 10.9 us,
// 8192x8192 19.1 against 22.2; with fewer rows half the units would idle: 1024x8192 12.2 against 9.5, 4096x11008 20.5 against 15.8).
// Six dense and two sparse waves while there is one workgroup per unit (4096x11008 at 16 columns 15.8 us; four and four 17.7, eight and
// two 15.6, eight and four 15.9; 8192x8192 19.1 / 19.0 / 20.1 / 19.2), and eight without a sparse term (8192x8192 14.3, four 15.8).  With
// more workgroups than units two of four and four waves share a unit where their LDS lets them, which is up to 16 columns with tables of 2
// and 3 bits and up to 5 with 4 bits (without a sparse term 7, and 9 to 11: with 8 the planes are wider) (13824x5120 at 5 columns 18.0 us, five and three 20.8, six and two 21.1).  Where it does not, one
// workgroup per unit has to keep the unit busy: five and three waves (4 bits, 22016x8192 at 8 columns 41.1 us; four and four 43.0; six and
// two 39.3, but at 13 columns and 13824x5120 28.3 against 27.1), and eight without a sparse term (same at 8 columns 33.2 us, four 39.6).
constexpr BatchSplit batch_split(int M, int N, int bits, int B, bool dense, bool sparse) {
    const int windows = N / 128, row_groups = M > 16 * kUnits ? 2 : 1;
    const int blocks = (int)(((int64_t)M + 16 * row_groups - 1) / (16 * row_groups));
    int nd = 0, ns = dense ? 0 : kMaxBatchWaves;
    if (dense) {
        const bool paired = blocks > kUnits && 2 * batch_lds_bytes(bits, B, row_groups, 4, sparse ? 4 : 0) <= (size_t)kUnitLds;
        nd = paired ? 4 : (!sparse ? 8 : (blocks > kUnits ? 5 : 6));
        ns = sparse ? kMaxBatchWaves - nd : 0;
        nd = windows < nd ? windows : nd;
    }
    return {row_groups, blocks, nd, ns, batch_lds_bytes(bits, B, row_groups, nd, ns)};
}

}  // namespace sqllm
