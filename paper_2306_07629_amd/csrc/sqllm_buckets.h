// Plain arithmetic of the k-means kernel: where its buckets are counted, and which of its shapes a matrix takes.  No HIP in here: the kernel, its
// launcher and the tests that run without a GPU use it.
#pragma once
#include <stdint.h>

namespace sqllm {

// Word of LDS in which the counters of the buckets 2 v and 2 v + 1 lie while they are counted.  Weights that come from another quantiser have a
// few levels whose keys lie powers of two apart: with 8192 buckets all of them are counted in the same one or two banks, and the lanes of a
// wave wait for each other.  Bits 3 to 5 of v, which choose the bank, are mixed with bits 5 to 7; the eight words of a thread of the scan stay
// together.
constexpr uint32_t spread_word(uint32_t v) { return v ^ ((v >> 2) & 56u); }

// The shape for M rows of N columns, named by the widest row it takes.  While one wave of a row iterates, the others have nothing to do, so as
// many rows share a compute unit as their LDS allows: few threads per row.  us before the narrower shapes (256 threads and 2048 buckets up
// to 4096 columns, 512 and 4096 up to 12288) and with them, Student-t weights: 8192x1024 at 3 bits 154 / 112, 8192x2048 at 4 bits 207 / 171,
// 4096x5120 at 4 bits 325 / 197, 4096x6144 at 3 bits 307 / 218, 4096x8192 at 3 bits 355 / 273.  Up to 11776 columns 8192 buckets instead of 4096
// halve the words read per update and still leave room for two rows (4096x11008 at 4 bits 429 / 353).
// Where the wider shape has all rows on the chip at once -- six to a unit up to 4096 columns, two beyond -- the narrower one only has fewer
// threads for the phases before and after the iterations.  Wider / narrower: 200x2048 at 3 bits 47.6 / 49.2 (two values 47.0 / 49.4), 1024x2048
// 57.5 / 56.5 (60.4 / 62.2), 1536x1536 64.2 / 63.6 (66.3 / 67.9), 200x5120 57 / 59 (59.7 / 61.2), 500x5120 at 4 bits 66.6 / 69.2 (76.1 / 77.2).  (Rows of up
// to 1024 columns are better off with 128 threads however few there are: 16x1024 39.9 / 40.0, two values 41.3 / 43.0.)  From 6145 columns on three
// rows of the narrower shape fit a unit instead of two, so that up to 1024 rows beyond 768 are two generations either way: 1000x7168
// 102 / 106 (two values 126 / 136), 1024x8192 at 2 bits 101 / 100 (132 / 140).  The same holds for 2561 to 3072 rows of 1025 to 2048 columns (2700x2048
// at 4 bits 91.6 / 89.2, two values 102.8 / 108.8) and for 769 to 1024 rows of 5889 to 6144 columns (1024x6144 98.7 / 94.9, 115.4 / 116.8), but there
// ordinary rows gain more from the narrower shape than those of two values lose.
constexpr int kKmeansUnits = 256;
constexpr int kmeans_columns(int M, int N) {
    if (N <= 1024) return 1024;
    if (N <= 2048) return M <= 6 * kKmeansUnits ? 4096 : 2048;
    if (N <= 4096) return 4096;
    if (N <= 6144) return M <= 2 * kKmeansUnits ? 11776 : 6144;
    if (N <= 8192) return M <= 2 * kKmeansUnits || (M > 3 * kKmeansUnits && M <= 4 * kKmeansUnits) ? 11776 : 8192;
    return N <= 11776 ? 11776 : (N <= 12288 ? 12288 : (N <= 16384 ? 16384 : 28672));
}

}  // namespace sqllm
