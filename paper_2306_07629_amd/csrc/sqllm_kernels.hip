// Dense-and-Sparse look-up-table matvec for gfx950 (CDNA4, wave64) — device code.
//
// What is computed (paper Sec. 4.2-4.3):  y = D x + S x,  D[i][j] = lut[i][idx(i,j)] with b-bit indices and
// one fp16 table per output row, S in CSR with fp16 values.  The storage format is described in sqllm.h.
//
// Work decomposition of the matvec kernel
//   * A workgroup owns R consecutive rows (R = 4 or 8, compile time) and all N columns.
//   * Dense waves: wave w owns the 2048-column slice [2048 w, 2048 w + 2048): lane l keeps the 32 activations
//     x[2048 w + 32 l .. +32) in registers for the whole kernel (x is read once per workgroup) and, per row,
//     loads its 32 indices (12 bytes for b = 3, 16 bytes for b = 4; the wave reads 768 / 1024 contiguous
//     bytes of the row).  D rows are requested up front, row u + D when row u has been handed to the look-ups.
//   * Dequantisation goes through PAIR TABLES in LDS: for every row of the block the workgroup first builds
//       b = 3:  64 entries,  entry (a | c << 3) = (lut[a], lut[c]) as two fp16 in one dword   (256 B / row)
//       b = 4: 256 entries,  entry (a | c << 4) = (lut[a], lut[c])                            (1 KB / row)
//       b = 2:  16 entries,  entry (a | c << 2) = (lut[a], lut[c])                            (64 B / row)
//     so ONE ds_read_b32, addressed by a 6- or 8-bit field of the index stream (two neighbouring indices),
//     returns a ready-made fp16 pair for v_dot2_f32_f16 (two products, fp32 accumulate).  Measured on MI355X
//     a wave-wide look-up occupies the LDS for ~4 cycles (64 entries) / ~7 cycles (256 entries, bank
//     conflicts), against ~7.3 for a ds_bpermute-based register table.  The field extraction is a shift + mask
//     (a funnel shift where a 3-bit pair straddles two dwords; a byte select for b = 4).
//   * The products of the sparse term join the lane sums of the dense term.  Per row the 64 lane sums are
//     reduced with DPP adds (no LDS traffic), the sums of the waves are combined through LDS in a fixed
//     order, and y is rounded to fp16 once.
//   * Sparse wave (balanced CSR, cf. Sec. 4.3): one extra wave per workgroup handles the nonzeros of the
//     block's rows while the dense waves stream.  The nonzeros of R consecutive rows are one contiguous
//     range of the CSR arrays; lane l takes nonzeros l, l + 64, ... of that range whatever rows they fall in
//     (equal work per lane), finds each one's row by comparing against the R + 1 row pointers held in
//     scalar registers, and adds the product to the lane's own partial sum of that row; the R partial sums
//     are reduced over the wave once.  No floating-point atomics, and the result does not depend on timing.
//   * With a plan of the sparse term (a one-time re-layout of the CSR arrays, see PlanView) there is no sparse wave: every
//     dense wave fetches one 64-entry batch of the workgroup's slot at wave start, gathers its activations once its last
//     index row has been requested, and adds every product to the lane's own partial sum of its row.
//   * matvec_multi_kernel / matvec_planned_multi_kernel run the workgroups of up to 16 layers in one grid: a workgroup
//     finds its layer from the first-block table in the kernel arguments and then runs the same per-block code, so every y
//     is bit for bit that of a launch of its own.
// Two to sixteen activation columns go to the matrix-core kernel in sqllm_batch.hip.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>
#include <type_traits>

#include "sqllm_csr.h"
#include "sqllm_decode.h"
#include "sqllm_kernels.h"

namespace sqllm {

// DPP controls (gfx9 encoding)
constexpr int kQuadXor1 = 0xB1;        // quad_perm:[1,0,3,2]
constexpr int kQuadXor2 = 0x4E;        // quad_perm:[2,3,0,1]
constexpr int kRowRor4 = 0x124, kRowRor8 = 0x128;
constexpr int kRowMirror = 0x140, kRowHalfMirror = 0x141;
constexpr int kRowBcast15 = 0x142, kRowBcast31 = 0x143;

template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ float dpp_f(float old, float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old), __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xF, false));
}
// Sum over the 64 lanes without LDS traffic; the total is valid in lane 63.
__device__ __forceinline__ float wave_sum_to_lane63(float v) {
    v += dpp_f<kQuadXor1>(0.f, v);
    v += dpp_f<kQuadXor2>(0.f, v);
    v += dpp_f<kRowHalfMirror>(0.f, v);
    v += dpp_f<kRowMirror>(0.f, v);                 // every lane: sum of its row of 16
    v += dpp_f<kRowBcast15, 0xA>(0.f, v);           // rows 1 and 3 add the row before them
    v += dpp_f<kRowBcast31, 0xC>(0.f, v);           // rows 2 and 3 add lane 31 (= rows 0 + 1)
    return v;
}

// the same from a uniform row pointer and the lane's dword offset inside the row: the address is formed by the load instruction
// (scalar base + 32-bit vector offset) instead of 64-bit vector arithmetic
template <int BITS>
__device__ __forceinline__ LaneChunk<BITS> load_chunk_at(const u32* __restrict__ row, u32 lane_dword) {
    LaneChunk<BITS> c;
    const u32* p = reinterpret_cast<const u32*>(reinterpret_cast<const char*>(row) + (size_t)(lane_dword * 4u));
#pragma unroll
    for (int k = 0; k < BITS; ++k) c.q[k] = __builtin_nontemporal_load(p + k);
    return c;
}

// Byte offsets (entry * 4) into the row's pair table of the 16 index pairs of a lane.
//   b = 3: pair p owns bits [6p, 6p + 6) of the 96-bit chunk; two of them straddle a dword boundary.
//   b = 4: pair p is byte p of the 128-bit chunk.
__device__ __forceinline__ void pair_offsets(const LaneChunk<3>& c, u32 (&a)[16]) {
    const u32 q0 = c.q[0], q1 = c.q[1], q2 = c.q[2];
    a[0] = (q0 << 2) & 0xFC;   a[1] = (q0 >> 4) & 0xFC;   a[2] = (q0 >> 10) & 0xFC;  a[3] = (q0 >> 16) & 0xFC;
    a[4] = (q0 >> 22) & 0xFC;
    a[5] = funnel_shr(q1, q0, 28) & 0xFC;               // bits 30..35 straddle dwords 0 and 1
    a[6] = (q1 >> 2) & 0xFC;   a[7] = (q1 >> 8) & 0xFC;   a[8] = (q1 >> 14) & 0xFC;  a[9] = (q1 >> 20) & 0xFC;
    a[10] = funnel_shr(q2, q1, 26) & 0xFC;              // bits 60..65 straddle dwords 1 and 2
    a[11] = q2 & 0xFC;         a[12] = (q2 >> 6) & 0xFC;  a[13] = (q2 >> 12) & 0xFC; a[14] = (q2 >> 18) & 0xFC;
    a[15] = (q2 >> 24) & 0xFC;
}
__device__ __forceinline__ void pair_offsets(const LaneChunk<4>& c, u32 (&a)[16]) {
#pragma unroll
    for (int p = 0; p < 16; ++p) a[p] = ((c.q[p >> 2] >> (8 * (p & 3))) & 0xFF) << 2;
}
//   b = 2: pair p is nibble p of the 64-bit chunk.
__device__ __forceinline__ void pair_offsets(const LaneChunk<2>& c, u32 (&a)[16]) {
#pragma unroll
    for (int p = 0; p < 16; ++p) a[p] = ((c.q[p >> 3] >> (4 * (p & 7))) & 0xF) << 2;
}

// the offset of pair p alone (p a compile-time constant after unrolling): the same values as pair_offsets
__device__ __forceinline__ u32 pair_offset_of(const LaneChunk<3>& c, int p) {
    const u32 q0 = c.q[0], q1 = c.q[1], q2 = c.q[2];
    switch (p) {
        case 0: return (q0 << 2) & 0xFC;
        case 1: return (q0 >> 4) & 0xFC;
        case 2: return (q0 >> 10) & 0xFC;
        case 3: return (q0 >> 16) & 0xFC;
        case 4: return (q0 >> 22) & 0xFC;
        case 5: return funnel_shr(q1, q0, 28) & 0xFC;
        case 6: return (q1 >> 2) & 0xFC;
        case 7: return (q1 >> 8) & 0xFC;
        case 8: return (q1 >> 14) & 0xFC;
        case 9: return (q1 >> 20) & 0xFC;
        case 10: return funnel_shr(q2, q1, 26) & 0xFC;
        case 11: return q2 & 0xFC;
        case 12: return (q2 >> 6) & 0xFC;
        case 13: return (q2 >> 12) & 0xFC;
        case 14: return (q2 >> 18) & 0xFC;
        default: return (q2 >> 24) & 0xFC;
    }
}
__device__ __forceinline__ u32 pair_offset_of(const LaneChunk<4>& c, int p) { return ((c.q[p >> 2] >> (8 * (p & 3))) & 0xFF) << 2; }
__device__ __forceinline__ u32 pair_offset_of(const LaneChunk<2>& c, int p) { return ((c.q[p >> 3] >> (4 * (p & 7))) & 0xF) << 2; }

// Pair tables of R rows from their fp16 tables staged in LDS (raw[u << BITS | k]); executed by ONE wave.
template <int BITS, int R>
__device__ __forceinline__ void build_tables(u32* __restrict__ tables, const uint16_t* __restrict__ raw, int lane) {
    constexpr int E = TableShape<BITS>::kEntries, K = 1 << BITS;
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const u32 lo = raw[u * K + (lane & (K - 1))];           // the same for all entries of this lane
#pragma unroll
        for (int e0 = 0; e0 < E; e0 += kWave) {
            const int e = e0 + lane;
            if (E >= kWave || e < E) {
                const u32 hi = raw[u * K + (e >> BITS)];
                tables[u * E + e] = lo | (hi << 16);
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------- x in registers
// xr[p] = (x[j0 + 2p], x[j0 + 2p + 1]) for the lane's 32 columns j0 .. j0 + 31 (j0 is in range, x is one column).
__device__ __forceinline__ void load_x(const uint16_t* __restrict__ x, u32 j0, u32 (&xr)[16]) {
    const u32x4* src = reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(x) + (size_t)(j0 * 2u));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const u32x4 v = src[k];
        xr[4 * k + 0] = v.x; xr[4 * k + 1] = v.y; xr[4 * k + 2] = v.z; xr[4 * k + 3] = v.w;
    }
}

// table look-ups of one row slice: 16 dwords, each an fp16 pair
template <int BITS>
__device__ __forceinline__ void lookup_chunk(const LaneChunk<BITS>& c, const u32* __restrict__ table, u32 (&w)[16]) {
    u32 a[16];
    pair_offsets(c, a);
    const char* tb = reinterpret_cast<const char*>(table);
#pragma unroll
    for (int p = 0; p < 16; ++p) w[p] = *reinterpret_cast<const u32*>(tb + a[p]);
}

// 16 packed dot products (two fp16 products each, fp32 accumulate) in two accumulator chains
__device__ __forceinline__ float dot_chunk(const u32 (&w)[16], const u32 (&xr)[16]) {
    float a0 = 0.f, a1 = 0.f;
#pragma unroll
    for (int p = 0; p < 16; p += 2) {
        a0 = __builtin_amdgcn_fdot2(as_half2(w[p]), as_half2(xr[p]), a0, false);
        a1 = __builtin_amdgcn_fdot2(as_half2(w[p + 1]), as_half2(xr[p + 1]), a1, false);
    }
    return a0 + a1;
}

// Joint reduction of C per-lane values over the lanes of each 16-lane row (C = 4 or 8).  On return v[0] holds, in the lanes
// named by row_block_slot(), the sum of one input v[c] over the 16 lanes of the lane's row.  Butterfly steps halve the number of
// live values (3 VALU per produced value instead of a full 4-step reduction per input).  The association of the additions is
// the same for every c and both C -- quads first (lane ^ 1, lane ^ 2), then quad k with quad k ^ 2, then the two pair sums:
// ((q0 + q2) + (q1 + q3)) up to commutativity -- so a row's sum does not depend on how many rows its workgroup owns, and
// projections stacked into one call give bit for bit the dense term of separate calls.
template <int C>
__device__ __forceinline__ void row_block_reduce(float (&v)[C], int lane) {
    static_assert(C == 4 || C == 8, "block size");
    {   // lane bit 0, partner lane ^ 1: v[k] <- class 2 k + (lane & 1)
        const bool hi = lane & 1;
#pragma unroll
        for (int k = 0; k < C / 2; ++k) {
            const float keep = hi ? v[2 * k + 1] : v[2 * k], send = hi ? v[2 * k] : v[2 * k + 1];
            v[k] = keep + dpp_f<kQuadXor1>(0.f, send);
        }
    }
    {   // lane bit 1, partner lane ^ 2: v[k] <- class 4 k + (lane & 3)
        const bool hi = lane & 2;
#pragma unroll
        for (int k = 0; k < C / 4; ++k) {
            const float keep = hi ? v[2 * k + 1] : v[2 * k], send = hi ? v[2 * k] : v[2 * k + 1];
            v[k] = keep + dpp_f<kQuadXor2>(0.f, send);
        }
    }
    // lane bit 3 (a rotation by 8 lanes pairs lane l with lane l ^ 8): quads k and k ^ 2
    if constexpr (C == 8) {
        const bool hi = lane & 8;
        const float keep = hi ? v[1] : v[0], send = hi ? v[0] : v[1];
        v[0] = keep + dpp_f<kRowRor8>(0.f, send);            // lanes 0..7: class lane & 3; lanes 8..15: class 4 + (lane & 3)
    } else {
        v[0] += dpp_f<kRowRor8>(0.f, v[0]);
    }
    // lane bit 2: a rotation by 4 lanes hands quad k the pair sum of quad k - 1, which holds the same class for odd k
    v[0] += dpp_f<kRowRor4>(0.f, v[0]);
}
// lane of a 16-lane row that holds class c after row_block_reduce<C>: a lane of quad 1 (c < 4) or quad 3 (c >= 4)
__device__ __forceinline__ bool row_block_valid(int lane) { return (lane & 4) != 0; }
template <int C>
__device__ __forceinline__ int row_block_class(int lane) { return (C == 8 && (lane & 8)) ? 4 + (lane & 3) : (lane & 3); }

// ---------------------------------------------------------------------------------------------- sparse term
// Balanced CSR (cf. Sec. 4.3).  The nonzeros of the block's R rows are ONE contiguous range [P0, P1) of the
// CSR arrays.  It is cut into batches of 64; batch b goes to wave (b mod NW) and lane l of that wave takes
// nonzero P0 + 64 b + l, whatever row it falls in -- every lane of the block gets the same amount of work
// and a heavy row is spread over all waves.  A wave handles up to UB batches per round: first all column /
// value loads, then all activation gathers, then the sums, so a round costs two memory round trips
// (which the dense decode of the same wave overlaps).  Every lane adds to its own partial sums of the R rows: fixed order, no atomics, no
// scan.  (A segmented scan over the lanes with one LDS add per row segment before: 22016x8192, 1 % of the rows with 30 % of the nonzeros,
// 21.1 us against 19.9, 11008x4096 7.6 against 7.2; one LDS float add per nonzero: lanes meeting in a slot are served one after the other,
// another 5.5 us at 22016x8192.)
template <int UB>
struct SparseRegs {
    int c[UB];
    uint16_t vb[UB];
    uint16_t xv[UB];
};

struct SparseRange {
    int P0, P1, nbatch;
};

// Loads of one round are unconditional (positions clamped to the range's last nonzero, surplus lanes and batches are masked
// in the sums), so that all of them are in flight at once.
template <int UB>
__device__ __forceinline__ void sparse_issue_cols_vals(const MatvecArgs& g, const SparseRange& sr, int b0, int NW, int lane, SparseRegs<UB>& q) {
    const int* __restrict__ cols = g.cols;
    const uint16_t* __restrict__ vals = static_cast<const uint16_t*>(g.vals);
#pragma unroll
    for (int k = 0; k < UB; ++k) {
        const int p = csr_position(sr.P1, csr_nonzero(sr.P0, b0 + k * NW, lane));
        q.c[k] = cols[p];
        q.vb[k] = vals[p];
    }
}

template <int UB>
__device__ __forceinline__ void sparse_issue_gathers(const uint16_t* __restrict__ x, SparseRegs<UB>& q) {
#pragma unroll
    for (int k = 0; k < UB; ++k) q.xv[k] = x[q.c[k]];
}

template <int R, int UB>
__device__ __forceinline__ void sparse_accumulate(const SparseRange& sr, const int (&rp)[R + 1], int b0, int NW, int lane, const SparseRegs<UB>& q, float (&acc)[R]) {
#pragma unroll
    for (int k = 0; k < UB; ++k) {
        const int b = b0 + k * NW;
        if (b < sr.nbatch) {                                         // uniform
            const float v = half_bits_to_float(q.vb[k]) * half_bits_to_float(q.xv[k]);
            const int row = csr_row<R>(rp, csr_nonzero(sr.P0, b, lane));   // R or more: nothing for this lane
#pragma unroll
            for (int i = 0; i < R; ++i) acc[i] = row == i ? acc[i] + v : acc[i];
        }
    }
}

template <int R, int U>
__device__ __forceinline__ void sparse_round(const MatvecArgs& g, const uint16_t* __restrict__ x, const SparseRange& sr, const int (&rp)[R + 1],
                                             int b0, int NW, int lane, float (&acc)[R]) {
    SparseRegs<U> q;
    sparse_issue_cols_vals<U>(g, sr, b0, NW, lane, q);
    sparse_issue_gathers<U>(x, q);
    sparse_accumulate<R, U>(sr, rp, b0, NW, lane, q, acc);
}

// ---------------------------------------------------------------------------------------------- the matvec kernel (one activation column)
// grid.x = ceil(M / R); block = (W + S) waves.  W = ceil(N / 2048) dense waves (0 without a dense term), wave w
// owning column slice w; S sparse waves (1 next to a dense term, kSparseOnlyWaves alone, 0 when nnz == 0).
// The sparse wave works through the first UB batches of the block's nonzeros while the dense waves stream
// (that is all of them except in blocks holding a very heavy row); whatever is left is dealt out to ALL
// waves once the dense waves have finished their rows, so a heavy row never serialises on one wave.
// The dense path is straight-line code: out-of-range lanes and rows load clamped (valid) addresses and are
// neutralised by zero activations / by not being stored.
constexpr int kSparseOnlyWaves = 4;

template <int R>
__device__ __forceinline__ void load_row_pointers(const MatvecArgs& g, int r0, int nrows, bool sparse, int (&rp)[R + 1], SparseRange& sr) {
#pragma unroll
    for (int k = 0; k <= R; ++k) rp[k] = sparse ? g.rowptr[r0 + min(k, nrows)] : 0;   // uniform -> scalar loads
    sr.P0 = rp[0]; sr.P1 = rp[R]; sr.nbatch = csr_batch_count(sr.P0, sr.P1);
}

// Total of one output row over the workgroup's n partial sums a[i * R + row].
// Eight lanes per row (lane = 8 row + p) each add every eighth value in order, then the eight are combined by a butterfly whose
// every lane forms the same sums; the order depends on the count only, not on R.  Valid in all eight lanes of a row < R.
template <int R>
__device__ __forceinline__ float block_row_total(const float* __restrict__ a, int n, int lane) {
    const int row = lane >> 3, p = lane & 7;
    float s = 0.f;
    if (row < R) {
        for (int i = p; i < n; i += 8) s += a[i * R + row];
    }
    s += dpp_f<kQuadXor1>(0.f, s);
    s += dpp_f<kQuadXor2>(0.f, s);
    s += dpp_f<kRowHalfMirror>(0.f, s);
    return s;
}

// The work of one workgroup: rows [R block, R block + R) of layer g, carried by the workgroup's first NW waves
// (W dense waves, then the sparse wave).
template <int BITS, int R, int D>
__device__ __forceinline__ void matvec_block(const MatvecArgs& g, int block, int NW) {
    static_assert(D >= 2 && D <= R && (R == 4 || R == 8), "prefetch depth, rows per workgroup");
    constexpr int E = TableShape<BITS>::kEntries, K = 1 << BITS;
    constexpr int kRawUnit = TableShape<BITS>::kRawUnit;             // bytes of fp16 tables one lane fetches (16, or 8 for b = 2)
    constexpr int UB = 8;                                            // sparse batches per wave and round
    constexpr int TD = TableShape<BITS>::kTableDwords;
    __shared__ __align__(8) u32 tables[R * TD];
    __shared__ __align__(16) uint16_t raw[R * K];
    __shared__ float part[(kMaxDenseWaves + 1) * 4 * R];             // [wave][16-lane row][r]

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform, and known to be
    const bool dense = g.qidx != nullptr, sparse = g.nnz > 0;
    const int W = dense ? (g.N + kSliceCols - 1) / kSliceCols : 0;
    const int r0 = block * R;
    const int nrows = min(R, g.M - r0);
    const uint16_t* __restrict__ x = static_cast<const uint16_t*>(g.x);

    int rp[R + 1];
    SparseRange sr;
    load_row_pointers<R>(g, r0, nrows, sparse, rp, sr);              // consumed late by the dense waves
    int next_batch = 0;                                              // first batch not yet handled (uniform)
    float acc[R];

    if (wave < W) {
        // ---- dense wave.  Issue order: (wave 0: fp16 tables), activations, first D rows of the index stream.
        // wave 0 fetches the fp16 tables of the block's rows (LPR lanes per row) and builds their pair tables
        constexpr int LPR = TableShape<BITS>::kRowBytes / kRawUnit;
        const int my_rows = wave == 0 ? R : 0;
        const int bu = lane / LPR;                                    // row of the block this lane fetches a piece of
        u32x4 rawv = {0, 0, 0, 0};
        if (lane < my_rows * LPR) {
            const int row = min(r0 + bu, g.M - 1);
            const char* src = static_cast<const char*>(g.lut) + (size_t)row * TableShape<BITS>::kRowBytes + (lane % LPR) * kRawUnit;
            if constexpr (kRawUnit == 16) {
                rawv = *reinterpret_cast<const u32x4*>(src);
            } else {
                const u32x2 v = *reinterpret_cast<const u32x2*>(src);
                rawv.x = v.x; rawv.y = v.y;
            }
        }
        const u32 j0 = (u32)wave * kSliceCols + (u32)lane * kLaneElems;
        const bool live = j0 < (u32)g.N;
        const u32 j0c = live ? j0 : (u32)g.N - kLaneElems;
        u32 xr[16];
        load_x(x, j0c, xr);
        const u32 row_bytes = (u32)g.N / 8u * BITS;
        const u32 lane_dword = (j0c >> 5) * BITS;                    // the lane's 32 indices inside a row of the index stream
        auto row_ptr = [&](int u) {                                  // uniform: the scalar unit works it out
            return reinterpret_cast<const u32*>(static_cast<const char*>(g.qidx) + (size_t)(u32)min(r0 + u, g.M - 1) * row_bytes);
        };
        LaneChunk<BITS> c[R];
#pragma unroll
        for (int u = 0; u < D; ++u) c[u] = load_chunk_at<BITS>(row_ptr(u), lane_dword);
        if (!live) {
#pragma unroll
            for (int p = 0; p < 16; ++p) xr[p] = 0;
        }
        if (my_rows > 0) {                                            // uniform
            if (lane < my_rows * LPR) {
                if constexpr (kRawUnit == 16) *reinterpret_cast<u32x4*>(raw + bu * K + (lane % LPR) * 8) = rawv;
                else *reinterpret_cast<u32x2*>(raw + bu * K) = u32x2{rawv.x, rawv.y};
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            build_tables<BITS, R>(tables, raw, lane);
        }
        __syncthreads();
        // software pipeline: the look-ups of row u + 1 are in flight while the products of row u are formed;
        // row u + D of the index stream is requested when row u has been handed to the look-ups
        u32 w[16];
        lookup_chunk<BITS>(c[0], tables, w);
        if constexpr (D < R) c[D] = load_chunk_at<BITS>(row_ptr(D), lane_dword);
#pragma unroll
        for (int u = 0; u < R; ++u) {
            if (u + 1 + D < R) c[(u + 1 + D) % R] = load_chunk_at<BITS>(row_ptr(u + 1 + D), lane_dword);
            // The look-ups of row u + 1 are issued one at a time between the products of row u (the product of a pair, two field
            // extractions, one look-up) instead of as a block of 16 -- the workgroups of a launch run in step, and blocks of
            // look-ups from all of them fill the LDS queue while the vector ALUs idle.
            // One set of 16 registers holds the pairs of both rows: the look-up of pair p of row u + 1 goes into the register the
            // product of pair p of row u has just read (two sets cost 8 to 16 registers per lane, i.e. a wave per SIMD).  The products
            // run in the two accumulator chains of dot_chunk; the scheduling barrier after every step keeps the order.
            {
                float a0 = 0.f, a1 = 0.f;
                const char* tb = reinterpret_cast<const char*>(tables + (u + 1 < R ? u + 1 : 0) * TD);
#pragma unroll
                for (int p = 0; p < 16; ++p) {
                    if (p & 1) a1 = __builtin_amdgcn_fdot2(as_half2(w[p]), as_half2(xr[p]), a1, false);
                    else a0 = __builtin_amdgcn_fdot2(as_half2(w[p]), as_half2(xr[p]), a0, false);
                    if (u + 1 < R) {
                        w[p] = *reinterpret_cast<const u32*>(tb + pair_offset_of(c[u + 1], p));
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                acc[u] = a0 + a1;
                asm volatile("" : "+v"(acc[u]));                     // formed here: sunk to its use behind the sparse term, a row's sum keeps its operands alive
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        next_batch = UB;                                             // the sparse wave takes batches 0 .. UB-1
    } else {
        // ---- sparse wave(s)
#pragma unroll
        for (int u = 0; u < R; ++u) acc[u] = 0.f;
        if (dense) {
            // columns and values of the first batches are requested BEFORE the dense waves' table barrier: the row pointers arrive
            // together with the fp16 tables, so the second hop of the chain (row pointers -> columns / values -> gathers -> sums)
            // runs while the tables are built instead of after (22016x8192 fused 21.3 -> 20.5 us)
            if (sr.nbatch > 2) {
                SparseRegs<UB> q;
                sparse_issue_cols_vals<UB>(g, sr, 0, 1, lane, q);
                __syncthreads();
                sparse_issue_gathers<UB>(x, q);
                sparse_accumulate<R, UB>(sr, rp, 0, 1, lane, q, acc);
            } else if (sr.nbatch > 0) {
                SparseRegs<2> q;
                sparse_issue_cols_vals<2>(g, sr, 0, 1, lane, q);
                __syncthreads();
                sparse_issue_gathers<2>(x, q);
                sparse_accumulate<R, 2>(sr, rp, 0, 1, lane, q, acc);
            } else {
                __syncthreads();
            }
            next_batch = UB;
        }
    }
    // ---- what is left of the sparse term (everything in a sparse-only launch): batch b goes to wave
    //      (b - next_batch) mod NW, UB batches per wave and round
    for (int b0 = next_batch + wave; b0 < sr.nbatch; b0 += NW * UB)   // uniform
        sparse_round<R, UB>(g, x, sr, rp, b0, NW, lane, acc);
    // reduce the R row sums jointly over each 16-lane row of the wave
    row_block_reduce<R>(acc, lane);
    if (row_block_valid(lane) && (R == 8 || !(lane & 8))) part[(wave * 4 + (lane >> 4)) * R + row_block_class<R>(lane)] = acc[0];
    __syncthreads();

    // combine the sums of the waves in a fixed order, round once
    uint16_t* __restrict__ y = static_cast<uint16_t*>(g.y);
    if (wave == 0) {
        float s = block_row_total<R>(part, 4 * NW, lane);
        const int row = lane >> 3;
        if ((lane & 7) == 0 && row < nrows) {
            if (g.accumulate) s += half_bits_to_float(y[r0 + row]);
            y[r0 + row] = float_to_half_bits(s);
        }
    }
}

// ---------------------------------------------------------------------------------------------- sparse term from a plan
// A plan (sqllm_kernels.h: PlanLayout) holds the nonzeros of every block of four rows (a "quad") as groups of 16 entries of one
// row, four groups to a batch of 64 lanes, the first C batches of a quad in a slot found from the quad index alone.  A workgroup
// of R rows serves R / 4 quads, each exactly as a four-row workgroup would (same batches on the same waves in the same order),
// so the sparse sums -- like the dense ones -- do not depend on R.  Against the
// CSR arrays this removes the first hop of the dependent chain (row pointers -> columns / values -> gathers), halves the loads
// per nonzero (column and value share a dword) and needs no scan: a lane adds its product to one of its R partial sums of the dense
// term, which are reduced over the wave anyway.  That is cheap enough for the dense waves to carry the sparse term themselves, so a
// workgroup needs no extra wave.
struct PlanView {
    const u32* slot_entries;    // [quads][C][64]
    const uint8_t* slot_tags;   // [quads][C][4]  one tag byte per group
    const int* ov_desc;         // [quads][2]     first overflow batch, overflow batches
    const u32* ov_entries;      // [ov batches][64]
    const uint8_t* ov_tags;     // [ov batches][4]
    int C;
    int ov_cap;                 // batches the overflow sections hold
};

constexpr int kPlanRows = 4;   // rows of a plan block ("quad"), whatever the rows per workgroup of the kernel that reads it

__device__ __forceinline__ PlanView plan_view(const void* plan, int M, long long nnz, int C) {
    // the offsets of plan_layout() on the host; C comes with the kernel arguments (its formula needs a 64-bit division)
    const size_t n_q = (size_t)((M + kPlanRows - 1) / kPlanRows);
    const size_t ov_cap = (size_t)((nnz / 16 + M) / 4) + n_q + 1;
    auto up = [](size_t v) { return (v + 255) & ~(size_t)255; };
    const char* b = static_cast<const char*>(plan);
    PlanView v;
    size_t o = 0;
    v.slot_entries = reinterpret_cast<const u32*>(b + o); o += up(n_q * C * 256);
    v.slot_tags = reinterpret_cast<const uint8_t*>(b + o); o += up(n_q * C * 4);
    v.ov_desc = reinterpret_cast<const int*>(b + o);      o += up(n_q * 8);
    v.ov_entries = reinterpret_cast<const u32*>(b + o);   o += up(ov_cap * 256);
    v.ov_tags = reinterpret_cast<const uint8_t*>(b + o);
    v.C = C;
    v.ov_cap = (int)ov_cap;
    return v;
}

// One batch: entry, gathered activation and the tag byte of the lane's group (valid << 7 | (count - 1) << 3 | row) per lane.  Each lane adds
// its product to its own partial sum of the entry's row, beside what the dense term left there.  Padded lanes add nothing, not a zero
// product: their column is 0, whose activation may be infinite.  About 17 vector instructions per batch, and none of them waits for the
// LDS; with a sum over the 16 lanes of a group and an LDS add per group (40 instructions) 8192x8192 took 9.9 us instead of 9.2 (1 % of the
// rows with 30 % of 0.45 % nonzeros), 4096x4096 at 4 bits 4.65 instead of 4.44, a 65B-shaped MLP pair 42.1 instead of 40.4 and a decode
// step of four 7B-shaped blocks in groups 122.2 instead of 117.3: a wave's instructions are issued in turn with those of six or seven
// others, so the workgroups that end last are as late as their chain is long.
__device__ __forceinline__ void plan_batch_add(u32 entry, u32 xv, u32 tb, int lane, float (&acc)[kPlanRows]) {
    const int t = (int)tb - 8 * (lane & 15);                         // 128 and above: a valid group that has an entry for the lane
    const float v = half_bits_to_float((uint16_t)(entry >> 16)) * half_bits_to_float((uint16_t)xv);
    const u32 row = t >= 128 ? (u32)t & 7u : 8u;
#pragma unroll
    for (int i = 0; i < kPlanRows; ++i) acc[i] = row == (u32)i ? acc[i] + v : acc[i];
}

template <int BITS, int R, int D>
__device__ __forceinline__ void matvec_planned_block(const MatvecArgs& g, int block, int W) {
    static_assert(D >= 2 && D <= R && (R == 4 || R == 8), "prefetch depth, rows per workgroup");
    constexpr int K = 1 << BITS;
    constexpr int kRawUnit = TableShape<BITS>::kRawUnit;
    constexpr int Q = R / kPlanRows;                                 // quads of the plan per workgroup; C <= W: one slot batch per wave and quad
    constexpr int UP = Q == 1 ? 2 : 1;                               // overflow batches per wave and quad requested ahead
    constexpr int TD = TableShape<BITS>::kTableDwords;
    __shared__ __align__(8) u32 tables[R * TD];
    __shared__ __align__(16) uint16_t raw[R * K];
    __shared__ float part[kMaxDenseWaves * 4 * R];                   // [wave][16-lane row][r]

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r0 = block * R;
    const int nrows = min(R, g.M - r0);
    const uint16_t* __restrict__ x = static_cast<const uint16_t*>(g.x);
    const PlanView pv = plan_view(g.plan, g.M, g.nnz, g.plan_c);
    const int n_quads = (g.M + kPlanRows - 1) / kPlanRows;

    // ---- Issue order: (wave 0: fp16 tables), activations, first D rows of the index stream, this wave's slot batches
    constexpr int LPR = TableShape<BITS>::kRowBytes / kRawUnit;
    const int my_rows = wave == 0 ? R : 0;
    const int bu = lane / LPR;
    u32x4 rawv = {0, 0, 0, 0};
    if (lane < my_rows * LPR) {
        const int row = min(r0 + bu, g.M - 1);
        const char* src = static_cast<const char*>(g.lut) + (size_t)row * TableShape<BITS>::kRowBytes + (lane % LPR) * kRawUnit;
        if constexpr (kRawUnit == 16) {
            rawv = *reinterpret_cast<const u32x4*>(src);
        } else {
            const u32x2 v = *reinterpret_cast<const u32x2*>(src);
            rawv.x = v.x; rawv.y = v.y;
        }
    }
    const u32 j0 = (u32)wave * kSliceCols + (u32)lane * kLaneElems;
    const bool live = j0 < (u32)g.N;
    const u32 j0c = live ? j0 : (u32)g.N - kLaneElems;
    u32 xr[16];
    load_x(x, j0c, xr);
    const u32 row_bytes = (u32)g.N / 8u * BITS;
    const u32 lane_dword = (j0c >> 5) * BITS;                        // the lane's 32 indices inside a row of the index stream
    auto row_ptr = [&](int u) {                                      // uniform: the scalar unit works it out
        return reinterpret_cast<const u32*>(static_cast<const char*>(g.qidx) + (size_t)(u32)min(r0 + u, g.M - 1) * row_bytes);
    };
    LaneChunk<BITS> c[R];
#pragma unroll
    for (int u = 0; u < D; ++u) c[u] = load_chunk_at<BITS>(row_ptr(u), lane_dword);
    // The slot batch of this wave in quad q is batch `wave` of that quad's slot; past the slot (wave >= C) the last batch is
    // re-read and ignored.  Entries, tag bytes (one per group, fetched by the group's own lanes) and the overflow descriptors all
    // come through vector loads: a scalar load would have to be waited for together with every LDS operation of the wave.
    u32 ent[Q], tags[Q], sx[Q], oe[Q][UP], ot[Q][UP];
    int ovd[Q], ov_first[Q], ov_nb[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int quad = min(block * Q + q, n_quads - 1);            // a workgroup at the end of M may have no second quad
        const size_t sb = (size_t)quad * pv.C + min(wave, pv.C - 1);
        ent[q] = pv.slot_entries[sb * 64 + lane];
        tags[q] = pv.slot_tags[sb * 4 + (lane >> 4)];
        ovd[q] = pv.ov_desc[2 * quad + (lane & 1)];                  // lane 0: first overflow batch, lane 1: their number
        ov_first[q] = 0; ov_nb[q] = 0;
    }
    if (!live) {
#pragma unroll
        for (int p = 0; p < 16; ++p) xr[p] = 0;
    }
    if (my_rows > 0) {                                                // uniform
        if (lane < my_rows * LPR) {
            if constexpr (kRawUnit == 16) *reinterpret_cast<u32x4*>(raw + bu * K + (lane % LPR) * 8) = rawv;
            else *reinterpret_cast<u32x2*>(raw + bu * K) = u32x2{rawv.x, rawv.y};
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        build_tables<BITS, R>(tables, raw, lane);
    }
    __syncthreads();
    float acc[Q][kPlanRows];
    u32 w[16];                                                       // the pairs of the current row; each is replaced by the next row's once its product is formed
    lookup_chunk<BITS>(c[0], tables, w);
    if constexpr (D < R) c[D] = load_chunk_at<BITS>(row_ptr(D), lane_dword);
#pragma unroll
    for (int u = 0; u < R; ++u) {
        if (u + 1 < R) {
            if (u + 1 + D < R) c[(u + 1 + D) % R] = load_chunk_at<BITS>(row_ptr(u + 1 + D), lane_dword);
        }
        // The activations of the slot batches are gathered once the last row of the index stream has been requested: memory
        // results return in request order, so gathers issued earlier would stand between the wave and its next rows, and a
        // gather has to wait for its entry first (the scheduling barrier keeps the compiler from moving that wait, and with it
        // the request for the last row, the other way round).
        // With them go the requests for this wave's first overflow batches (a workgroup with a heavy row has some): their
        // place is known once the descriptor has arrived, which it has when the entries have.
        if (u + 1 + D == R - 1 || (D == R - 1 && u == 0)) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < Q; ++q) sx[q] = x[ent[q] & 0x7FFFu];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                ov_first[q] = __builtin_amdgcn_readlane(ovd[q], 0);
                ov_nb[q] = __builtin_amdgcn_readlane(ovd[q], 1);
#pragma unroll
                for (int k = 0; k < UP; ++k) {
                    const int b = min(ov_first[q] + min(wave + k * W, max(ov_nb[q] - 1, 0)), pv.ov_cap - 1);
                    oe[q][k] = pv.ov_entries[(size_t)b * 64 + lane];
                    ot[q][k] = pv.ov_tags[(size_t)b * 4 + (lane >> 4)];
                }
            }
        }
        // products of row u in the two accumulator chains of dot_chunk; the look-ups of row u + 1 take over its registers one by one
        // (as in matvec_block)
        {
            float a0 = 0.f, a1 = 0.f;
            const char* tb = reinterpret_cast<const char*>(tables + (u + 1 < R ? u + 1 : 0) * TD);
#pragma unroll
            for (int p = 0; p < 16; ++p) {
                if (p & 1) a1 = __builtin_amdgcn_fdot2(as_half2(w[p]), as_half2(xr[p]), a1, false);
                else a0 = __builtin_amdgcn_fdot2(as_half2(w[p]), as_half2(xr[p]), a0, false);
                if (u + 1 < R) {
                    w[p] = *reinterpret_cast<const u32*>(tb + pair_offset_of(c[u + 1], p));
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            acc[u / kPlanRows][u % kPlanRows] = a0 + a1;
            asm volatile("" : "+v"(acc[u / kPlanRows][u % kPlanRows]));   // formed here: sunk to its use behind the sparse term, a row's sum keeps its operands alive (125 registers)
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // ---- sparse term, quad by quad: this wave's slot batch, then its share of the quad's overflow batches (batches wave, wave + W,
    // wave + 2 W, ... in this order whatever UP and R are)
    constexpr int UO = 8;                                            // batches per wave and round in the loop for very heavy rows
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const bool have = block * Q + q < n_quads;                   // uniform; the last workgroup of an odd number of quads has one
        const int nb = have ? ov_nb[q] : 0, first = ov_first[q];
        if (wave < pv.C && have) plan_batch_add(ent[q], sx[q], tags[q], lane, acc[q]);        // uniform
        if (wave < nb) {                                                                      // uniform
            u32 ox[UP];
#pragma unroll
            for (int k = 0; k < UP; ++k) ox[k] = x[oe[q][k] & 0x7FFFu];
#pragma unroll
            for (int k = 0; k < UP; ++k)
                if (wave + k * W < nb) plan_batch_add(oe[q][k], ox[k], ot[q][k], lane, acc[q]);
        }
        // what a very heavy row leaves after that: UO batches per wave and round, all requested before the first is used (the
        // workgroup that owns such a row ends last, and every round costs it two memory latencies)
        for (int ob = wave + UP * W; ob < nb; ob += UO * W) {                                 // uniform
            u32 e2[UO], t2[UO], x2[UO];
#pragma unroll
            for (int k = 0; k < UO; ++k) {
                const int b = min(ob + k * W, nb - 1);
                e2[k] = pv.ov_entries[(size_t)(first + b) * 64 + lane];
                t2[k] = pv.ov_tags[(size_t)(first + b) * 4 + (lane >> 4)];
            }
#pragma unroll
            for (int k = 0; k < UO; ++k) x2[k] = x[e2[k] & 0x7FFFu];
#pragma unroll
            for (int k = 0; k < UO; ++k)
                if (ob + k * W < nb) plan_batch_add(e2[k], x2[k], t2[k], lane, acc[q]);
        }
    }
    float sum[R];
#pragma unroll
    for (int u = 0; u < R; ++u) sum[u] = acc[u / kPlanRows][u % kPlanRows];
    row_block_reduce<R>(sum, lane);
    if (row_block_valid(lane) && (R == 8 || !(lane & 8))) part[(wave * 4 + (lane >> 4)) * R + row_block_class<R>(lane)] = sum[0];
    __syncthreads();
    uint16_t* __restrict__ y = static_cast<uint16_t*>(g.y);
    if (wave == 0) {
        const float s = block_row_total<R>(part, 4 * W, lane);
        const int row = lane >> 3;
        if ((lane & 7) == 0 && row < nrows) y[r0 + row] = float_to_half_bits(s);
    }
}

template <int BITS, int R, int D>
__global__ void __launch_bounds__(1024) matvec_planned_kernel(MatvecArgs g) {
    matvec_planned_block<BITS, R, D>(g, blockIdx.x, blockDim.x >> 6);
}

// The arguments of a multi-layer launch as the kernel takes them (by value): only the fields its class reads, and room for 8 or
// 16 layers, whichever the launch needs.  The block stays under 1 KiB (16 planned layers: 968 bytes, 8 CSR layers: 616): launches
// with a larger one were measured 7 to 17 % slower over a whole decode step, whatever the layout of the fields, and a small block
// is a little faster than a large one below that size too.
struct PlannedLayer { int M, N, nnz, plan_c; const void *qidx, *lut, *x; void* y; const void* plan; };                            // 56 bytes
struct CsrLayer { int M, N, nnz, pad; const void *qidx, *lut, *x; void* y; const int* rowptr; const int* cols; const void* vals; };   // 72 bytes
template <class L, int K>
struct MultiKernArgs {
    int count;
    int first_block[K + 1];
    L layer[K];
};
template <class L, int K>
__device__ __forceinline__ int layer_of_block(const MultiKernArgs<L, K>& m) {
    int l = 0;
#pragma unroll
    for (int k = 1; k < K; ++k) l += (k < m.count && (int)blockIdx.x >= m.first_block[k]) ? 1 : 0;   // uniform
    return l;
}

template <int BITS, int R, int D, int K>
__global__ void __launch_bounds__(1024) matvec_planned_multi_kernel(MultiKernArgs<PlannedLayer, K> m) {
    const int l = layer_of_block(m);
    MatvecArgs g;
    const PlannedLayer& a = m.layer[l];
    g.M = a.M; g.N = a.N; g.bits = BITS; g.B = 1; g.bt0 = 0; g.bn = 1; g.accumulate = 0; g.nnz = a.nnz;
    g.qidx = a.qidx; g.lut = a.lut; g.rowptr = nullptr; g.cols = nullptr; g.vals = nullptr; g.x = a.x; g.y = a.y; g.plan = a.plan; g.plan_c = a.plan_c;
    const int W = (g.N + kSliceCols - 1) / kSliceCols;
    if ((int)(threadIdx.x >> 6) >= W) return;
    matvec_planned_block<BITS, R, D>(g, (int)blockIdx.x - m.first_block[l], W);
}

// ---- building a plan from the CSR arrays: count the batches of every workgroup, scan the overflow, fill
__device__ __forceinline__ int plan_groups_of(int cnt) { return (cnt + 15) >> 4; }

template <int R>
__global__ void __launch_bounds__(256) plan_count_kernel(int M, int n_wg, int C, const int* __restrict__ rowptr, int* __restrict__ ov_desc) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n_wg) return;
    int groups = 0;
    for (int i = 0; i < R; ++i) {
        const int r = b * R + i;
        if (r < M) groups += plan_groups_of(rowptr[r + 1] - rowptr[r]);
    }
    const int nb = (groups + 3) >> 2;
    ov_desc[2 * b + 1] = nb > C ? nb - C : 0;
}

// exclusive scan of the overflow counts over the workgroups (one block; n_wg is a few thousand)
__global__ void __launch_bounds__(1024) plan_scan_kernel(int n_wg, int* __restrict__ ov_desc) {
    __shared__ int sums[1024];
    const int t = threadIdx.x;
    const int per = (n_wg + 1023) / 1024;
    const int lo = min(t * per, n_wg), hi = min(lo + per, n_wg);
    int s = 0;
    for (int b = lo; b < hi; ++b) s += ov_desc[2 * b + 1];
    sums[t] = s;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        const int v = t >= d ? sums[t - d] : 0;
        __syncthreads();
        sums[t] += v;
        __syncthreads();
    }
    int run = sums[t] - s;
    for (int b = lo; b < hi; ++b) { ov_desc[2 * b] = run; run += ov_desc[2 * b + 1]; }
}

// one wave per workgroup of the matvec: lane l fills entry l of every batch
template <int R>
__global__ void __launch_bounds__(64) plan_fill_kernel(int M, int C, const int* __restrict__ rowptr, const int* __restrict__ cols, const uint16_t* __restrict__ vals,
                                                       u32* __restrict__ slot_entries, uint8_t* __restrict__ slot_tags, const int* __restrict__ ov_desc,
                                                       u32* __restrict__ ov_entries, uint8_t* __restrict__ ov_tags) {
    const int b = blockIdx.x, lane = threadIdx.x;
    int gp[R + 1], rs[R + 1];                                        // first group / first nonzero of every row of the workgroup (uniform)
    gp[0] = 0;
#pragma unroll
    for (int i = 0; i <= R; ++i) rs[i] = rowptr[min(b * R + i, M)];
#pragma unroll
    for (int i = 0; i < R; ++i) gp[i + 1] = gp[i] + plan_groups_of(rs[i + 1] - rs[i]);
    const int groups = gp[R], nb = (groups + 3) >> 2;
    const int ov_first = ov_desc[2 * b];
    const int total = max(nb, C);                                    // unused slot batches are cleared
    for (int k = 0; k < total; ++k) {
        const int gidx = 4 * k + (lane >> 4);
        u32 entry = 0, tag = 0;
        if (gidx < groups) {
            int i = 0;
#pragma unroll
            for (int t = 1; t < R; ++t) i += gidx >= gp[t] ? 1 : 0;
            const int j = gidx - gp[i];
            const int left = rs[i + 1] - rs[i] - 16 * j;              // >= 1
            const int cnt = left < 16 ? left : 16;
            const int p = rs[i] + 16 * j + (lane & 15);
            if ((lane & 15) < cnt) entry = ((u32)cols[p] & 0x7FFFu) | ((u32)vals[p] << 16);
            tag = 0x80u | ((u32)(cnt - 1) << 3) | (u32)i;
        }
        if (k < C) {
            slot_entries[((size_t)b * C + k) * 64 + lane] = entry;
            if ((lane & 15) == 0) slot_tags[((size_t)b * C + k) * 4 + (lane >> 4)] = (uint8_t)tag;
        } else {
            ov_entries[((size_t)ov_first + k - C) * 64 + lane] = entry;
            if ((lane & 15) == 0) ov_tags[((size_t)ov_first + k - C) * 4 + (lane >> 4)] = (uint8_t)tag;
        }
    }
}

template <int BITS, int R, int D>
__global__ void __launch_bounds__(1024) matvec_kernel(MatvecArgs g) {
    matvec_block<BITS, R, D>(g, blockIdx.x, blockDim.x >> 6);
}

// Several independent layers in ONE launch (one activation column each): the grid is the concatenation of the layers' grids,
// workgroup b belongs to the layer l with first_block[l] <= b < first_block[l + 1].  The launch has as many waves per workgroup
// as its widest layer needs; in a narrower layer the surplus waves leave at once (a finished wave no longer takes part in the
// workgroup's barriers).  That is correct but slow -- two-wave layers in six-wave workgroups took 30 % longer than in a launch of
// their own -- so the host gives every wave count launches of its own and the early exit is only a guard.  Every layer is computed by the same code, in the same order of operations, as in a launch of its own,
// so the results are bit for bit those of separate calls -- what is saved is the launch and the ramp between them: the last
// workgroups of a layer run beside the first of the next.
template <int BITS, int R, int D, int K>
__global__ void __launch_bounds__(1024) matvec_multi_kernel(MultiKernArgs<CsrLayer, K> m) {
    const int l = layer_of_block(m);
    MatvecArgs g;
    const CsrLayer& a = m.layer[l];
    g.M = a.M; g.N = a.N; g.bits = BITS; g.B = 1; g.bt0 = 0; g.bn = 1; g.accumulate = 0; g.nnz = a.nnz;
    g.qidx = a.qidx; g.lut = a.lut; g.rowptr = a.rowptr; g.cols = a.cols; g.vals = a.vals; g.x = a.x; g.y = a.y; g.plan = nullptr;
    const int NW = (g.N + kSliceCols - 1) / kSliceCols + (g.nnz > 0 ? 1 : 0);
    if ((int)(threadIdx.x >> 6) >= NW) return;
    matvec_block<BITS, R, D>(g, (int)blockIdx.x - m.first_block[l], NW);
}

// ---------------------------------------------------------------------------------------------- standard CSR kernel
// one thread per row (the kernel the paper's App. C calls "standard")
template <int NB>
__global__ void __launch_bounds__(256) csr_rowwise_kernel(MatvecArgs g) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.M) return;
    const uint16_t* __restrict__ x = static_cast<const uint16_t*>(g.x) + g.bt0;
    const uint16_t* __restrict__ vals = static_cast<const uint16_t*>(g.vals);
    uint16_t* __restrict__ y = static_cast<uint16_t*>(g.y) + g.bt0;
    float acc[NB];
#pragma unroll
    for (int t = 0; t < NB; ++t) acc[t] = 0.f;
    if (g.nnz > 0) {
        for (int p = g.rowptr[i]; p < g.rowptr[i + 1]; ++p) {
            const int c = g.cols[p];
            const float v = half_bits_to_float(vals[p]);
#pragma unroll
            for (int t = 0; t < NB; ++t)
                if (t < g.bn) acc[t] += v * half_bits_to_float(x[(size_t)c * g.B + t]);
        }
    }
#pragma unroll
    for (int t = 0; t < NB; ++t) {
        if (t >= g.bn) continue;
        const size_t o = (size_t)i * g.B + t;
        float s = acc[t];
        if (g.accumulate) s += half_bits_to_float(y[o]);
        y[o] = float_to_half_bits(s);
    }
}

// ---------------------------------------------------------------------------------------------- expansion to fp16 (or to one byte per index)
// One wave expands up to kExpandUnits x 512 columns of a row: a lane handles eight neighbouring weights per unit, so that a wave reads a
// contiguous piece of the index stream and writes 1 KB of fp16 (512 bytes of indices) with one instruction.  Same pair tables and field
// order as the matvec; without a table the entries are the indices 0, 1, 2, ... themselves and the low bytes of the pairs are kept.
// Every wave owns its table, so nothing waits for a barrier.  Bound by the writes: 13824x5120 at 3 bits 33.2 us with indices from HBM and a
// cold output (5.1 TB/s in and out, the rate of a large copy), 28.7 where the last-level cache holds them; 57 and 52 us with 32 weights per
// lane and 16 dword stores at a stride of 64 bytes.
// Eight units of requests in flight per wave; a wider row is split evenly so that no wave gets a short rest.
constexpr int kExpandUnits = 8, kExpandWaves = 4;
// Few rows are split further, until there are eight waves per compute unit: 256x4096 2.9 us, with a wave per row 4.0 (512 waves 3.3, 1024
// and 4096 2.9); 512x4096 3.3 (1024 waves 3.5, 4096 3.5).
constexpr int kExpandMinWaves = 2048;
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));                  // the outputs need not be aligned to more than one element
typedef u32x2 u32x2_a1 __attribute__((aligned(1)));

// v[k]: the 8 BITS index bits of the eight weights of group (u0 + k) * 64 + lane, for the n units of a wave (above them: other weights' bits).
// Lanes past the row repeat its last group.  With 2 and 4 bits a unit is 128 or 256 bytes and lies in lines of its own.  With 3 bits it is
// 192 and every other line holds pieces of two units: fetched per unit, 13824x5120 took 40.0 us from HBM and 36.6 from the last-level cache
// (41.5 and 27.0 with plain loads in place of non-temporal ones).  So the wave's dwords are fetched 64 at a time and the groups read from
// LDS: 33.2 and 28.7.
constexpr int kExpandStage = 3 * kExpandUnits * kWave / 4;          // dwords of eight units at 3 bits
template <int BITS>
__device__ __forceinline__ void load_groups(const char* __restrict__ qrow, int u0, int n, int groups, int lane, u32* __restrict__ stage, u32 (&v)[kExpandUnits]) {
    if constexpr (BITS == 3) {
        const u32* q = reinterpret_cast<const u32*>(qrow) + 48 * u0;
        const int own = min(n * kWave, groups - u0 * kWave), dwords = own / 4 * 3;   // whole chunks of 32 weights: N is a multiple of 128
        u32 raw[kExpandStage / kWave];
#pragma unroll
        for (int j = 0; j < kExpandStage / kWave; ++j)
            if (64 * j < dwords) raw[j] = __builtin_nontemporal_load(q + min(64 * j + lane, dwords - 1));   // uniform branch
#pragma unroll
        for (int j = 0; j < kExpandStage / kWave; ++j)
            if (64 * j < dwords) stage[64 * j + lane] = raw[j];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int k = 0; k < kExpandUnits; ++k)
            if (k < n) {
                const int g = min(k * kWave + lane, own - 1), d = 3 * g / 4;   // bits 24 g: dword d on; the last group of a chunk ends with dword d
                v[k] = funnel_shr(stage[min(d + 1, dwords - 1)], stage[d], (24u * (u32)g) & 31u);
            }
    } else {
#pragma unroll
        for (int k = 0; k < kExpandUnits; ++k)
            if (k < n) {                                             // uniform branch
                const int g = min((u0 + k) * kWave + lane, groups - 1);
                v[k] = BITS == 4 ? __builtin_nontemporal_load(reinterpret_cast<const u32*>(qrow) + g)
                                 : (u32)__builtin_nontemporal_load(reinterpret_cast<const uint16_t*>(qrow) + g);
            }
    }
}

template <int BITS, bool INDICES>
__global__ void __launch_bounds__(kExpandWaves * kWave) expand_kernel(int M, int N, int segs, const void* __restrict__ qidx, const uint16_t* __restrict__ lut, void* __restrict__ out) {
    constexpr int K = 1 << BITS, E = TableShape<BITS>::kEntries;
    __shared__ __align__(8) u32 tables[kExpandWaves][E];
    __shared__ u32 stage[BITS == 3 ? kExpandWaves : 1][BITS == 3 ? kExpandStage : 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int id = blockIdx.x * kExpandWaves + wave, row = id / segs, seg = id - row * segs;   // uniform
    if (row >= M) return;
    const int groups = N / 8, units = (groups + kWave - 1) / kWave, per = (units + segs - 1) / segs;   // per <= kExpandUnits, and every wave has a unit
    const int u0 = seg * per, n = min(per, units - u0);
    const char* qrow = static_cast<const char*>(qidx) + (size_t)row * groups * BITS;
    u32 v[kExpandUnits];
    load_groups<BITS>(qrow, u0, n, groups, lane, stage[BITS == 3 ? wave : 0], v);
    u32* table = tables[wave];
    {
        const uint16_t* t = INDICES ? nullptr : lut + (size_t)row * K;
        const u32 kl = (u32)lane & (K - 1), lo = INDICES ? kl : t[kl];
#pragma unroll
        for (int e0 = 0; e0 < E; e0 += kWave) {
            const u32 kh = (u32)((e0 + lane) >> BITS) & (K - 1), hi = INDICES ? kh : t[kh];
            if (E >= kWave || lane < E) table[e0 + lane] = lo | (hi << 16);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int k = 0; k < kExpandUnits; ++k) {
        if (k >= n) break;                                           // uniform
        u32 p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = table[(v[k] >> (2 * BITS * i)) & (E - 1)];
        const int g = (u0 + k) * kWave + lane;
        if (g < groups) {
            if constexpr (INDICES) {
                // bytes 0 and 2 of each pair
                const u32x2 o = {__builtin_amdgcn_perm(p[1], p[0], 0x06040200u), __builtin_amdgcn_perm(p[3], p[2], 0x06040200u)};
                *reinterpret_cast<u32x2_a1*>(static_cast<uint8_t*>(out) + (size_t)row * N + (size_t)g * 8) = o;
            } else {
                *reinterpret_cast<u32x4_a2*>(static_cast<uint16_t*>(out) + (size_t)row * N + (size_t)g * 8) = u32x4{p[0], p[1], p[2], p[3]};
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------- fp16 baseline
// y = W x, W fp16 row-major.  One wave per row group; lane reads 16 bytes (8 weights) per step.
template <int NB, int RB>
__global__ void __launch_bounds__(256) fp16_gemv_kernel(int M, int N, int B, const void* wv, const void* xv, void* yv) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row0 = (blockIdx.x * (blockDim.x >> 6) + wave) * RB;
    if (row0 >= M) return;
    const uint16_t* __restrict__ w = static_cast<const uint16_t*>(wv);
    const uint16_t* __restrict__ x = static_cast<const uint16_t*>(xv);
    float acc[RB][NB];
#pragma unroll
    for (int u = 0; u < RB; ++u)
#pragma unroll
        for (int t = 0; t < NB; ++t) acc[u][t] = 0.f;
    for (int j = lane * 8; j < N; j += kWave * 8) {
        u32 xr[NB][4];
        if (NB == 1) {
            const u32x4 v = *reinterpret_cast<const u32x4*>(x + j);
            xr[0][0] = v.x; xr[0][1] = v.y; xr[0][2] = v.z; xr[0][3] = v.w;
        } else {
#pragma unroll
            for (int t = 0; t < NB; ++t)
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    xr[t][p] = t < B ? ((u32)x[(size_t)(j + 2 * p) * B + t] | ((u32)x[(size_t)(j + 2 * p + 1) * B + t] << 16)) : 0u;
        }
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            if (row0 + u >= M) continue;
            const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(w + (size_t)(row0 + u) * N + j));
            const u32 wr[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int t = 0; t < NB; ++t) acc[u][t] = __builtin_amdgcn_fdot2(as_half2(wr[p]), as_half2(xr[t][p]), acc[u][t], false);
        }
    }
    uint16_t* __restrict__ y = static_cast<uint16_t*>(yv);
#pragma unroll
    for (int u = 0; u < RB; ++u)
#pragma unroll
        for (int t = 0; t < NB; ++t) {
            const float s = wave_sum_to_lane63(acc[u][t]);
            if (lane == 63 && row0 + u < M && t < B) y[(size_t)(row0 + u) * B + t] = float_to_half_bits(s);
        }
}

// ---------------------------------------------------------------------------------------------- launchers
template <int BITS, int R, int D>
static hipError_t launch_matvec_r(const MatvecArgs& g, hipStream_t s) {
    const int W = g.qidx ? (g.N + kSliceCols - 1) / kSliceCols : 0;
    const int S = g.nnz > 0 ? (W ? 1 : kSparseOnlyWaves) : (W ? 0 : 1);
    hipLaunchKernelGGL((matvec_kernel<BITS, R, D>), dim3((g.M + R - 1) / R), dim3((W + S) * kWave), 0, s, g);
    return hipGetLastError();
}

// One activation column.  Rows per workgroup, measured at 3 bits with weights from HBM (us with 4 rows / with 8; dense, then with 0.45 %
// nonzeros from the CSR arrays, then from a plan): 4096x4096 4.4 / 5.1, 4.9 / 5.5, 4.6 / 5.2; 11008x4096 6.6 / 7.1, 7.4 / 8.3, 7.5 / 8.0;
// 8192x8192 8.6 / 8.8, 9.6 / 9.8, 9.8 / 9.4; 22016x8192 18.2 / 19.5, 20.6 / 19.9, 20.0 / 19.1; 8192x16384 14.8 / 14.4, 19.2 / 18.4, 17.9 / 17.4;
// 8192x22016 22.9 / 20.5, 25.3 / 23.4, 25.3 / 22.6; 4096x28672 16.2 / 13.3, 17.4 / 15.9, 19.8 / 16.8.  Rows of eight or more slices -- 8192x22016 with
// its 11 waves per workgroup, of which a compute unit holds only two -- want 8 rows: the fixed cost of a workgroup (tables, barriers, the
// final combination) is then spread over twice the stream.  Below that 4 rows are the better choice for narrow rows and without nonzeros.
template <int BITS>
static hipError_t launch_matvec_one(const MatvecArgs& g, hipStream_t s) {
    return g.qidx && multi_rows_per_workgroup(g.N) == 8 ? launch_matvec_r<BITS, 8, 2>(g, s) : launch_matvec_r<BITS, 4, 2>(g, s);
}

PlanLayout plan_layout(int M, int N, long long nnz) {
    PlanLayout L;
    L.R = kPlanRows;                                                // blocks of four rows, whatever the kernel's rows per workgroup
    L.n_wg = (M + L.R - 1) / L.R;
    const long long n_wg = L.n_wg;
    const long long groups = nnz / 16 + M / 2 + 1;                  // a row of c nonzeros has ceil(c / 16) groups
    const int W = (N + kSliceCols - 1) / kSliceCols;
    long long C = n_wg > 0 ? (groups * 115 / 100 + 4 * n_wg - 1) / (4 * n_wg) : 1;   // 15 % above the mean; a wave carries at most one slot batch per block
    L.C = (int)(C < 1 ? 1 : (C > W ? W : C));
    L.ov_cap = (nnz / 16 + M) / 4 + n_wg + 1;
    auto up = [](size_t v) { return (v + 255) & ~(size_t)255; };
    size_t o = 0;
    L.off_slot_entries = o; o += up((size_t)n_wg * L.C * 256);
    L.off_slot_tags = o;    o += up((size_t)n_wg * L.C * 4);
    L.off_ov_desc = o;      o += up((size_t)n_wg * 8);
    L.off_ov_entries = o;   o += up((size_t)L.ov_cap * 256);
    L.off_ov_tags = o;      o += up((size_t)L.ov_cap * 4);
    L.bytes = o;
    return L;
}

hipError_t launch_plan_build(int M, int N, long long nnz, const int* rowptr, const int* cols, const void* vals, void* plan, hipStream_t s) {
    const PlanLayout L = plan_layout(M, N, nnz);
    if (L.n_wg == 0) return hipSuccess;
    char* b = static_cast<char*>(plan);
    u32* slot_entries = reinterpret_cast<u32*>(b + L.off_slot_entries);
    uint8_t* slot_tags = reinterpret_cast<uint8_t*>(b + L.off_slot_tags);
    int* ov_desc = reinterpret_cast<int*>(b + L.off_ov_desc);
    u32* ov_entries = reinterpret_cast<u32*>(b + L.off_ov_entries);
    uint8_t* ov_tags = reinterpret_cast<uint8_t*>(b + L.off_ov_tags);
    const uint16_t* v16 = static_cast<const uint16_t*>(vals);
    hipLaunchKernelGGL((plan_count_kernel<kPlanRows>), dim3((L.n_wg + 255) / 256), dim3(256), 0, s, M, L.n_wg, L.C, rowptr, ov_desc);
    hipLaunchKernelGGL(plan_scan_kernel, dim3(1), dim3(1024), 0, s, L.n_wg, ov_desc);
    hipLaunchKernelGGL((plan_fill_kernel<kPlanRows>), dim3(L.n_wg), dim3(64), 0, s, M, L.C, rowptr, cols, v16, slot_entries, slot_tags, ov_desc, ov_entries, ov_tags);
    return hipGetLastError();
}

template <int BITS>
static hipError_t launch_matvec_planned(const MatvecArgs& g0, hipStream_t s) {
    MatvecArgs g = g0;
    g.plan_c = plan_layout(g.M, g.N, g.nnz).C;
    const int W = (g.N + kSliceCols - 1) / kSliceCols;
    if (multi_rows_per_workgroup(g.N) == 8) hipLaunchKernelGGL((matvec_planned_kernel<BITS, 8, 2>), dim3((g.M + 7) / 8), dim3(W * kWave), 0, s, g);
    else hipLaunchKernelGGL((matvec_planned_kernel<BITS, 4, 2>), dim3((g.M + 3) / 4), dim3(W * kWave), 0, s, g);
    return hipGetLastError();
}

template <int BITS, int R, int K, bool PLANNED>
static hipError_t launch_multi_k(const MultiArgs& m, hipStream_t s) {
    int total = 0, waves = 1, w2 = 1;
    typedef typename std::conditional<PLANNED, PlannedLayer, CsrLayer>::type L;
    MultiKernArgs<L, K> k;
    memset(&k, 0, sizeof k);
    k.count = m.count;
    for (int l = 0; l < m.count; ++l) {
        const LayerArgs& a = m.layer[l];
        k.first_block[l] = total;
        total += (a.M + R - 1) / R;
        w2 = max(w2, (a.N + kSliceCols - 1) / kSliceCols);
        waves = max(waves, (a.N + kSliceCols - 1) / kSliceCols + (a.nnz > 0 ? 1 : 0));
        L& d = k.layer[l];
        d.M = a.M; d.N = a.N; d.nnz = (int)a.nnz; d.qidx = a.qidx; d.lut = a.lut; d.x = a.x; d.y = a.y;
        if constexpr (PLANNED) {
            d.plan = a.plan;
            d.plan_c = plan_layout(a.M, a.N, a.nnz).C;
        } else {
            d.rowptr = a.rowptr; d.cols = a.cols; d.vals = a.vals;
        }
    }
    for (int l = m.count; l <= K; ++l) k.first_block[l] = total;
    if (total == 0) return hipSuccess;
    if constexpr (PLANNED) hipLaunchKernelGGL((matvec_planned_multi_kernel<BITS, R, 2, K>), dim3(total), dim3(w2 * kWave), 0, s, k);
    else hipLaunchKernelGGL((matvec_multi_kernel<BITS, R, 2, K>), dim3(total), dim3(waves * kWave), 0, s, k);
    return hipGetLastError();
}
template <int BITS, int R>
static hipError_t launch_multi_r(const MultiArgs& m, hipStream_t s) {
    if (m.count < 1 || m.count > kMaxLayersPerLaunch) return hipErrorInvalidValue;
    const bool planned = m.layer[0].plan != nullptr;
    for (int l = 0; l < m.count; ++l)
        if ((m.layer[l].plan != nullptr) != planned) return hipErrorInvalidValue;   // one class per launch
    if (!planned && m.count > kMaxCsrLayersPerLaunch) return hipErrorInvalidValue;
    if (m.count <= 8) return planned ? launch_multi_k<BITS, R, 8, true>(m, s) : launch_multi_k<BITS, R, 8, false>(m, s);
    return launch_multi_k<BITS, R, 16, true>(m, s);
}

int multi_rows_per_workgroup(int N) { return (N + kSliceCols - 1) / kSliceCols >= 8 ? 8 : 4; }

hipError_t launch_matvec_multi(const MultiArgs& m, int bits, int R, hipStream_t s) {
    if (R == 8) return bits == 2 ? launch_multi_r<2, 8>(m, s) : (bits == 3 ? launch_multi_r<3, 8>(m, s) : launch_multi_r<4, 8>(m, s));
    return bits == 2 ? launch_multi_r<2, 4>(m, s) : (bits == 3 ? launch_multi_r<3, 4>(m, s) : launch_multi_r<4, 4>(m, s));
}

hipError_t launch_matvec(const MatvecArgs& g, hipStream_t s) {
    // one column: the vector-ALU kernel; two or more: one launch of the batch kernel (every weight is decoded once for all
    // columns), also without a dense term
    if (g.B == 1 && g.plan && g.qidx && g.nnz > 0 && !g.accumulate)
        return g.bits == 2 ? launch_matvec_planned<2>(g, s) : (g.bits == 3 ? launch_matvec_planned<3>(g, s) : launch_matvec_planned<4>(g, s));
    if (g.B == 1) return g.bits == 2 ? launch_matvec_one<2>(g, s) : (g.bits == 3 ? launch_matvec_one<3>(g, s) : launch_matvec_one<4>(g, s));
    return launch_matvec_batch(g, s);
}

hipError_t launch_csr_rowwise(const MatvecArgs& g0, hipStream_t s) {
    const int grid = (g0.M + 255) / 256;
    for (int t0 = 0; t0 < g0.B; t0 += 8) {                           // windows of at most eight columns
        MatvecArgs g = g0;
        g.bt0 = t0; g.bn = min(8, g0.B - t0);
        if (g.bn == 1) hipLaunchKernelGGL((csr_rowwise_kernel<1>), dim3(grid), dim3(256), 0, s, g);
        else if (g.bn == 2) hipLaunchKernelGGL((csr_rowwise_kernel<2>), dim3(grid), dim3(256), 0, s, g);
        else if (g.bn <= 4) hipLaunchKernelGGL((csr_rowwise_kernel<4>), dim3(grid), dim3(256), 0, s, g);
        else hipLaunchKernelGGL((csr_rowwise_kernel<8>), dim3(grid), dim3(256), 0, s, g);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int BITS>
static void launch_expand(int M, int N, const void* qidx, const void* lut, void* idx_out, void* w_out, hipStream_t s) {
    const int units = (N + 8 * kWave - 1) / (8 * kWave);
    const int want = max((units + kExpandUnits - 1) / kExpandUnits, (kExpandMinWaves + M - 1) / M);
    const int per = (units + want - 1) / want, segs = (units + per - 1) / per;   // units per wave, the last one's may be fewer
    const dim3 grid((unsigned)((M * segs + kExpandWaves - 1) / kExpandWaves)), block(kExpandWaves * kWave);
    if (w_out) hipLaunchKernelGGL((expand_kernel<BITS, false>), grid, block, 0, s, M, N, segs, qidx, static_cast<const uint16_t*>(lut), w_out);
    else hipLaunchKernelGGL((expand_kernel<BITS, true>), grid, block, 0, s, M, N, segs, qidx, nullptr, idx_out);
}
hipError_t launch_decode(int M, int N, int bits, const void* qidx, const void* lut, void* idx_out, void* w_out, hipStream_t s) {
    constexpr int kRows = 1 << 22;                                   // per launch: waves and threads of the grid stay below 2^31
    for (int m0 = 0; m0 < M; m0 = M - m0 > kRows ? m0 + kRows : M) {
        const int m = min(kRows, M - m0);
        const void* q = static_cast<const char*>(qidx) + (size_t)m0 * N * bits / 8;
        const void* l = lut ? static_cast<const char*>(lut) + (size_t)m0 * (1 << bits) * 2 : nullptr;
        void* io = idx_out ? static_cast<char*>(idx_out) + (size_t)m0 * N : nullptr;
        void* wo = w_out ? static_cast<char*>(w_out) + (size_t)m0 * N * 2 : nullptr;
        if (bits == 2) launch_expand<2>(m, N, q, l, io, wo, s);
        else if (bits == 3) launch_expand<3>(m, N, q, l, io, wo, s);
        else launch_expand<4>(m, N, q, l, io, wo, s);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_fp16_gemv(int M, int N, int B, const void* w, const void* x, void* y, hipStream_t s) {
    constexpr int RB = 2, WAVES = 4;
    const int grid = (M + WAVES * RB - 1) / (WAVES * RB);
    if (B == 1) hipLaunchKernelGGL((fp16_gemv_kernel<1, RB>), dim3(grid), dim3(WAVES * kWave), 0, s, M, N, B, w, x, y);
    else if (B == 2) hipLaunchKernelGGL((fp16_gemv_kernel<2, RB>), dim3(grid), dim3(WAVES * kWave), 0, s, M, N, B, w, x, y);
    else if (B <= 4) hipLaunchKernelGGL((fp16_gemv_kernel<4, RB>), dim3(grid), dim3(WAVES * kWave), 0, s, M, N, B, w, x, y);
    else if (B <= 8) hipLaunchKernelGGL((fp16_gemv_kernel<8, RB>), dim3(grid), dim3(WAVES * kWave), 0, s, M, N, B, w, x, y);
    else hipLaunchKernelGGL((fp16_gemv_kernel<16, RB>), dim3(grid), dim3(WAVES * kWave), 0, s, M, N, B, w, x, y);
    return hipGetLastError();
}

}  // namespace sqllm
