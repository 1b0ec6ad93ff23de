// Dense-and-Sparse look-up-table matvec for 2 to 16 activation columns on the matrix cores -- device code for gfx950 (wave64).
//
// y[M][B] = (D + S) x[N][B] as a product of 16 x 16 tiles.  v_mfma_f32_16x16x32_f16 multiplies A (16 rows x 32 k) by B (32 k x 16
// columns): lane l = (r, q) = (l % 16, l / 16) supplies eight k of row r and the same eight k of column r, and keeps rows 4 q + e,
// e = 0..3, of column r.
//   * A workgroup owns R = 16 RG rows and all N columns.  Its first ND waves are dense waves: they deal the 128-column windows of the
//     row out among themselves (wave w takes windows w, w + ND, ...).  In a window, lane (r, q) loads the 32 indices of row r of each
//     row group at columns 128 t + 32 q + [0, 32), looks them up in that row's pair table and feeds weights 8 m .. 8 m + 7 to MFMA m
//     (m = 0..3); as B operand the same lane holds the activations of batch column r at the same 32 columns, transposed through LDS once
//     per window and used for all RG row groups.
//   * The other waves are sparse waves: they take the sparse term while the dense waves stream, so that its chain of loads (row pointers
//     -> columns and values -> activations) runs beside the dense term; what a very heavy row leaves over is shared by all waves at the
//     end.  128 consecutive nonzeros are a window too: the rows of x that their columns name take the place of 128 consecutive rows, and
//     the A operand holds value p in the row of nonzero p (the lanes of the other rows hold zero there).
//   * Accumulators of the waves are combined through LDS in a fixed order; y is rounded to fp16 once.
// Bound by what the compute units fetch: every workgroup reads all of x (67 MB through the L2s at 8192x8192 and 16 columns) beside its
// indices and the gathered rows; the LDS is busy for 45 % of the launch, the vector ALU for 35 %.  8192x8192, 3 bits, 16 columns, 0.45 %
// nonzeros: 15.4 us with the weights in the last-level cache, 18.6 from HBM (21.2 when the sparse term followed the dense one on the same waves and a nonzero's activations were gathered in 8-byte
// pieces); 13824x5120, 4 bits, 5 columns: 11.9 us, 17.2 from HBM (28.7 when batches other than 2, 4, 8, 12 and 16 picked their columns out of LDS with
// 16-bit reads, and each of 864 workgroups built its tables through LDS).
// Lanes of absent columns (r >= B) carry some other column's activations: their products only reach columns that are not stored.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "sqllm_batch_split.h"
#include "sqllm_decode.h"
#include "sqllm_kernels.h"

namespace sqllm {

typedef _Float16 half8v_t __attribute__((ext_vector_type(8)));
typedef float float4v_t __attribute__((ext_vector_type(4)));
typedef u32 u32x3 __attribute__((ext_vector_type(3)));
typedef u32x4 u32x4_a4 __attribute__((aligned(4)));
typedef u32x3 u32x3_a4 __attribute__((aligned(4)));
typedef u32x2 u32x2_a4 __attribute__((aligned(4)));
typedef __attribute__((address_space(3))) u32 lds_u32;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;

__device__ __forceinline__ void wave_fence() {                       // orders the LDS accesses of one wave
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Pair tables of a row group in LDS: entry e of row r lies at byte e * 128 + r * 4 and a second copy 64 bytes further.  Lanes with an even
// q read the first copy, lanes with an odd q the second, so the 32 lanes the LDS serves together read 32 different banks whatever their
// indices are.  (One copy: two lanes of a row share its bank, 4.5 cycles per look-up.)
template <int BITS>
__device__ __forceinline__ void entry_offsets(const LaneChunk<BITS>& c, u32 base, u32 (&a)[16]) {
#pragma unroll
    for (int p = 0; p < 16; ++p) {
        if constexpr (BITS == 4) {
            a[p] = __builtin_amdgcn_udot4(c.q[p >> 2], kEntryStride << (8 * (p & 3)), base, false);   // byte p times 128 plus base
        } else {
            constexpr int F = 2 * BITS;
            const int bit = F * p, d = bit >> 5, pos = bit & 31;
            const u32 f = pos + F <= 32 ? (c.q[d] >> pos) & ((1u << F) - 1u) : funnel_shr(c.q[(d + 1) % BITS], c.q[d], pos) & ((1u << F) - 1u);
            a[p] = (f << 7) | base;
        }
    }
}
template <int BITS>
__device__ __forceinline__ void lookup_window(const LaneChunk<BITS>& c, u32 base, u32 (&w)[16]) {
    u32 a[16];
    entry_offsets<BITS>(c, base, a);
#pragma unroll
    for (int p = 0; p < 16; ++p) w[p] = *reinterpret_cast<const lds_u32*>(a[p]);
}

// A wave's staging area (sizes: sqllm_batch_split.h).
template <int BT>
struct BatchStage {
    static constexpr bool kRotated = batch_rotated(BT);
    static constexpr int kPitch = batch_pitch(BT);
    template <int BITS>
    __device__ static u32 index_piece(int row, int part) {           // LDS offset of 16-byte piece `part` of a row
        return BITS == 4 ? 64u * (u32)row + 16u * (((u32)part + (u32)(row >> 1)) & 3u) : 48u * (u32)row + 16u * (u32)part;
    }
    template <int BITS>
    __device__ static u32 index_chunk(int row, int q) {              // LDS offset of the 32 indices of lane (row, q)
        return BITS == 4 ? index_piece<4>(row, q) : 48u * (u32)row + 4u * BITS * (u32)q;
    }
};

constexpr int kSparseWindowsPerWave = 6;                             // windows a sparse wave takes before the rest is shared by all waves

template <int BITS, int RG, int BT>
__global__ void __launch_bounds__(kMaxBatchWaves * kWave, batch_waves_per_simd(RG, BT)) matvec_batch_kernel(MatvecArgs g, int ND) {
    constexpr int R = 16 * RG, K = 1 << BITS, E = TableShape<BITS>::kEntries;
    constexpr int kWinCols = 128;
    typedef BatchStage<BT> Stage;
    extern __shared__ __align__(2048) char smem16[];                 // tables (at LDS address 0), then one staging area per dense wave; at the end the partial sums

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);       // uniform, and known to be: addresses derived from it stay in scalar registers
    const int NW = blockDim.x >> 6;
    const int r = lane & 15, q = lane >> 4;
    const int r0 = blockIdx.x * R;
    const int nrows = min(R, g.M - r0);
    const bool sparse = g.nnz > 0;
    const uint16_t* __restrict__ x = static_cast<const uint16_t*>(g.x);
    const int nwin = g.N / kWinCols;
    const bool dense_wave = wave < ND;                               // ND == 0: no dense term

    // row pointers of the lane's own row in every row group (rows past M are empty)
    int lo[RG], hi[RG];
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
        lo[rg] = sparse ? g.rowptr[min(r0 + 16 * rg + r, g.M)] : 0;
        hi[rg] = sparse ? g.rowptr[min(r0 + 16 * rg + r + 1, g.M)] : 0;
    }
    const size_t row_dwords = (size_t)g.N * BITS / 32;
    // LDS byte address of the wave's own area (uniform): indices or values, then activations
    const u32 wave_lds = dense_wave ? (u32)(RG * E) * kEntryStride + (u32)wave * (u32)batch_dense_bytes(BITS, BT)
                                    : (ND > 0 ? (u32)(RG * E) * kEntryStride : 0u) + (u32)ND * (u32)batch_dense_bytes(BITS, BT) + (u32)(wave - ND) * (u32)batch_sparse_bytes(BT);
    // Indices are fetched in pieces of 16 bytes, BITS to a row and window: piece l of a row group to lane l, row by row, so that neighbouring lanes
    // read neighbouring bytes; they reach the lanes that use them through LDS.  Fetched by those lanes themselves -- neighbouring lanes on
    // different rows -- every lane is a cache access of its own: 144 per load at 3 bits, the vector L1 busy for 65 % of the launch.
    constexpr int NP = RG;                                           // pieces per lane: 16 BITS <= 64 of a row group
    const u32x4* piece[NP];
    u32 idx_wr;
    {
        const int p = min(lane, 16 * BITS - 1), row = p / BITS, part = p % BITS;   // surplus lanes repeat the last piece
#pragma unroll
        for (int rg = 0; rg < RG; ++rg)
            piece[rg] = reinterpret_cast<const u32x4*>(static_cast<const u32*>(g.qidx) + (size_t)min(r0 + 16 * rg + row, g.M - 1) * row_dwords) + part;
        idx_wr = wave_lds + Stage::template index_piece<BITS>(row, part);
    }
    // Plain loads: a line of 128 bytes holds the windows of two or three waves, and non-temporal ones fetch it for each (8192x8192 at 16
    // columns 15.4 against 18.6 us a call, 19.2 against 20.9 with the weights coming from HBM).
    auto load_idx = [&](int t, u32x4 (&c)[NP]) {
#pragma unroll
        for (int j = 0; j < NP; ++j) c[j] = piece[j][t * BITS];
    };
    const u32 idx_rd = wave_lds + Stage::template index_chunk<BITS>(r, q);
    const u32 stage_lds = wave_lds + (dense_wave ? (u32)batch_index_bytes(BITS) : 256u);
    const u32 tab0 = (u32)r * 4u + 64u * (q & 1);
    auto load_xblock = [&](int t, u32 (&v)[16]) {
        if constexpr (Stage::kRotated) {
            // the window lies in memory as 16 BT units of 16 bytes: unit l + 64 i to lane l
            const u32x4* src = reinterpret_cast<const u32x4*>(x + (size_t)t * kWinCols * BT) + lane;
#pragma unroll
            for (int i = 0; i < BT / 4; ++i) {
                const u32x4 v4 = src[64 * i];
                v[4 * i] = v4.x; v[4 * i + 1] = v4.y; v[4 * i + 2] = v4.z; v[4 * i + 3] = v4.w;
            }
        } else {
            // lane l fetches rows 2 l and 2 l + 1 of the window: BT dwords
            const u32* src = reinterpret_cast<const u32*>(x + (size_t)t * kWinCols * BT) + (u32)lane * BT;
#pragma unroll
            for (int i = 0; i + 4 <= BT; i += 4) {
                const u32x4 v4 = *reinterpret_cast<const u32x4_a4*>(src + i);
                v[i] = v4.x; v[i + 1] = v4.y; v[i + 2] = v4.z; v[i + 3] = v4.w;
            }
            constexpr int i = BT & ~3;
            if constexpr (BT % 4 == 3) { const u32x3 t3 = *reinterpret_cast<const u32x3_a4*>(src + i); v[i] = t3.x; v[i + 1] = t3.y; v[i + 2] = t3.z; }
            if constexpr (BT % 4 == 2) { const u32x2 t2 = *reinterpret_cast<const u32x2_a4*>(src + i); v[i] = t2.x; v[i + 1] = t2.y; }
            if constexpr (BT % 4 == 1) v[i] = src[i];
        }
    };
    const u32 nb = r < BT ? (u32)r : 0u;
    // The rows of x in v (as load_xblock leaves them, or, `apart`, each of a lane's two rows from a dword of its own) go to the planes;
    // returns where the lane (r, q) finds the pairs of its 32 rows.
    auto put_x = [&](const u32 (&v)[16], auto apart) -> u32 {
        constexpr int kSecond = decltype(apart)::value ? (BT + 1) / 2 * 2 : BT;   // first half of the second row
        if constexpr (Stage::kRotated) {
            // own row k and its neighbour k ^ 1 (lane ^ 2 for 16 columns, lane ^ 1 for 8): the lane of the even row forms
            // the pair (x[k][n], x[k + 1][n]) of the even column n of each dword, the lane of the odd row that of the odd column
            const bool keven = BT == 16 ? (lane & 2) == 0 : (lane & 1) == 0;
            const u32 sel = keven ? 0x05040100u : 0x03020706u;
            // Plane n holds the 64 row pairs of column n, rotated by rot(n) dwords (planes of 100 dwords, so a
            // rotated plane needs no wrap-around).  The rotation makes BOTH sides conflict-free: the 32 lanes the LDS
            // serves together write 8 (16) consecutive row pairs of 4 (2) planes whose bank offsets 4 n + rot(n) are 0, 8,
            // 16, 24 (0, 16) apart, and 8 neighbouring lanes read 16 bytes of 8 planes whose offsets are the 8 multiples
            // of 4.  Without it every write was a 4-way conflict (counters: 61 % of the LDS cycles).
            //   16 columns: rot(n) = 4 + 4 [n%4 == 1] - 4 [n%4 == 2] + 16 [n >= 8];   8 columns: rot(n) = 12 - 4 (n / 2) + 12 (n % 2)
            const u32 odd = keven ? 0u : 1u, h = (u32)lane & 1u;
            const u32 wr = BT == 16 ? stage_lds + (8u * h + odd) * Stage::kPitch + ((u32)(lane >> 2) + 4u * odd + 16u * h) * 4u
                                    : stage_lds + odd * Stage::kPitch + ((u32)(lane >> 1) + 12u * odd) * 4u;
#pragma unroll
            for (int i = 0; i < BT / 4; ++i)
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const u32 own = v[4 * i + d];
                    const u32 other = (u32)__builtin_amdgcn_mov_dpp((int)own, BT == 16 ? 0x4E : 0xB1, 0xF, 0xF, true);   // quad_perm [2,3,0,1] / [1,0,3,2]
                    const u32 pair = __builtin_amdgcn_perm(other, own, sel);
                    const u32 off = BT == 16 ? (u32)(2 * d) * Stage::kPitch + 64u * i + 16u * (1 - (d & 1))
                                             : (u32)(2 * d) * Stage::kPitch + 128u * i + 4u * (12 - 4 * d);
                    *reinterpret_cast<lds_u32*>(wr + off) = pair;
                }
            const u32 n3 = nb & 3u;
            const u32 rot = BT == 16 ? 4u + (n3 == 1u ? 4u : 0u) - (n3 == 2u ? 4u : 0u) + 16u * (nb >> 3)
                                     : 12u - 4u * ((nb & 7u) >> 1) + 12u * (nb & 1u);
            return stage_lds + nb * Stage::kPitch + ((u32)q * 16u + rot) * 4u;
        } else {
            // halves 0 .. BT - 1 of v: row 2 l, BT halves from kSecond on: row 2 l + 1.  The pair (x[2 l][n], x[2 l + 1][n]) goes to dword l
            // of column n's plane; lane (n, q) then reads 64 bytes of plane n.
#pragma unroll
            for (int n = 0; n < BT; ++n) {
                const u32 sel = ((n & 1) ? 0x0302u : 0x0100u) | (((kSecond + n) & 1) ? 0x07060000u : 0x05040000u);
                const u32 pair = __builtin_amdgcn_perm(v[(kSecond + n) / 2], v[n / 2], sel);
                *reinterpret_cast<lds_u32*>(stage_lds + (u32)n * Stage::kPitch + (u32)lane * 4u) = pair;
            }
            return stage_lds + nb * Stage::kPitch + (u32)q * 64u;
        }
    };
    auto get_x = [&](u32 at, u32 (&xb)[16]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32x4 v4 = *reinterpret_cast<const lds_u32x4*>(at + 16u * i);
            xb[4 * i] = v4.x; xb[4 * i + 1] = v4.y; xb[4 * i + 2] = v4.z; xb[4 * i + 3] = v4.w;
        }
    };
    auto stage = [&](const u32 (&v)[16], const u32x4 (&c)[NP], u32 (&xb)[16], LaneChunk<BITS> (&d)[RG]) {
        // the row groups take turns with one area for indices: the LDS serves a wave's accesses in order
#pragma unroll
        for (int rg = 0; rg < RG; ++rg) {
            wave_fence();
            *reinterpret_cast<lds_u32x4*>(idx_wr) = c[rg];
            wave_fence();
            if constexpr (BITS == 4) { const u32x4 i4 = *reinterpret_cast<const lds_u32x4*>(idx_rd); d[rg].q[0] = i4.x; d[rg].q[1] = i4.y; d[rg].q[2] = i4.z; d[rg].q[3] = i4.w; }
            else {
#pragma unroll
                for (int k = 0; k < BITS; ++k) d[rg].q[k] = *reinterpret_cast<const lds_u32*>(idx_rd + 4 * k);
            }
        }
        const u32 at = put_x(v, std::false_type{});
        wave_fence();
        get_x(at, xb);
        wave_fence();
    };

    // ---- requested before the tables are built: the first two windows of a dense wave (ND <= nwin)
    u32x4 c0[NP], c1[NP];                                            // indices of windows ahead, as fetched
    LaneChunk<BITS> d[RG];                                           // of the current window, the lane's own
    // Activations are requested two windows ahead where the registers for them are free, else one.  (One ahead everywhere: 22016x8192, 3 bits,
    // 8 columns 39.6 against 35.1 us; 8192x8192 and smaller are the same either way, but for 12 columns, 17.8 against 18.8.)
    constexpr bool kFar = !(RG == 2 && BT >= 13);
    u32 xb[16], xv0[16], xv1[16];
    int t = wave;
    const int last_t = dense_wave ? wave + ((nwin - 1 - wave) / ND) * ND : 0;   // this wave's last window
    // ---- pair tables: thread (row, hi) writes the entries (k, hi), k = 0 .. K - 1, of its row, both copies
    if (ND > 0) {
        const u32 rho = (u32)tid % R;
        const uint16_t* lrow = static_cast<const uint16_t*>(g.lut) + (size_t)min(r0 + (int)rho, g.M - 1) * K;
        u32 tv[K / 2];
        if constexpr (K == 4) { const u32x2 v2 = *reinterpret_cast<const u32x2*>(lrow); tv[0] = v2.x; tv[1] = v2.y; }
        else {
#pragma unroll
            for (int i = 0; i < K / 8; ++i) {
                const u32x4 v4 = reinterpret_cast<const u32x4*>(lrow)[i];
                tv[4 * i] = v4.x; tv[4 * i + 1] = v4.y; tv[4 * i + 2] = v4.z; tv[4 * i + 3] = v4.w;
            }
        }
        u32 hi16 = lrow[min(tid / R, K - 1)];
        if (dense_wave) {
            load_xblock(t, xv0);
            load_idx(t, c0);
            if constexpr (kFar) load_xblock(min(t + ND, last_t), xv1);
            load_idx(min(t + ND, last_t), c1);
        }
        for (int h = tid / R; h < K; ) {
            const u32 at = (rho >> 4) * (E * kEntryStride) + (u32)h * (K * kEntryStride) + (rho & 15u) * 4u;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const u32 e = __builtin_amdgcn_perm(hi16, tv[k >> 1], (k & 1) ? 0x05040302u : 0x05040100u);
                *reinterpret_cast<lds_u32*>(at + k * kEntryStride) = e;
                *reinterpret_cast<lds_u32*>(at + k * kEntryStride + 64u) = e;
            }
            h += (int)blockDim.x / R;
            if (h < K) hi16 = lrow[h];
        }
    }
    float4v_t acc[RG];
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) acc[rg] = float4v_t{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const u32 (&w)[16], float4v_t& a4) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const half8v_t a = __builtin_bit_cast(half8v_t, u32x4{w[4 * m], w[4 * m + 1], w[4 * m + 2], w[4 * m + 3]});
            const half8v_t b = __builtin_bit_cast(half8v_t, u32x4{xb[4 * m], xb[4 * m + 1], xb[4 * m + 2], xb[4 * m + 3]});
            a4 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, a4, 0, 0, 0);
        }
    };
    // ---- the windows of the sparse term: 128 consecutive nonzeros of one row group each, the groups one after the other
    int gp[RG], wins[RG], total = 0;                                 // first nonzero, windows of every row group (uniform)
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
        gp[rg] = __builtin_amdgcn_readlane(lo[rg], 0);
        wins[rg] = window_count(gp[rg], __builtin_amdgcn_readlane(hi[rg], 15));
        total += wins[rg];
    }
    struct Entries { u32 col[4], val[2]; };
    auto find_window = [&](int f, int& rg, int& p0) {                // f < total
        rg = RG == 2 && f >= wins[0] ? 1 : 0;
        p0 = (rg == 0 ? gp[0] : gp[RG - 1]) + kWindowNonzeros * (rg == 0 ? f : f - wins[0]);
    };
    auto load_entries = [&](int f, Entries& e) {                     // positions past the row group repeat its last nonzero
        int rg, p0;
        find_window(f, rg, p0);
        const int rest = window_rest(p0, __builtin_amdgcn_readlane(rg == 0 ? hi[0] : hi[RG - 1], 15));
        const int* __restrict__ cols = g.cols + p0;                  // uniform
        const uint16_t* __restrict__ vals = static_cast<const uint16_t*>(g.vals) + p0;
        constexpr int n = BT == 16 ? 4 : 2;
#pragma unroll
        for (int i = 0; i < n; ++i) {
            const int k = BT == 16 ? (lane >> 1) + 32 * i : (BT == 8 ? lane + 64 * i : 2 * lane + i);
            e.col[i] = (u32)cols[min(k, rest)];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) e.val[i] = vals[min(2 * lane + i, rest)];
    };
    auto gather = [&](const Entries& e, u32 (&v)[16]) {              // byte offsets fit 32 bits: N * B * 2 < 2^20
        const char* xc = reinterpret_cast<const char*>(x);
        if constexpr (Stage::kRotated) {
#pragma unroll
            for (int i = 0; i < BT / 4; ++i) {
                const u32x4 v4 = *reinterpret_cast<const u32x4*>(xc + (e.col[i] * (2u * BT) + (BT == 16 ? 16u * ((u32)lane & 1u) : 0u)));
                v[4 * i] = v4.x; v[4 * i + 1] = v4.y; v[4 * i + 2] = v4.z; v[4 * i + 3] = v4.w;
            }
        } else {
            constexpr int H = (BT + 1) / 2;                          // dwords of a row; the last one of an odd batch is half used
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                // An odd batch's rows of odd columns begin in the middle of a dword.  They are read from that dword on: with the half in front,
                // rows of even columns with the half behind them (the last column is odd: N is even), which rows_to_dwords drops.
                const u32* row = reinterpret_cast<const u32*>(xc + ((e.col[k] * (2u * BT)) & ~3u));
#pragma unroll
                for (int i = 0; i + 4 <= H; i += 4) {
                    const u32x4 v4 = *reinterpret_cast<const u32x4_a4*>(row + i);
                    v[H * k + i] = v4.x; v[H * k + i + 1] = v4.y; v[H * k + i + 2] = v4.z; v[H * k + i + 3] = v4.w;
                }
                constexpr int i = H & ~3;
                if constexpr (H % 4 == 3) { const u32x3 t3 = *reinterpret_cast<const u32x3_a4*>(row + i); v[H * k + i] = t3.x; v[H * k + i + 1] = t3.y; v[H * k + i + 2] = t3.z; }
                if constexpr (H % 4 == 2) { const u32x2 t2 = *reinterpret_cast<const u32x2_a4*>(row + i); v[H * k + i] = t2.x; v[H * k + i + 1] = t2.y; }
                if constexpr (H % 4 == 1) v[H * k + i] = row[i];
            }
        }
    };
    // which of the lane's two rows begin in the middle of a dword, and the rows moved down by that half
    auto half_starts = [&](const Entries& e) -> u32 { return BT % 2 == 1 ? (e.col[0] & 1u) | ((e.col[1] & 1u) << 1) : 0u; };
    auto rows_to_dwords = [&](u32 (&v)[16], u32 odd) {
        if constexpr (BT % 2 == 1) {
            constexpr int H = (BT + 1) / 2;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const u32 by = (odd << (4 - k)) & 16u;
#pragma unroll
                for (int i = 0; i < H; ++i) v[H * k + i] = funnel_shr(v[H * k + (i + 1 < H ? i + 1 : i)], v[H * k + i], by);
            }
        }
    };
    // windows f, f + stride, ... below `end`: columns and values are requested two windows ahead, activations one
    auto sparse_windows = [&](int f, int stride, int end) {
        if (f >= end) return;                                        // uniform
        const int last_f = f + (end - 1 - f) / stride * stride;
        Entries e0, e1;
        u32 v[16], vals = 0, odd = 0;
        load_entries(f, e0);
        load_entries(min(f + stride, last_f), e1);
        gather(e0, v);
        odd = half_starts(e0);
        vals = e0.val[0] | (e0.val[1] << 16);
        for (; f < end; f += stride) {
            int wg, p0;
            find_window(f, wg, p0);
            *reinterpret_cast<lds_u32*>(wave_lds + 4u * (u32)lane) = vals;
            rows_to_dwords(v, odd);
            const u32 at = put_x(v, std::true_type{});
            gather(e1, v);                                           // the next window's
            odd = half_starts(e1);
            vals = e1.val[0] | (e1.val[1] << 16);
            load_entries(min(f + 2 * stride, last_f), e1);
            wave_fence();
            get_x(at, xb);
            u32 vw[16];
            get_x(wave_lds + 64u * (u32)q, vw);                      // the 32 values of the lane's nonzeros
            wave_fence();
            const u32 bits = window_row_bits(wg == 0 ? lo[0] : lo[RG - 1], wg == 0 ? hi[0] : hi[RG - 1], p0, q);
            u32 w[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const u32 m0 = (u32)__builtin_amdgcn_sbfe((int)bits, 2 * i, 1), m1 = (u32)__builtin_amdgcn_sbfe((int)bits, 2 * i + 1, 1);
                w[i] = vw[i] & ((m0 & 0xFFFFu) | (m1 & 0xFFFF0000u));
            }
            if (RG == 1 || wg == 0) multiply(w, acc[0]);             // uniform
            else multiply(w, acc[RG - 1]);
        }
    };
    const int NS = NW - ND;
    const int own = ND > 0 ? min(total, NS * kSparseWindowsPerWave) : total;   // windows the sparse waves take alone
    __syncthreads();
    if (dense_wave) {
        // ---- dense term: windows t, t + ND, ...  Indices are requested two windows ahead, activations two or one.  Past the wave's last window
        //      the requests repeat that window (valid addresses, results unused) instead of branching around loads.
        auto advance = [&](u32 (&xv)[16], u32x4 (&c)[NP]) {          // window t, which xv and c hold, is put in place; the next ones are requested
            stage(xv, c, xb, d);
            load_xblock(min(t + (kFar ? 2 : 1) * ND, last_t), xv);
            load_idx(min(t + 2 * ND, last_t), c);
        };
        auto window = [&]() {
            u32 w[2][16];
            lookup_window<BITS>(d[0], tab0, w[0]);
#pragma unroll
            for (int rg = 0; rg < RG; ++rg) {
                if (rg + 1 < RG) lookup_window<BITS>(d[rg + 1], tab0 + (u32)(rg + 1) * (E * kEntryStride), w[(rg + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
                multiply(w[rg & 1], acc[rg]);
                __builtin_amdgcn_sched_barrier(0);
            }
            t += ND;
        };
        for (;;) {
            advance(xv0, c0);
            window();
            if (t >= nwin) break;
            if constexpr (kFar) advance(xv1, c1);
            else advance(xv0, c1);
            window();
            if (t >= nwin) break;
        }
    } else {
        sparse_windows(wave - ND, NS, own);
    }
    if (own < total) sparse_windows(own + wave, NW, total);          // uniform
    __syncthreads();

    // ---- combine the waves' accumulators in a fixed order: lane (r, q) holds rows 4 q + e of column r
    float* part = reinterpret_cast<float*>(smem16);                  // [wave][row][column]
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
        const float v[4] = {acc[rg].x, acc[rg].y, acc[rg].z, acc[rg].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) part[(wave * R + 16 * rg + 4 * q + e) * 16 + r] = v[e];
    }
    __syncthreads();
    uint16_t* __restrict__ y = static_cast<uint16_t*>(g.y);
    for (int o = tid; o < R * 16; o += blockDim.x) {
        const int row = o >> 4, n = o & 15;
        if (row < nrows && n < BT) {
            float sum = 0.f;
            for (int wv = 0; wv < NW; ++wv) sum += part[wv * R * 16 + o];
            const size_t yo = (size_t)(r0 + row) * BT + n;
            if (g.accumulate) sum += half_bits_to_float(y[yo]);
            y[yo] = float_to_half_bits(sum);
        }
    }
}

// ---------------------------------------------------------------------------------------------- launcher
// Rows and waves per workgroup: batch_split.
template <int BITS, int RG, int BT>
static hipError_t launch_batch_r(const MatvecArgs& g, const BatchSplit& b, hipStream_t s) {
    if (b.lds > 64 * 1024) {
        // the attribute belongs to the current device's copy of the kernel; the call is a host-side table update
        const hipError_t ea = hipFuncSetAttribute(reinterpret_cast<const void*>(&matvec_batch_kernel<BITS, RG, BT>), hipFuncAttributeMaxDynamicSharedMemorySize, kUnitLds);
        if (ea != hipSuccess) return ea;
    }
    hipLaunchKernelGGL((matvec_batch_kernel<BITS, RG, BT>), dim3(b.blocks), dim3((b.dense_waves + b.sparse_waves) * kWave), b.lds, s, g, b.dense_waves);
    return hipGetLastError();
}
template <int BITS, int RG>
static hipError_t launch_batch_b(const MatvecArgs& g, const BatchSplit& b, hipStream_t s) {
    switch (g.B) {
#define SQ_B(n) case n: return launch_batch_r<BITS, RG, n>(g, b, s);
        SQ_B(2) SQ_B(3) SQ_B(4) SQ_B(5) SQ_B(6) SQ_B(7) SQ_B(8) SQ_B(9) SQ_B(10) SQ_B(11) SQ_B(12) SQ_B(13) SQ_B(14) SQ_B(15) SQ_B(16)
#undef SQ_B
        default: return hipErrorInvalidValue;
    }
}
template <int BITS>
static hipError_t launch_batch(const MatvecArgs& g, hipStream_t s) {
    const BatchSplit b = batch_split(g.M, g.N, BITS, g.B, g.qidx != nullptr, g.nnz > 0);
    return b.row_groups == 2 ? launch_batch_b<BITS, 2>(g, b, s) : launch_batch_b<BITS, 1>(g, b, s);
}

hipError_t launch_matvec_batch(const MatvecArgs& g, hipStream_t s) {
    return g.bits == 2 ? launch_batch<2>(g, s) : (g.bits == 3 ? launch_batch<3>(g, s) : launch_batch<4>(g, s));
}

}  // namespace sqllm
