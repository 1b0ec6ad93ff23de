// Offline side for gfx950: Dense-and-Sparse split and sensitivity-weighted k-means (paper Sec. 4.1-4.2) -- device code.
//
// What is computed, per weight matrix W (fp16, M x N) with per-weight sensitivities s (16-bit unsigned, the
// stand-in for the diagonal Fisher information of Eq. 4):
//   1. Thresholds (Sec. 4.2, "T_min / T_max from the percentile of the distribution"): the n_lo-th smallest and
//      the n_hi-th largest weight and the n_sens-th largest sensitivity of the whole matrix, found exactly with two
//      passes of 256-bin histograms over monotone 16-bit keys (high byte, then low byte inside the selected bin).
//   2. The split: a weight goes to the sparse matrix S iff it lies strictly outside [T_min, T_max] or its
//      sensitivity is strictly above the sensitivity threshold; S is written in CSR (count per row, scan, ordered fill).
//   3. Per output row, weighted 1-D k-means over the remaining weights (Eq. 4: minimise sum_j s_j (w_j - Q(w_j))^2
//      over 2^b values) by Lloyd iterations: equal-count start, nearest-centroid assignment, sensitivity-weighted
//      means.  Every integer decision is taken in fp32 exactly as written below and the weighted sums are exact
//      integers, so the result does not depend on the order of the additions.  The row is sorted into buckets once and
//      the iterations move the K - 1 cluster boundaries (see quant_kmeans_kernel).
//   4. fp16 tables, final indices (nearest table entry in exact arithmetic, ties to the lower index; an extracted
//      position gets the entry nearest to zero) and the packed index stream in the layout the matvec reads.
#include <hip/hip_runtime.h>
#include <atomic>
#include <stdint.h>
#include <type_traits>

#include "sqllm_buckets.h"
#include "sqllm_csr.h"
#include "sqllm_kernels.h"

namespace sqllm {

typedef uint32_t u32;
typedef unsigned long long u64;
typedef long long i64;
typedef u32 u32x4 __attribute__((ext_vector_type(4)));

// monotone key: a < b as reals  =>  key(a) < key(b)  (-0 sorts below +0)
__device__ __forceinline__ u32 half_key(u32 h) { return (h & 0x8000u) ? (~h & 0xFFFFu) : (h | 0x8000u); }
__device__ __forceinline__ u32 key_half(u32 k) { return (k & 0x8000u) ? (k & 0x7FFFu) : (~k & 0xFFFFu); }
__device__ __forceinline__ float half_bits_to_f32(u32 h) { return (float)__builtin_bit_cast(_Float16, (uint16_t)h); }
// exact value of a finite fp16 bit pattern times 2^24
__device__ __forceinline__ i64 half_to_fixed(u32 h) {
    const u32 e = (h >> 10) & 31u, m = h & 1023u;
    const i64 mag = e == 0 ? (i64)m : ((i64)(m + 1024u) << (e - 1u));
    return (h & 0x8000u) ? -mag : mag;
}

__device__ __forceinline__ u32 umin(u32 a, u32 b) { return a < b ? a : b; }
__device__ __forceinline__ u32 umax(u32 a, u32 b) { return a < b ? b : a; }
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ u32 dpp_u32(u32 old, u32 v) { return (u32)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROW_MASK, 0xF, false); }
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kRowHalfMirror = 0x141, kRowMirror = 0x140, kRowShl1 = 0x101, kRowRor8 = 0x128;
constexpr int kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114, kRowShr8 = 0x118, kRowBcast15 = 0x142, kRowBcast31 = 0x143;
// the value of the lane and of the lane in the neighbouring row of 16 (row ^ 1), or in the other half of the wave
struct Two { u32 a, b; };
__device__ __forceinline__ Two row_pair(u32 v) { const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false); return {r[0], r[1]}; }
__device__ __forceinline__ Two half_pair(u32 v) { const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false); return {r[0], r[1]}; }
struct Plain {                                                       // a 32-bit count or sum
    u32 v;
    __device__ __forceinline__ Plain operator+(const Plain& o) const { return {v + o.v}; }
    template <int CTRL, int ROW_MASK = 0xF>
    __device__ __forceinline__ Plain moved() const { return {dpp_u32<CTRL, ROW_MASK>(0, v)}; }
    __device__ __forceinline__ Plain rows_added() const { const Two t = row_pair(v); return {t.a + t.b}; }
    __device__ __forceinline__ Plain halves_added() const { const Two t = half_pair(v); return {t.a + t.b}; }
};
// sum over each group of eight lanes, in all its lanes
template <class T>
__device__ __forceinline__ T group_sum(T v) {
    v = v + v.template moved<kQuadXor1>();
    v = v + v.template moved<kQuadXor2>();
    v = v + v.template moved<kRowHalfMirror>();
    return v;
}
// sum over the lanes l, l ^ STEP, l ^ 2 STEP, ... (STEP = 8 or 16) of the wave, in all of them
template <int STEP, class T>
__device__ __forceinline__ T strided_sum(T v) {
    if constexpr (STEP == 8) v = v + v.template moved<kRowRor8>();
    v = v.rows_added();
    return v.halves_added();
}
// inclusive prefix sum over the 64 lanes
template <class T>
__device__ __forceinline__ T wave_scan(T v) {
    v = v + v.template moved<kRowShr1>();
    v = v + v.template moved<kRowShr2>();
    v = v + v.template moved<kRowShr4>();
    v = v + v.template moved<kRowShr8>();
    v = v + v.template moved<kRowBcast15, 0xA>();
    v = v + v.template moved<kRowBcast31, 0xC>();
    return v;
}

// ---------------------------------------------------------------------------------------------- thresholds and row pointers
// Workspace layout (32-bit words).  Bins are the RAW bytes of the fp16 patterns and of the sensitivities; the order of the keys is
// applied when a rank is looked up.
constexpr int kWsHist1W = 0, kWsHist1S = 256, kWsHist2 = 512 /* 3 x 256 */, kWsSel = 1280 /* 3 x (raw bin, residual rank) */,
              kWsThr = 1296 /* key_min, key_max, s_thr */, kWsDone = 1300 /* blocks finished: hist1, hist2, count */, kWsWords = 1312;
constexpr int kPassThreads = 1024, kPassBlocks = 256;                // a pass over the matrix: one block per compute unit

__global__ void __launch_bounds__(256) quant_clear_kernel(u32* ws) {
    for (int i = threadIdx.x + blockIdx.x * blockDim.x; i < kWsWords; i += blockDim.x * gridDim.x) ws[i] = 0;
}

__device__ __forceinline__ u32 load_shared(const u32* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// The last block of a launch to come here.  What the blocks hand over is written with agent-scope atomics only, which take effect in
// memory that all of the GPU sees, so it is enough that every wave waits for its own to complete before the block is counted.  The order
// atomics -> wait -> barrier -> count is pinned: the compiler moves no memory access over a release fence of any scope (this one emits
// nothing but the wait for LDS), nor the wait over the barrier; tests/test_block_handover.py looks at the emitted code.  A release at agent
// scope says the same in the language's terms, but writes back the caches as well: by one thread per block 7 us of the 158 of a 4096x4096
// call, by every wave 120.  Called by all threads of the block.
__device__ __forceinline__ bool last_block(u32* done, u32* flag /* LDS */) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) *flag = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == gridDim.x ? 1u : 0u;
    __syncthreads();
    const bool last = *flag != 0;
    if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return last;
}
// Of 256 bins whose counts the threads 0 .. 255 hold: the bin in which rank r falls and the rank inside it, written by the thread of that
// bin.  All threads of the block call this; wsum: 4 words of LDS.
__device__ __forceinline__ void select_bin(u32 mine, u32 r, u32* wsum, u32* bin_out, u32* residual_out, u32 bin) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const u32 inc = wave_scan(Plain{threadIdx.x < 256 ? mine : 0u}).v;
    if (wave < 4 && lane == 63) wsum[wave] = inc;
    __syncthreads();
    u32 before = inc - mine;
    for (int k = 0; k < wave && k < 4; ++k) before += wsum[k];
    if (threadIdx.x < 256 && r >= before && r - before < mine) { *bin_out = bin; *residual_out = r - before; }
    __syncthreads();
}
// raw high byte of the weights whose key has high byte t, and back
__device__ __forceinline__ u32 raw_high(u32 t) { return t & 0x80u ? t & 0x7Fu : ~t & 0xFFu; }
__device__ __forceinline__ u32 key_high(u32 raw) { return raw & 0x80u ? ~raw & 0xFFu : raw | 0x80u; }

// pass 1: histograms of the high bytes of all weights and of all sensitivities, then the bins that hold the three ranks (by the block
// that finishes last, instead of in a launch of its own).  Bound by the read of the matrix (67 MB at 4096x4096: 13 us of the 17.5).
__global__ void __launch_bounds__(kPassThreads) quant_hist1_kernel(long long units, const u32x4* __restrict__ w, const u32x4* __restrict__ s, u32* __restrict__ ws,
                                                                   u32 r_min, u32 r_max, u32 r_sens) {
    // 32 copies of each histogram, one per lane of half a wave and each in a bank of its own: counting never waits for a bank, whatever
    // the data.  256 blocks end with 512 global atomics each.  (Eight copies one after the other, 1024 blocks of 256 threads and a select
    // kernel behind it: 36 + 4.7 us at 4096x4096, 81 + 4.6 at 4096x11008, against 17.5 and 43.)
    extern __shared__ __align__(16) u32 h[];                         // [2][256][32]
    for (int i = threadIdx.x; i < 2 * 256 * 32 / 4; i += kPassThreads) reinterpret_cast<u32x4*>(h)[i] = u32x4{0, 0, 0, 0};
    __syncthreads();
    const u32 lane4 = 4u * (threadIdx.x & 31);
    auto count = [&](const u32x4& v, u32 base) {
        const u32 d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            // bin * 128 + base from bytes 1 and 3 of the dword
            atomicAdd(reinterpret_cast<u32*>(reinterpret_cast<char*>(h) + __builtin_amdgcn_udot4(d[k], 128u << 8, base, false)), 1u);
            atomicAdd(reinterpret_cast<u32*>(reinterpret_cast<char*>(h) + __builtin_amdgcn_udot4(d[k], 128u << 24, base, false)), 1u);
        }
    };
    const long long stride = (long long)gridDim.x * kPassThreads;
    long long i = (long long)blockIdx.x * kPassThreads + threadIdx.x;
    for (; i + stride < units; i += 2 * stride) {
        const u32x4 w0 = w[i], s0 = s[i], w1 = w[i + stride], s1 = s[i + stride];
        count(w0, lane4); count(s0, 256 * 128 + lane4);
        count(w1, lane4); count(s1, 256 * 128 + lane4);
    }
    if (i < units) { count(w[i], lane4); count(s[i], 256 * 128 + lane4); }
    __syncthreads();
    if (threadIdx.x < 512) {
        u32 t = 0;
#pragma unroll 8
        for (int c = 0; c < 32; ++c) t += h[threadIdx.x * 32 + ((c + threadIdx.x) & 31)];
        if (t) __hip_atomic_fetch_add(&ws[kWsHist1W + threadIdx.x], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!last_block(&ws[kWsDone], h)) return;
    __syncthreads();
    const u32 t = threadIdx.x & 255;
    const u32 hw = load_shared(&ws[kWsHist1W + raw_high(t)]), hs = load_shared(&ws[kWsHist1S + t]);
    select_bin(hw, r_min, h, &ws[kWsSel], &ws[kWsSel + 1], raw_high(t));
    select_bin(hw, r_max, h, &ws[kWsSel + 4], &ws[kWsSel + 5], raw_high(t));
    select_bin(hs, r_sens, h, &ws[kWsSel + 8], &ws[kWsSel + 9], t);
}

// pass 2: histograms of the low bytes inside the three selected bins, then the thresholds (23 + 4.9 us at 4096x4096 with 1024 blocks and a
// select kernel of its own, against 18)
__global__ void __launch_bounds__(kPassThreads) quant_hist2_kernel(long long units, const u32x4* __restrict__ w, const u32x4* __restrict__ s, u32* __restrict__ ws) {
    __shared__ u32 h[3][256];
    __shared__ u32 flag;
    if (threadIdx.x < 768) h[threadIdx.x >> 8][threadIdx.x & 255] = 0;
    const u32 bin_min = ws[kWsSel], bin_max = ws[kWsSel + 4], bin_s = ws[kWsSel + 8];
    __syncthreads();
    auto count = [&](const u32x4& wv, const u32x4& sv) {
        const u32 wd[4] = {wv.x, wv.y, wv.z, wv.w}, sd[4] = {sv.x, sv.y, sv.z, sv.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const u32 wb = e ? wd[k] >> 24 : (wd[k] >> 8) & 255u, sb = e ? sd[k] >> 24 : (sd[k] >> 8) & 255u;
                if (wb == bin_min) atomicAdd(&h[0][(wd[k] >> (16 * e)) & 255u], 1u);
                if (wb == bin_max) atomicAdd(&h[1][(wd[k] >> (16 * e)) & 255u], 1u);
                if (sb == bin_s) atomicAdd(&h[2][(sd[k] >> (16 * e)) & 255u], 1u);
            }
        }
    };
    const long long stride = (long long)gridDim.x * kPassThreads;
    long long i = (long long)blockIdx.x * kPassThreads + threadIdx.x;
    for (; i + stride < units; i += 2 * stride) {
        const u32x4 w0 = w[i], s0 = s[i], w1 = w[i + stride], s1 = s[i + stride];
        count(w0, s0);
        count(w1, s1);
    }
    if (i < units) count(w[i], s[i]);
    __syncthreads();
    if (threadIdx.x < 768 && h[threadIdx.x >> 8][threadIdx.x & 255])
        __hip_atomic_fetch_add(&ws[kWsHist2 + threadIdx.x], h[threadIdx.x >> 8][threadIdx.x & 255], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!last_block(&ws[kWsDone + 1], &flag)) return;
    __syncthreads();
    const u32 t = threadIdx.x & 255;
    for (int k = 0; k < 3; ++k) {
        const u32 bin = k == 0 ? bin_min : (k == 1 ? bin_max : bin_s);
        const bool down = k < 2 && (bin & 0x80u);                    // negative weights: the key's low byte is the complement
        const u32 high = k < 2 ? key_high(bin) : bin;
        u32* tmp = &h[0][0];
        select_bin(load_shared(&ws[kWsHist2 + 256 * k + (down ? 255u - t : t)]), ws[kWsSel + 4 * k + 1], tmp, &ws[kWsThr + k], tmp + 8, (high << 8) | t);
    }
}

__device__ __forceinline__ bool is_extracted(u32 wbits, u32 sv, u32 key_min, u32 key_max, u32 s_thr) {
    const u32 key = half_key(wbits);
    return key < key_min || key > key_max || sv > s_thr;
}

// pass 3: extracted entries per row, one wave per row; the last block turns the counts into row pointers
__global__ void __launch_bounds__(kPassThreads) quant_count_kernel(int M, int N, const uint16_t* __restrict__ w, const uint16_t* __restrict__ s, u32* __restrict__ ws, int* __restrict__ rowptr) {
    __shared__ u32 flag, wsum[kPassThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = blockIdx.x * (kPassThreads / 64) + wave;
    const u32 key_min = ws[kWsThr], key_max = ws[kWsThr + 1], s_thr = ws[kWsThr + 2];
    if (row < M) {
        const u32x4* wr = reinterpret_cast<const u32x4*>(w + (size_t)row * N);
        const u32x4* sr = reinterpret_cast<const u32x4*>(s + (size_t)row * N);
        u32 cnt = 0;
        for (int i = lane; i < N / 8; i += 64) {
            const u32x4 wv = wr[i], sv = sr[i];
            const u32 wd[4] = {wv.x, wv.y, wv.z, wv.w}, sd[4] = {sv.x, sv.y, sv.z, sv.w};
#pragma unroll
            for (int k = 0; k < 4; ++k)
                cnt += (u32)is_extracted(wd[k] & 0xFFFFu, sd[k] & 0xFFFFu, key_min, key_max, s_thr) + (u32)is_extracted(wd[k] >> 16, sd[k] >> 16, key_min, key_max, s_thr);
        }
        cnt = wave_scan(Plain{cnt}).v;
        if (lane == 63) __hip_atomic_store(reinterpret_cast<u32*>(&rowptr[row + 1]), cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!last_block(&ws[kWsDone + 2], &flag)) return;
    u32 carry = 0;
    for (int t0 = 0; t0 < M; t0 += 4 * kPassThreads) {               // four rows per thread and round
        const int r = t0 + 4 * threadIdx.x;
        u32 c[4], mine = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) { c[k] = r + k < M ? load_shared(reinterpret_cast<const u32*>(&rowptr[r + k + 1])) : 0u; mine += c[k]; }
        const u32 inc = wave_scan(Plain{mine}).v;
        __syncthreads();
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        u32 run = carry + inc - mine;
        for (int k = 0; k < kPassThreads / 64; ++k) {
            run += k < wave ? wsum[k] : 0u;
            carry += wsum[k];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            run += c[k];
            if (r + k < M) rowptr[r + k + 1] = (int)run;
        }
    }
    if (threadIdx.x == 0) rowptr[0] = 0;
}

// ---------------------------------------------------------------------------------------------- k-means of one row
// Exact sum of products s * w * 2^24.  Narrow rows, -128 < w < 127.9375 (the fp16 number below 128): w * 2^24 fits an int, a product is
// below 2^47 and a row's sum below 2^63; in wide rows the low and the high words of the products are summed apart.
constexpr u32 kNarrowEnd = 0x57FF;                                   // fp16 bits of 127.9375
static_assert(127.9375 * 16777216.0 < 2147483648.0 && 127.9375 * 2 > 2 * 127.875, "an int holds it, and it lies above every boundary of a narrow row");
template <bool WIDE>
struct Moment {
    i64 v;
    __device__ __forceinline__ static Moment zero() { return {0}; }
    // w24: a weight times 2^24 (exact in fp32), s: its sensitivity
    __device__ __forceinline__ static Moment product(float w24, u32 /*half*/, u32 s) { return {(i64)(int)w24 * (i64)(int)s}; }
    __device__ __forceinline__ Moment operator+(const Moment& o) const { return {v + o.v}; }
    __device__ __forceinline__ Moment operator-(const Moment& o) const { return {v - o.v}; }
    __device__ __forceinline__ double value() const { return (double)v; }
    template <int CTRL, int ROW_MASK = 0xF>
    __device__ __forceinline__ Moment moved() const {
        const u32 lo = dpp_u32<CTRL, ROW_MASK>(0, (u32)(u64)v), hi = dpp_u32<CTRL, ROW_MASK>(0, (u32)((u64)v >> 32));
        return {(i64)((u64)lo | ((u64)hi << 32))};
    }
    __device__ __forceinline__ static Moment joined(const Two& lo, const Two& hi) {
        return {(i64)(((u64)lo.a | ((u64)hi.a << 32)) + ((u64)lo.b | ((u64)hi.b << 32)))};
    }
    __device__ __forceinline__ Moment rows_added() const { return joined(row_pair((u32)(u64)v), row_pair((u32)((u64)v >> 32))); }
    __device__ __forceinline__ Moment halves_added() const { return joined(half_pair((u32)(u64)v), half_pair((u32)((u64)v >> 32))); }
};
template <>
struct Moment<true> {
    i64 lo, hi;
    __device__ __forceinline__ static Moment zero() { return {0, 0}; }
    __device__ __forceinline__ static Moment product(float /*w24*/, u32 half, u32 s) {
        const i64 p = half_to_fixed(half) * (i64)s;
        return {(i64)((u64)p & 0xFFFFFFFFull), p >> 32};
    }
    __device__ __forceinline__ Moment operator+(const Moment& o) const { return {lo + o.lo, hi + o.hi}; }
    __device__ __forceinline__ Moment operator-(const Moment& o) const { return {lo - o.lo, hi - o.hi}; }
    __device__ __forceinline__ double value() const { return (double)hi * 4294967296.0 + (double)lo; }   // both exact: one rounding
    template <int CTRL, int ROW_MASK = 0xF>
    __device__ __forceinline__ Moment moved() const {
        const Moment<false> a = Moment<false>{lo}.template moved<CTRL, ROW_MASK>(), b = Moment<false>{hi}.template moved<CTRL, ROW_MASK>();
        return {a.v, b.v};
    }
    __device__ __forceinline__ Moment rows_added() const { return {Moment<false>{lo}.rows_added().v, Moment<false>{hi}.rows_added().v}; }
    __device__ __forceinline__ Moment halves_added() const { return {Moment<false>{lo}.halves_added().v, Moment<false>{hi}.halves_added().v}; }
};
template <int W> struct U32Vec { typedef u32 type __attribute__((ext_vector_type(W))); };
template <int W> using u32vec = typename U32Vec<W>::type;
// Largest key k with 2 w(k) <= t, t between the smallest and the largest fp16 value doubled.  Half of t rounded to zero is that weight unless
// it lies above (t negative and no fp16 number doubled): then the next one down, whose bits are one higher.  0 * t is added so that -0
// counts as +0, the higher of the two keys of zero.
__device__ __forceinline__ u32 key_below(float t) {
    typedef __fp16 fp16x2 __attribute__((ext_vector_type(2)));
    const float half = __builtin_fmaf(0.5f, t, 0.f);
    const u32 h = __builtin_bit_cast(u32, __builtin_amdgcn_cvt_pkrtz(half, 0.f));
    return half_key(h + (half_bits_to_f32(h) > half ? 1u : 0u));
}

// A word of the row in LDS: fp16 bits << 16 | sensitivity
__device__ __forceinline__ float weight24(u32 word) { return half_bits_to_f32(word >> 16) * 16777216.0f; }
// Behind the row: sensitivity 0, so it adds nothing, and a weight above every boundary of the row.  In narrow rows, whose words are converted
// to integers, a finite one.
constexpr u32 kBeyondNarrow = kNarrowEnd << 16, kBeyondWide = 0x7C000000u;   // 127.9375, +infinity
constexpr int kPad = 16;                                             // words of it behind the row: a round of the iterations ends there at the latest
// float(double(sum * 2^-24) / double(mass)), mass > 0, as one correctly rounded division and one rounding to fp32 give it.  The quotient below
// is within a unit of the last place of the correctly rounded one (a reciprocal good to 2^-24, one Newton step, one correction), which
// rounds to another float only next to the middle between two; `near` says so.
__device__ __forceinline__ float mean_of(double sum, u32 mass, bool& near) {
    const double d = (double)mass;
    double r = __builtin_amdgcn_rcp(d);
    r = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
    double q = sum * r;
    q = __builtin_fma(__builtin_fma(-d, q, sum), r, q);
    near = ((u32)__builtin_bit_cast(u64, q) & 0x1FFFFFFFu) - 0x0FFFFFF8u <= 16u;   // the 29 bits that fp32 drops
    return (float)(q * 5.9604644775390625e-08);
}
// Words from which a bucket is sorted and searched instead of read through.  A round reads 16 words and a bisection step one, in about the
// same time.  At 128 words rows of 8-bit levels, whose fullest buckets hold 137, lose (4096x11008 at 4 bits 639 us, 515 at 256 words;
// 4096x11776 at 2 bits 443, 320), though some rows of 16 levels gain (451, 512); at 512 rows with buckets in between lose (8192x1024 at 2
// bits, two values 215, 130; 4096x8320 at 3 bits, 16 levels 469, 401).
constexpr int kHeavy = 256;

// One block of T threads per row.  In one dimension the clusters of Lloyd's method are intervals of the sorted weights, so an update
// only needs, for each of the K - 1 boundaries, how many weights lie below it and their exact sums.  The row is not sorted for that:
//   * it is read once; every thread keeps its weights as words (key << 16 | sensitivity) in registers until the indices are written;
//   * a counting sort puts the words, with the fp16 bits in place of the key, into NB buckets of 2^shift consecutive keys (shift from the
//     row's smallest and largest key); the
//     atomic that counts a word also gives its place in the bucket; the order inside a bucket does not matter, all sums are integers;
//   * C0 / C1 hold the sums in front of every chunk of eight words;
//   * eight lanes (four with 16 entries) evaluate a boundary: the key below it names the bucket, and the sums are those in front of the chunk
//     in which the bucket starts plus the words from there on that lie below the boundary.  A bucket holds a handful of words, so that is
//     one or two rounds of 16 words.  One wave iterates: neighbouring boundaries are neighbouring lanes, so no barrier and no LDS stand
//     between two updates;
//   * pruned, constant or already quantised rows have few keys and many words of each.  Buckets of kHeavy words or more are therefore put in
//     the order of their keys, and an update bisects them instead of reading them through (nine tenths zeros, 32 updates: 4096x11008 at 4
//     bits 0.81 ms, read through 16.3; 1024x28672 0.50 ms, read through 18.7).
// The decisions and integers are those of a pass over all weights per update, hence the same result.
// Bound by the latency of the chain boundary -> bucket -> words -> reduction -> division (1150 cycles at 4096 weights and 8 entries, 1130 at
// 11008 and 16; with 4096 buckets 1480), which the other rows on the unit cover only in part (what their LDS allows: six at 4096 weights, two
// at 11008).  It was 1570 and 1920 with the key of a boundary corrected in two steps, the two bucket ends read one after the other under a
// branch, a test in front of the first round, a full fp64 division behind the test for the end, and no priority over the waves of other rows.
// Against a bitonic sort of the row in LDS and a 64-way search per boundary with reductions over 64 lanes: 4096x4096 at 3 bits 409 us, now 89
// (22 updates per row), 4096x11008 at 4 bits 1164, now 258 (32 updates).
// Threads T, units of eight weights per thread V, buckets, words per chunk of running sums (twice as many in wide rows), and the waves per
// SIMD the registers are held down for.  All shapes but the narrowest keep scalar registers in lanes of vector registers: 17 to 19 of them with
// two units per thread, 47 to 79 with three and four.
template <int T_, int V_, int LOG_NB, int CHUNK, int WAVES>
struct KmeansShape {
    static constexpr int T = T_, V = V_, kWavesPerSimd = WAVES, kChunk = CHUNK;
    static constexpr int kMaxN = 8 * T_ * V_ < 28672 ? 8 * T_ * V_ : 28672;
    static constexpr int kLogNB = LOG_NB, NB = 1 << LOG_NB;
    // The CSR entries of a row are written while wave 0 iterates, by the threads behind it: one per 32 columns.  Where those are too few, and
    // with 1024 threads, where the two registers it takes until then are spilled (1024x28672 341 us against 330), they are written at once.
    static constexpr int kFirst = T_ <= 512 && kMaxN / 32 <= T_ - 64 ? 64 : 0;
    static constexpr int kChunksPerThread = (kMaxN / CHUNK + T_ - 1) / T_;
    static constexpr size_t sum_bytes(int N) { return ((size_t)(N / CHUNK + 1) * 12 + 15) & ~(size_t)15; }   // also holds (N / (2 CHUNK) + 1) * 20; the counters behind it are read four at a time
    // Counters of neighbouring buckets apart in the banks (spread_word).  With 4096 buckets the levels of a quantised row lie in more banks
    // anyway: 1024x28672, Student-t 298 us with it, 294 without.
    static constexpr u32 counter_word(u32 v) { return LOG_NB > 12 ? spread_word(v) : v; }
    static constexpr size_t lds(int N) { return (size_t)(N + kPad) * 4 + sum_bytes(N) + (size_t)(NB + 2) * 2; }
    // the counters of the heavy buckets, 16 bits for each of a bucket's keys (2^shift, keys have 16 bits), take the place of the sums
    static constexpr bool counters_fit() {
        for (int N = 128; N <= kMaxN; N += 128)
            if (((size_t)((N + kHeavy - 1) / kHeavy) * 2 << (16 - kLogNB)) > sum_bytes(N)) return false;
        return true;
    }
};
typedef KmeansShape<128, 1, 11, 8, 6> KmeansUpTo1024;                // 10 KB of LDS at 1024 weights: fourteen rows per compute unit
typedef KmeansShape<128, 2, 11, 8, 5> KmeansUpTo2048;                // ten rows
typedef KmeansShape<256, 2, 11, 8, 6> KmeansUpTo4096;                // 26 KB of LDS at 4096 weights: six rows per compute unit
typedef KmeansShape<256, 3, 12, 8, 4> KmeansUpTo6144;                // 36 KB at 5120: four
typedef KmeansShape<256, 4, 12, 8, 3> KmeansUpTo8192;                // 53 KB at 8192: three, which is three waves per SIMD; registers held down for
                                                                     // four spilled 11 to 14 (8192 columns, two values 442 us, now 424; Student-t 285, 272)
typedef KmeansShape<512, 3, 13, 8, 4> KmeansUpTo11776;               // 77 KB at 11008: two.  16 levels at 3 bits, 4096x11008: 502 us, with the counters
                                                                     // apart in the banks and four of them per access 475 (4096 buckets 477)
typedef KmeansShape<512, 3, 12, 8, 4> KmeansUpTo12288;
typedef KmeansShape<512, 4, 12, 8, 4> KmeansUpTo16384;
typedef KmeansShape<1024, 4, 12, 16, 4> KmeansBeyond;                // 145 KB at 28672: one (four registers spilled; 1024x28672 at 4 bits 0.29 ms)

constexpr int kMaxN11776 = 11776;
static_assert(KmeansUpTo11776::lds(kMaxN11776) + 512 <= 80 * 1024, "two rows per compute unit");

template <int BITS, class S>
__global__ void __launch_bounds__(S::T, S::kWavesPerSimd) quant_kmeans_kernel(int M, int N, int max_iter, int capacity, const uint16_t* __restrict__ w, const uint16_t* __restrict__ sens,
                                                         const u32* __restrict__ ws, const int* __restrict__ rowptr, void* __restrict__ qidx,
                                                         uint16_t* __restrict__ lut, int* __restrict__ cols, uint16_t* __restrict__ vals, int* __restrict__ iters) {
    constexpr int K = 1 << BITS, SETS = K > 8 ? K / 8 : 1;           // eight boundaries per wave
    constexpr int T = S::T, V = S::V, NB = S::NB, NBT = NB / T, NWAVES = T / 64;
    extern __shared__ __align__(16) char smem[];
    u32* A = reinterpret_cast<u32*>(smem);                           // words by bucket
    char* sums = smem + (size_t)(N + kPad) * 4;                               // sums in front of every chunk: moments, then sensitivities
    u32* start32 = reinterpret_cast<u32*>(sums + S::sum_bytes(N));   // first place of every bucket, two to a word; counts before the scan
    const uint16_t* start = reinterpret_cast<const uint16_t*>(start32);
    u32* emask = A;                                                  // bit j: weight j is extracted (A is filled after its last use)
    __shared__ u32 wsum[NWAVES];
    __shared__ i64 wmom[2 * NWAVES];
    __shared__ u32 kmm[2], crowded;                                  // smallest and largest key; is there a heavy bucket?
    __shared__ float cen_s[K];
    __shared__ u32 bound[K], nearest;

    u32* rank_bucket = bound;                                        // buckets of the start ranks, until the boundaries of the table take their place
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), row = blockIdx.x;
    const int n = lane & 7, q = lane >> 3;                           // eight lanes per boundary
    const u32 key_min = ws[kWsThr], key_max = ws[kWsThr + 1], s_thr = ws[kWsThr + 2];
    const uint16_t* __restrict__ wrow = w + (size_t)row * N;
    const int units = N / 8;

    // ---- 1. the row into registers; extracted weights become 0xFFFFFFFF
    u32 word[V][8];
    {
        const u32x4* wr = reinterpret_cast<const u32x4*>(wrow);
        const u32x4* sr = reinterpret_cast<const u32x4*>(sens + (size_t)row * N);
        u32x4 wv[V], sv[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int i = min(tid + T * v, units - 1);
            wv[v] = wr[i]; sv[v] = sr[i];
        }
        for (int b = tid; b < NB / 8; b += T) reinterpret_cast<u32x4*>(start32)[b] = u32x4{0, 0, 0, 0};
        if (tid == 0) { kmm[0] = 0xFFFFu; kmm[1] = 0; crowded = 0; nearest = 0xFFFFFFFFu; }
        u32 kmin = 0xFFFFu, kmax = 0;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const bool live = tid + T * v < units;
            const u32 wd[4] = {wv[v].x, wv[v].y, wv[v].z, wv[v].w}, sd[4] = {sv[v].x, sv[v].y, sv[v].z, sv[v].w};
            u32 mask = 0;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const u32 wb = (e & 1) ? wd[e >> 1] >> 16 : wd[e >> 1] & 0xFFFFu, sb = (e & 1) ? sd[e >> 1] >> 16 : sd[e >> 1] & 0xFFFFu;
                const u32 key = half_key(wb);
                const bool out = !live || key < key_min || key > key_max || sb > s_thr;
                word[v][e] = out ? 0xFFFFFFFFu : (key << 16) | sb;
                mask |= (out ? 1u : 0u) << e;
                kmin = umin(kmin, out ? 0xFFFFu : key);
                kmax = umax(kmax, out ? 0u : key);
            }
            if (live) reinterpret_cast<uint8_t*>(emask)[tid + T * v] = (uint8_t)mask;
        }
        __syncthreads();
#define SQ_MINMAX(CTRL, MASK) { kmin = umin(kmin, dpp_u32<CTRL, MASK>(0xFFFFu, kmin)); kmax = umax(kmax, dpp_u32<CTRL, MASK>(0u, kmax)); }
        SQ_MINMAX(kQuadXor1, 0xF) SQ_MINMAX(kQuadXor2, 0xF) SQ_MINMAX(kRowHalfMirror, 0xF) SQ_MINMAX(kRowMirror, 0xF)
        SQ_MINMAX(kRowBcast15, 0xA) SQ_MINMAX(kRowBcast31, 0xC)
#undef SQ_MINMAX
        if (lane == 63) { atomicMin(&kmm[0], kmin); atomicMax(&kmm[1], kmax); }
    }
    __syncthreads();
    const u32 kmin = (u32)__builtin_amdgcn_readfirstlane((int)kmm[0]), kmax = (u32)__builtin_amdgcn_readfirstlane((int)kmm[1]);   // kmax < kmin: no dense weight
    const u32 range = kmax >= kmin ? kmax - kmin : 0u;
    const int shift = max(0, 32 - __builtin_clz(range | 1u) - S::kLogNB);
    auto bucket_of = [&](u32 wd) { return ((wd >> 16) - kmin) >> shift; };

    // ---- 2. count the buckets; the count before gives a word its place
    u32 rank[V][4], most = 0;                                        // two to a word
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            u32 r = 0;
            if (word[v][e] != 0xFFFFFFFFu) {
                const u32 b = bucket_of(word[v][e]), sh = 16 * (b & 1);
                r = (atomicAdd(&start32[S::counter_word(b >> 1)], 1u << sh) >> sh) & 0xFFFFu;   // a bucket holds fewer than 2^15 words
            }
            rank[v][e >> 1] = (e & 1) ? rank[v][e >> 1] | (r << 16) : r;
            most = umax(most, r);
        }
    if (most >= kHeavy - 1) crowded = 1;
    const u32 ext = tid >= S::kFirst && tid - S::kFirst < N / 32 ? emask[tid - S::kFirst] : 0u;
    __syncthreads();
    // CSR entries of the row, columns ascending.  Where the inputs change under the call there may be more of them than were counted: the
    // result is wrong then, but nothing is written outside the arrays.
    int entry = 0;
    auto write_entries = [&]() {
        const int end = rowptr[row + 1];
        for (u32 m = ext; m; m &= m - 1) {
            const int j = 32 * (tid - S::kFirst) + __builtin_ctz(m);
            if (csr_has_room(entry, end, capacity)) {
                cols[entry] = j;
                vals[entry] = wrow[j];
            }
            ++entry;
        }
    };
    // ---- 3. one scan over the threads for the places of the buckets (low half) and of the CSR entries (high half); both are below 2^15
    int n_dense;
    {
        constexpr int VW = NBT / 2 < 4 ? NBT / 2 : 4;                // counters read and written at a time
        typedef u32vec<VW> vec;
        const u32 own = (u32)tid * (NBT / 2), counted = S::counter_word(own);
        u32 pair[NBT / 2], mine = 0;
#pragma unroll
        for (int k = 0; k < NBT / 2; k += VW) *reinterpret_cast<vec*>(pair + k) = *reinterpret_cast<const vec*>(start32 + counted + k);
#pragma unroll
        for (int k = 0; k < NBT / 2; ++k) { mine += (pair[k] & 0xFFFFu) + (pair[k] >> 16); }
        const u32 dense = mine;
        mine |= (u32)__builtin_popcount(ext) << 16;
        const Plain inc = wave_scan(Plain{mine});
        if (lane == 63) wsum[wave] = inc.v;
        __syncthreads();
        u32 before = inc.v - mine, total = 0;
#pragma unroll
        for (int k = 0; k < NWAVES; ++k) {
            const u32 t = wsum[k];
            before += k < wave ? t : 0u;
            total += t;
        }
        n_dense = __builtin_amdgcn_readfirstlane((int)(total & 0xFFFFu));
        u32 run = before & 0xFFFFu;
        // the buckets of the ranks the k-means starts from
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const u32 r = (u32)(((u64)(2 * k + 1) * (u64)n_dense) / (u64)(2 * K));
            if (r - run < dense) {                                   // a bucket of this thread (run <= r < run + dense)
                u32 at = run, b = 0;
#pragma unroll
                for (int i = 0; i < NBT - 1; ++i) {
                    at += (i & 1) ? pair[i >> 1] >> 16 : pair[i >> 1] & 0xFFFFu;
                    b += r >= at ? 1u : 0u;
                }
                rank_bucket[k] = tid * NBT + b;
            }
        }
#pragma unroll
        for (int k = 0; k < NBT / 2; ++k) {
            const u32 second = run + (pair[k] & 0xFFFFu), next = second + (pair[k] >> 16);
            pair[k] = run | (second << 16);
            run = next;
        }
        // behind the barrier in front of the totals: all counters have been read
#pragma unroll
        for (int k = 0; k < NBT / 2; k += VW) *reinterpret_cast<vec*>(start32 + own + k) = *reinterpret_cast<const vec*>(pair + k);
        if (tid == 0) start32[NB / 2] = (u32)n_dense;
        entry = rowptr[row] + (int)(before >> 16);
        if constexpr (S::kFirst == 0) write_entries();
    }
    __syncthreads();
    const bool heavy = __builtin_amdgcn_readfirstlane((int)crowded) != 0;   // uniform in the block
    // ---- 4. the words by bucket; those of a heavy bucket by key: a second count, over the 2^shift keys of the bucket, gives their places.
    //         A heavy bucket holds a multiple of kHeavy among its first kHeavy places, which names its counters.
    static_assert(S::counters_fit(), "");
    if (heavy && shift > 0) {
        u32* sub32 = reinterpret_cast<u32*>(sums);                   // [slots][2^shift] 16-bit counters, then first places
        const uint16_t* sub = reinterpret_cast<const uint16_t*>(sums);
        u32 least = kmin;                                            // a copy the compiler cannot see through: the words' bucket numbers are not
        asm volatile("" : "+s"(least));                              // kept in registers from one pass over them to the next
        auto counter_of = [&](u32 wd, int& i) {                      // false: not in a heavy bucket
            const u32 key = (wd >> 16) - least, b = key >> shift, p = start[b];
            i = (int)(((p + kHeavy - 1) / kHeavy << shift) | (key & ((1u << shift) - 1u)));
            return (u32)start[b + 1] - p >= (u32)kHeavy;
        };
        const int half = 1 << (shift - 1), slots = (N + kHeavy - 1) / kHeavy;   // words per bucket, buckets with counters
        for (int i = tid; i < slots * half; i += T) sub32[i] = 0;
        __syncthreads();
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                int i;
                if (word[v][e] != 0xFFFFFFFFu && counter_of(word[v][e], i)) {
                    const u32 sh = 16 * (i & 1), r = (atomicAdd(&sub32[i >> 1], 1u << sh) >> sh) & 0xFFFFu;
                    rank[v][e >> 1] = (e & 1) ? (rank[v][e >> 1] & 0xFFFFu) | (r << 16) : (rank[v][e >> 1] & 0xFFFF0000u) | r;
                }
                __builtin_amdgcn_sched_barrier(0);                   // one word after the other: no registers for several
            }
        __syncthreads();
        for (int s = tid; s < slots; s += T) {
            u32 run = 0;
            for (int i = s * half; i < (s + 1) * half; ++i) {
                const u32 c = sub32[i], second = run + (c & 0xFFFFu);
                sub32[i] = run | (second << 16);
                run = second + (c >> 16);
            }
        }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                int i;
                if (word[v][e] != 0xFFFFFFFFu && counter_of(word[v][e], i)) rank[v][e >> 1] += (u32)sub[i] << (16 * (e & 1));
                __builtin_amdgcn_sched_barrier(0);
            }
    }
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (word[v][e] != 0xFFFFFFFFu)
                A[start[bucket_of(word[v][e])] + ((e & 1) ? rank[v][e >> 1] >> 16 : rank[v][e >> 1] & 0xFFFFu)] = (key_half(word[v][e] >> 16) << 16) | (word[v][e] & 0xFFFFu);
    const bool wide = kmax >= (kNarrowEnd | 0x8000u) || kmin <= 0x27FFu;   // keys of 127.9375 and -128
    for (int j = n_dense + tid; j < N + kPad; j += T) A[j] = wide ? kBeyondWide : kBeyondNarrow;
    __syncthreads();

    int it = 0;
    auto solve = [&](auto wide_row, auto crowded_row) {
        constexpr bool WIDE = decltype(wide_row)::value, CROWDED = decltype(crowded_row)::value;   // may there be heavy buckets?
        constexpr int CW = WIDE ? 2 * S::kChunk : S::kChunk, CT = S::kChunksPerThread;
        typedef Moment<WIDE> Mom;
        const int NC = N / CW;                                       // whole chunks: N is a multiple of 128
        Mom* C1 = reinterpret_cast<Mom*>(sums);                      // [NC + 1] sum of s w 2^24 in front of chunk c
        u32* C0 = reinterpret_cast<u32*>(C1 + NC + 1);               // [NC + 1] sum of s
        Mom* wm = reinterpret_cast<Mom*>(wmom);
        // ---- 5. sums in front of every chunk; thread t owns the chunks CT t ..
        const int nchunks = (n_dense + CW - 1) / CW;
        {
            u32 s0[CT], t0 = 0;
            Mom s1[CT], t1 = Mom::zero();
#pragma unroll
            for (int k = 0; k < CT; ++k) {
                const int c = CT * tid + k;
                s0[k] = 0; s1[k] = Mom::zero();
                if (c < nchunks) {
#pragma unroll
                    for (int i = 0; i < CW / 4; ++i) {
                        const int j = CW * c + 4 * ((i + tid) & (CW / 4 - 1));   // a rotated order: neighbouring threads read different banks
                        const u32x4 v4 = *reinterpret_cast<const u32x4*>(A + j);
                        const u32 vv[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            s0[k] += vv[e] & 0xFFFFu;                // 0 past the last word
                            s1[k] = s1[k] + Mom::product(weight24(vv[e]), vv[e] >> 16, vv[e] & 0xFFFFu);
                        }
                    }
                }
                t0 += s0[k]; t1 = t1 + s1[k];
            }
            const Plain i0 = wave_scan(Plain{t0});
            const Mom i1 = wave_scan(t1);
            if (lane == 63) { wsum[wave] = i0.v; wm[wave] = i1; }
            __syncthreads();
            u32 b0 = i0.v - t0;
            Mom b1 = i1 - t1;
            for (int k = 0; k < wave; ++k) { b0 += wsum[k]; b1 = b1 + wm[k]; }   // uniform
#pragma unroll
            for (int k = 0; k < CT; ++k) {
                const int c = CT * tid + k;
                if (c <= NC) { C0[c] = b0; C1[c] = b1; }
                b0 += s0[k]; b1 = b1 + s1[k];
            }
            if (tid == T - 1 && CT * T == NC) { C0[NC] = b0; C1[NC] = b1; }
        }
        __syncthreads();
        // ---- 6. equal-count start: the key of the weight of rank r, found bit by bit inside its bucket, by the eight lanes that will work on
        //         the boundary above that centroid
        if (wave < SETS) {
            const int k0 = 8 * wave + q;
            const int kr = min(k0, K - 1);
            const int r = (int)(((u64)(2 * kr + 1) * (u64)n_dense) / (u64)(2 * K));
            const int b0 = (int)rank_bucket[kr], p0 = (int)start[b0], p1 = (int)start[b0 + 1];
            constexpr int HELD = 4;                                  // words of the bucket a lane holds in registers: 32 in all (read again for
                                                                     // every bit of the key: 2800 instead of 1800 cycles at 4096 columns)
            u32 held[HELD];
#pragma unroll
            for (int i = 0; i < HELD; ++i) {
                const int j = p0 + n + 8 * i;
                const u32 key = half_key(A[min(j, N - 1)] >> 16);
                held[i] = j < p1 ? key : 0xFFFFFFFFu;                // above every candidate
            }
            const bool sorted = CROWDED && p1 - p0 >= kHeavy;
            const bool more = __builtin_amdgcn_ballot_w64(!sorted && p1 - p0 > 8 * HELD) != 0;   // uniform
            u32 key = sorted ? half_key(A[r] >> 16) : kmin + ((u32)b0 << shift);
            for (int b = shift - 1; b >= 0; --b) {
                const u32 cand = key + (1u << b);                    // no more than r - p0 words below cand: the key is cand or above
                u32 below = 0;
#pragma unroll
                for (int i = 0; i < HELD; ++i) below += held[i] < cand ? 1u : 0u;
                if (more)
                    for (int j0 = p0 + 8 * HELD; __any(!sorted && j0 < p1); j0 += 8) {
                        const int j = j0 + n;
                        const u32 v = half_key(A[min(j, N - 1)] >> 16);
                        below += j < p1 && v < cand ? 1u : 0u;
                    }
                if (!sorted && (int)group_sum(Plain{below}).v <= r - p0) key = cand;
            }
            if (n == 0 && k0 < K) cen_s[k0] = half_bits_to_f32(key_half(key));
        }
        __syncthreads();
        if (wave != 0) return;                                       // uniform
        // ---- 7. Lloyd iterations, by one wave: lane l belongs to boundary k = l % COLS (between the centroids k and k + 1) and holds
        //         centroid k.  Neighbouring boundaries are neighbouring lanes, so centroids and sums change hands without LDS.
        constexpr int COLS = K > 8 ? 16 : 8, SUBS = 64 / COLS, WPL = 16 / SUBS;   // words per lane and round
        const int k = lane & (COLS - 1), sub = lane / COLS;
        const bool boundary = k < K - 1;
        const u32 all0 = C0[nchunks];
        const Mom all1 = C1[nchunks];
        float cen = cen_s[min(k, K - 1)];
        u32 prev = 0xFFFFFFFFu;
        __builtin_amdgcn_s_setprio(3);                               // a chain of single instructions beside blocks that have many in flight
        for (;;) {
            const float t = __fadd_rn(cen, __builtin_bit_cast(float, dpp_u32<kRowShl1>(__builtin_bit_cast(u32, cen), __builtin_bit_cast(u32, cen))));
            const u32 kk = key_below(t);
            const u32 b = (umin(umax(kk, kmin), kmax) - kmin) >> shift;
            u32 p0 = start[b], p1 = start[b + 1];                    // both reads at once, and no branch around them
            if (kk < kmin) p0 = p1 = 0;
            // 2 w <= t, with both sides scaled exactly.  It holds for all words in front of the bucket and for none behind it, which a lane
            // may read as well; behind the last word lie kPad that are above every t.
            const float t24 = t * 8388608.0f;
            if constexpr (CROWDED) {
                const bool sorted = p1 - p0 >= (u32)kHeavy;          // the words below the boundary end at `at`
                u32 at = p0, end = sorted ? p1 : p0;
                while (__any(at < end)) {
                    const u32 mid = (at + end) / 2;                  // no word of this lane is left: at == end == mid, and both stay
                    const bool below = weight24(A[mid]) <= t24;
                    at = below && at < end ? mid + 1 : at;
                    end = below ? end : mid;
                }
                if (sorted) p0 = p1 = at;
            }
            const u32 j0 = p0 & ~(u32)(CW - 1);
            const u32 c0 = C0[j0 / CW];
            const Mom c1 = C1[j0 / CW];
            u32 pos = 0, s0 = 0;
            Mom s1 = Mom::zero();
            u32 j = j0 + WPL * sub;
            do {                                                     // most updates need one round
                u32 v[WPL];
                *reinterpret_cast<u32vec<WPL>*>(v) = *reinterpret_cast<const u32vec<WPL>*>(A + umin(j, N + kPad - WPL));
#pragma unroll
                for (int i = 0; i < WPL; ++i) {
                    const float w24 = weight24(v[i]);
                    const bool in = j < (u32)(N + kPad) && w24 <= t24;
                    const u32 s = in ? v[i] & 0xFFFFu : 0u;
                    pos += in ? 1u : 0u;
                    s0 += s;
                    s1 = s1 + Mom::product(w24, v[i] >> 16, s);
                }
                j += 16;
            } while (__builtin_amdgcn_ballot_w64(j - WPL * sub < p1) != 0);
            pos = strided_sum<COLS>(Plain{pos}).v + j0;
            s0 = strided_sum<COLS>(Plain{s0}).v + c0;
            s1 = strided_sum<COLS>(s1) + c1;
            if (!boundary) { s0 = all0; s1 = all1; }
            const Plain below0 = Plain{s0}.template moved<kRowShr1>();
            const Mom below1 = s1.template moved<kRowShr1>();
            // 16 lanes: nothing moves into lane 0
            const u32 m0 = s0 - (COLS == 8 && k == 0 ? 0u : below0.v);
            const Mom m1 = COLS == 8 && k == 0 ? s1 : s1 - below1;
            bool near;
            const double sum = m1.value();
            float next = mean_of(sum, m0, near);
            if (__builtin_amdgcn_ballot_w64(boundary && pos != prev) == 0 || it == max_iter) break;   // uniform; behind the means, whose chain it does not lengthen
            if (__builtin_amdgcn_ballot_w64(near && m0 > 0) != 0) next = (float)(sum * 5.9604644775390625e-08 / (double)m0);
            prev = pos;
            if (m0 > 0) cen = next;
            ++it;
        }
        __builtin_amdgcn_s_setprio(0);
        if (lane < K) cen_s[lane] = cen;
    };
    if (n_dense > 0) {
        // One form for rows with and without heavy buckets would make an update of an ordinary 4096x11008 matrix 8 % longer; with the two-word
        // sums in all rows with heavy buckets, 1024x28672 of 8-bit levels takes 897 us instead of 623.  The ordinary form stands first: behind
        // the others it took 4 % longer.
        if (__builtin_expect(!wide && !heavy, 1)) solve(std::false_type{}, std::false_type{});
        else if (wide) solve(std::true_type{}, std::true_type{});
        else solve(std::false_type{}, std::true_type{});
    } else if (tid < K) {
        cen_s[tid] = 0.f;
    }
    if (S::kFirst != 0 && wave != 0) write_entries();               // beside the iterations
    // ---- 8. fp16 tables; an index is the number of boundaries between table entries below the weight, as keys
    __syncthreads();
    if (tid < K) {
        const uint16_t hb = __builtin_bit_cast(uint16_t, (_Float16)cen_s[tid]);
        lut[(size_t)row * K + tid] = hb;
        u32 k = 0xFFFFu;                                             // the last one: above every key
        if (tid < K - 1) {
            const uint16_t hn = __builtin_bit_cast(uint16_t, (_Float16)cen_s[tid + 1]);
            // largest key whose weight is at most the middle of the two entries, which fp64 holds exactly; +0 where it is zero
            const double mid = __builtin_fma(0.5, (double)half_bits_to_f32(hb) + (double)half_bits_to_f32(hn), 0.0);
            typedef __fp16 fp16x2 __attribute__((ext_vector_type(2)));
            const fp16x2 h2 = __builtin_amdgcn_cvt_pkrtz((float)mid, 0.f);
            const u32 h = __builtin_bit_cast(u32, h2) & 0xFFFFu;     // that weight or the next one up: one step down is a larger magnitude below zero
            const bool up = (double)half_bits_to_f32(h) > mid;
            k = half_key(h) - (up ? 1u : 0u);
        }
        bound[tid] = (k << 16) | 0xFFFFu;
        atomicMin(&nearest, ((u32)(hb & 0x7FFFu) << 4) | tid);       // the entry nearest to zero, the first of several
    }
    if (tid == 0 && iters) iters[row] = it;
    __syncthreads();
    const u32 zero = nearest & 15u;
    const char* bounds = reinterpret_cast<const char*>(bound);
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int i = tid + T * v;
        if (i >= units) continue;                                    // whole quads of lanes
        u32 at[8];                                                   // binary search over the ascending boundaries; four times the index
#pragma unroll
        for (int e = 0; e < 8; ++e) at[e] = 0;
#pragma unroll
        for (int step = K / 2; step > 0; step >>= 1)
#pragma unroll
            for (int e = 0; e < 8; ++e) at[e] += word[v][e] > *reinterpret_cast<const u32*>(bounds + at[e] + 4 * (step - 1)) ? 4u * step : 0u;
        u32 packed = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) packed |= (word[v][e] == 0xFFFFFFFFu ? zero : at[e] >> 2) << (BITS * e);
        if constexpr (BITS == 2) {
            static_cast<uint16_t*>(qidx)[(size_t)row * units + i] = (uint16_t)packed;
        } else if constexpr (BITS == 4) {
            static_cast<u32*>(qidx)[(size_t)row * units + i] = packed;
        } else {
            // four lanes hold 24 bits each: lane l of the quad writes dword l of the three
            const u32 up = dpp_u32<0x39>(0u, packed);                // quad_perm [1,2,3,0]
            const int l = lane & 3;
            const u32 d = (packed >> (8 * l)) | (up << (24 - 8 * l));
            if (l < 3) static_cast<u32*>(qidx)[((size_t)row * units + (i & ~3)) / 4 * 3 + l] = d;
        }
    }
}

// ---------------------------------------------------------------------------------------------- launcher
size_t quantize_workspace_bytes() { return (size_t)kWsWords * 4; }

// Scratch of the entry point that allocates nothing: the same 5.2 KB workspace, held by the library itself in device memory
// of every GPU the code object is loaded on.  In host code the array's name only stands for the symbol; its device address
// is asked for once per device (with that device current) and remembered.
static __device__ __align__(256) u32 scratch[kWsWords];

hipError_t quantize_static_scratch(void** out) {
    constexpr int kMaxDevices = 64;
    static std::atomic<void*> ptrs[kMaxDevices];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    void* p = dev >= 0 && dev < kMaxDevices ? ptrs[dev].load(std::memory_order_acquire) : nullptr;
    if (!p) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        if (dev >= 0 && dev < kMaxDevices) ptrs[dev].store(p, std::memory_order_release);
    }
    *out = p;
    return hipSuccess;
}

template <int BITS, class S>
static hipError_t launch_kmeans(const QuantArgs& a, hipStream_t s) {
    // the limit belongs to the current device's copy of the kernel; raising it is a host-side table update
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&quant_kmeans_kernel<BITS, S>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::lds(S::kMaxN));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((quant_kmeans_kernel<BITS, S>), dim3(a.M), dim3(S::T), S::lds(a.N), s, a.M, a.N, a.max_iter,
                       (int)(a.n_lo + a.n_hi + a.n_sens), static_cast<const uint16_t*>(a.w), static_cast<const uint16_t*>(a.sens), static_cast<const u32*>(a.workspace), a.rowptr, a.qidx,
                       static_cast<uint16_t*>(a.lut), a.cols, static_cast<uint16_t*>(a.vals), a.iters);
    return hipGetLastError();
}
template <class S>
static hipError_t launch_kmeans_bits(const QuantArgs& a, hipStream_t s) {
    return a.bits == 2 ? launch_kmeans<2, S>(a, s) : (a.bits == 3 ? launch_kmeans<3, S>(a, s) : launch_kmeans<4, S>(a, s));
}
static hipError_t launch_kmeans_shape(const QuantArgs& a, hipStream_t s) {
    switch (kmeans_columns(a.M, a.N)) {
        case 1024: return launch_kmeans_bits<KmeansUpTo1024>(a, s);
        case 2048: return launch_kmeans_bits<KmeansUpTo2048>(a, s);
        case 4096: return launch_kmeans_bits<KmeansUpTo4096>(a, s);
        case 6144: return launch_kmeans_bits<KmeansUpTo6144>(a, s);
        case 8192: return launch_kmeans_bits<KmeansUpTo8192>(a, s);
        case 11776: return launch_kmeans_bits<KmeansUpTo11776>(a, s);
        case 12288: return launch_kmeans_bits<KmeansUpTo12288>(a, s);
        case 16384: return launch_kmeans_bits<KmeansUpTo16384>(a, s);
        default: return launch_kmeans_bits<KmeansBeyond>(a, s);
    }
}

hipError_t launch_quantize(const QuantArgs& a, hipStream_t s) {
    u32* ws = static_cast<u32*>(a.workspace);
    const long long units = (long long)a.M * a.N / 8;
    const u64 total = (u64)a.M * (u64)a.N;
    const int blocks = (int)min((long long)kPassBlocks, (units + kPassThreads - 1) / kPassThreads);
    const u32x4* w4 = static_cast<const u32x4*>(a.w);
    const u32x4* s4 = static_cast<const u32x4*>(a.sens);
    constexpr int kHist1Lds = 2 * 256 * 32 * 4;
    hipLaunchKernelGGL(quant_clear_kernel, dim3(2), dim3(256), 0, s, ws);
    hipLaunchKernelGGL(quant_hist1_kernel, dim3(blocks), dim3(kPassThreads), kHist1Lds, s, units, w4, s4, ws, (u32)a.n_lo, (u32)(total - 1 - (u64)a.n_hi), (u32)(total - 1 - (u64)a.n_sens));
    hipLaunchKernelGGL(quant_hist2_kernel, dim3(blocks), dim3(kPassThreads), 0, s, units, w4, s4, ws);
    hipLaunchKernelGGL(quant_count_kernel, dim3((a.M + kPassThreads / 64 - 1) / (kPassThreads / 64)), dim3(kPassThreads), 0, s, a.M, a.N,
                       static_cast<const uint16_t*>(a.w), static_cast<const uint16_t*>(a.sens), ws, a.rowptr);
    return launch_kmeans_shape(a, s);
}

}  // namespace sqllm
