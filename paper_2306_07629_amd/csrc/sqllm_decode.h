// Device code shared by the one-column and the batch kernels: the index stream of a row and the shape of its pair tables.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sqllm {

typedef _Float16 half_t;
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32;
typedef u32 u32x4 __attribute__((ext_vector_type(4)));
typedef u32 u32x2 __attribute__((ext_vector_type(2)));

constexpr int kWave = 64;
constexpr int kLaneElems = 32;                      // indices per lane per row
constexpr int kSliceCols = kWave * kLaneElems;      // 2048 columns per wave
constexpr int kMaxDenseWaves = 14;                  // N <= 28672 (two more waves of the block take the sparse term)

// ---------------------------------------------------------------------------------------------- helpers
__device__ __forceinline__ u32 funnel_shr(u32 hi, u32 lo, u32 sh) { return __builtin_amdgcn_alignbit(hi, lo, sh); }
__device__ __forceinline__ half2_t as_half2(u32 v) { return __builtin_bit_cast(half2_t, v); }
__device__ __forceinline__ float half_bits_to_float(uint16_t h) { return (float)__builtin_bit_cast(half_t, h); }
__device__ __forceinline__ uint16_t float_to_half_bits(float f) { return __builtin_bit_cast(uint16_t, (half_t)f); }

// ---------------------------------------------------------------------------------------------- index stream
// A lane's share of one row: BITS dwords = 32 indices.
template <int BITS>
struct LaneChunk {
    u32 q[BITS];
};

template <int BITS>
__device__ __forceinline__ LaneChunk<BITS> load_chunk(const u32* __restrict__ p) {
    LaneChunk<BITS> c;
#pragma unroll
    for (int k = 0; k < BITS; ++k) c.q[k] = __builtin_nontemporal_load(p + k);
    return c;
}

template <int BITS>
struct TableShape {
    static constexpr int kEntryBits = 2 * BITS;               // a table entry holds the pair of two neighbouring indices: 4, 6 or 8 bits
    static constexpr int kEntries = 1 << kEntryBits;          // 16, 64 or 256
    static constexpr int kTableDwords = kEntries;             // LDS dwords of one row's table (one dword = two fp16 per entry)
    static constexpr int kRowBytes = 2 << BITS;               // bytes of one row's fp16 table: 8, 16 or 32
    static constexpr int kRawUnit = kRowBytes < 16 ? kRowBytes : 16;   // bytes of fp16 table one lane fetches
};

}  // namespace sqllm
