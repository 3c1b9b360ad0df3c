// What the projection kernels share: operand types, the exact three-term bf16
// split, the output layouts and the per-record references.  Device code,
// included by the translation units that hold the kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "plan.hpp"

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int TN = saq::kGemmTileN;   // 128 kept dims per tile
constexpr int SK = saq::kSplitK;              // input dims per k-step
constexpr int SCB = saq::kSplitChunks;        // B chunks per buffer

enum { LAYOUT_ROWS = 0, LAYOUT_DIMS = 1, LAYOUT_TILES = 2 };

// Per-record reference vectors (Section 3.1's c; the IVF centroid of each
// record's list in the paper's experiments): record i is centered on row
// ids[i] of refs [K x D] (all records on row 0 when ids is null) instead of
// the plan's c.  A record whose id is outside [0, K) is centered on row 0 and
// gets a NaN norm, so its factors show it.
struct RefRows {
    const float* refs;   // null: the plan's c
    const int32_t* ids;
    int32_t K;
};

// Stores rows row .. row+3 of column col of O in the output layout.
template <int LAYOUT>
__device__ __forceinline__ void store_quad(float* __restrict__ O, int64_t ld, int64_t n, int64_t row,
                                           int col, float v0, float v1, float v2, float v3) {
    if (LAYOUT == LAYOUT_TILES) {
        // whole 64-row tiles: rows of the last tile past n (copies of row
        // n-1) are stored too
        if (row < ((n + 63) & ~int64_t(63))) {
            float* dst = O + ((row >> 6) * ld + col) * 64 + (row & 63);
            *reinterpret_cast<float4*>(dst) = make_float4(v0, v1, v2, v3);
        }
    } else if (LAYOUT == LAYOUT_DIMS) {
        float* dst = O + int64_t(col) * ld + row;
        if (row + 3 < n) {
            *reinterpret_cast<float4*>(dst) = make_float4(v0, v1, v2, v3);
        } else {
            if (row + 0 < n) dst[0] = v0;
            if (row + 1 < n) dst[1] = v1;
            if (row + 2 < n) dst[2] = v2;
            if (row + 3 < n) dst[3] = v3;
        }
    } else {
        if (row + 0 < n) O[(row + 0) * ld + col] = v0;
        if (row + 1 < n) O[(row + 1) * ld + col] = v1;
        if (row + 2 < n) O[(row + 2) * ld + col] = v2;
        if (row + 3 < n) O[(row + 3) * ld + col] = v3;
    }
}

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    const bf16x2 v = {static_cast<__bf16>(a), static_cast<__bf16>(b)};
    return __builtin_bit_cast(uint32_t, v);
}
// (a, b) -> three packed bf16 pairs, a = a0 + a1 + a2 exactly (normal a)
__device__ __forceinline__ void split3(float a, float b, uint32_t& h0, uint32_t& h1, uint32_t& h2) {
    h0 = pack_bf16x2(a, b);
    const float ra = a - __uint_as_float(h0 << 16), rb = b - __uint_as_float(h0 & 0xffff0000u);
    h1 = pack_bf16x2(ra, rb);
    h2 = pack_bf16x2(ra - __uint_as_float(h1 << 16), rb - __uint_as_float(h1 & 0xffff0000u));
}
__device__ __forceinline__ floatx16 mfma_bf16(u32x4 a, u32x4 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

}  // namespace
