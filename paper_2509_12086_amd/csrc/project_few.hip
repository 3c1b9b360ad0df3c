// The projection o = M (x - c) for few rows (gfx950): one workgroup per 32 x 32
// block of the output, its eight waves sharing the input dims.
//
// project_kernel (device.hip) gives a wave a 64 x 64 part of the output and
// walks all input dims in it; with few rows that is a handful of workgroups,
// each waiting for its loads k-step by k-step (35 us for one row of 768
// dims, 180 us for 100 rows of 3072).  Here every wave loads its share of the
// dims at once.  Each output element still sees project_kernel's sequence of
// operations, so both give the same bits:
//   FP64 totals (ACC64): the 32-wide k-tiles are FP32 sums from zero, so they
//     are independent; the waves write their tiles' sums to LDS and all threads
//     add them to the FP64 totals in the order of the tiles;
//   FP32 accumulation: one chain over all dims, handed from wave to wave
//     through LDS, each wave's operands already split in its registers.
// ||x - c||^2 is a chain of FP64 operations per row and k half; workgroups of
// their own compute it (norm_block), the squares' roots prepared by all waves.
//
// Bound: latency, of a load from L2 per round of dims and of the chains (6
// dependent MFMAs per 16 dims; one FP64 operation per 2 dims).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "gemm_common.hpp"
#include "launch.hpp"

using saq::ProjectItem;

namespace {

constexpr int FB = 32;             // rows and columns of a block
constexpr int FW = 8;              // waves
constexpr int TILE_STEPS = 4;      // k-steps per wave and round with FP64 totals (two k-tiles)
constexpr int CHAIN_STEPS = 8;     // k-steps per wave and round in the FP32 chain
constexpr int NORM_DIMS = 128;     // dims per round of a norm block
constexpr int NORM_STRIDE = NORM_DIMS + 2;

struct ProjectFewArgs {
    ProjectItem item[SAQ_BATCH_MAX];
    int64_t first_block[SAQ_BATCH_MAX];
    int count;
};

union FewLds {
    float tile[FW * TILE_STEPS / 2][16][64];   // k-tile sums: [tile][register][lane]
    float chain[16][64];
    double root[2][FB * NORM_STRIDE];
};

// 8 consecutive values of a row from dim kb on, zero past D.  The loads are
// unconditional, at an address inside the row.
template <bool VEC>
__device__ __forceinline__ void load8(const float* __restrict__ row, int kb, int D, float (&v)[8]) {
    if (VEC) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int k = kb + 4 * q;
            const float4 x = *reinterpret_cast<const float4*>(row + (k < D ? k : 0));
            v[4 * q + 0] = k < D ? x.x : 0.f; v[4 * q + 1] = k < D ? x.y : 0.f;
            v[4 * q + 2] = k < D ? x.z : 0.f; v[4 * q + 3] = k < D ? x.w : 0.f;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float x = row[min(kb + e, D - 1)];
            v[e] = kb + e < D ? x : 0.f;
        }
    }
}
// the plan's c is zero padded to whole k-steps
template <bool VEC, bool REF>
__device__ __forceinline__ void load_center(const float* __restrict__ c, int kb, int D, float (&v)[8]) {
    if (REF) {
        load8<VEC>(c, kb, D, v);
    } else {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float4 x = *reinterpret_cast<const float4*>(c + kb + 4 * q);
            v[4 * q + 0] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
        }
    }
}

struct Operands { u32x4 a[3], b[3]; };

__device__ __forceinline__ void split_row(const float (&x)[8], const float (&c)[8], u32x4 (&a)[3]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t h0, h1, h2;
        split3(x[2 * q] - c[2 * q], x[2 * q + 1] - c[2 * q + 1], h0, h1, h2);
        a[0][q] = h0; a[1][q] = h1; a[2][q] = h2;
    }
}
// one k-step: the six products, smallest terms first
__device__ __forceinline__ floatx16 step_products(const Operands& o, floatx16 acc) {
    constexpr int TA[6] = {2, 1, 0, 1, 0, 0};
    constexpr int TB[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
    for (int u = 0; u < 6; ++u) acc = mfma_bf16(o.a[TA[u]], o.b[TB[u]], acc);
    return acc;
}

// the row's reference (the plan's c, or its list's); false: no such id
template <bool REF>
__device__ __forceinline__ bool center_of(const ProjectItem& I, int64_t row, const float*& c) {
    c = I.c;
    if (!REF) return true;
    const int32_t id = I.ref_ids != nullptr ? I.ref_ids[row] : 0;
    const bool ok = id >= 0 && id < I.n_refs;
    c = I.refs + int64_t(ok ? id : 0) * I.D;
    return ok;
}

template <int LAYOUT, bool VEC, bool REF, bool ACC64>
__device__ __forceinline__ void few_block(const ProjectItem& I, int rb, int cb, FewLds& lds) {
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ksteps = I.k_pad / SK;
    const int64_t arow = min(int64_t(rb) * FB + li, I.n - 1);
    const float* xrow = I.X + arow * I.D;
    const float* crow;
    center_of<REF>(I, arow, crow);
    // chunk (step, term): 16 bytes of column 32 cb + li, k half lh
    const u32x4* msrc = reinterpret_cast<const u32x4*>(I.M_split) + int64_t(cb / 4) * ksteps * SCB +
                        lh * TN + (cb % 4) * FB + li;
    auto load_b = [&](int kt, u32x4 (&b)[3]) {
#pragma unroll
        for (int p = 0; p < 3; ++p) b[p] = msrc[int64_t(kt) * SCB + p * 2 * TN];
    };
    const int64_t row0 = int64_t(rb) * FB;
    const int col = cb * FB + li;
    if constexpr (ACC64) {
        constexpr int ROUND = FW * TILE_STEPS;
        double tot[2] = {0.0, 0.0};                 // registers 2 wave, 2 wave + 1 of the block
        struct Raw { float x[8], c[8]; u32x4 b[3]; } g[TILE_STEPS];
        auto load = [&](int k0) {
#pragma unroll
            for (int i = 0; i < TILE_STEPS; ++i) {
                // past the last step: the last one again, its sums not added
                const int kt = min(k0 + wave * TILE_STEPS + i, ksteps - 1);
                load8<VEC>(xrow, kt * SK + 8 * lh, I.D, g[i].x);
                load_center<VEC, REF>(crow, kt * SK + 8 * lh, I.D, g[i].c);
                load_b(kt, g[i].b);
            }
        };
        load(0);
        for (int k0 = 0; k0 < ksteps; k0 += ROUND) {
#pragma unroll
            for (int j = 0; j < TILE_STEPS / 2; ++j) {
                floatx16 acc;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
                for (int i = 2 * j; i < 2 * j + 2; ++i) {
                    Operands o;
                    split_row(g[i].x, g[i].c, o.a);
#pragma unroll
                    for (int p = 0; p < 3; ++p) o.b[p] = g[i].b[p];
                    acc = step_products(o, acc);
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) lds.tile[wave * (TILE_STEPS / 2) + j][r][lane] = acc[r];
            }
            if (k0 + ROUND < ksteps) load(k0 + ROUND);
            __syncthreads();
            const int tiles = min(ROUND, ksteps - k0) / 2;     // ksteps is even
            for (int j = 0; j < tiles; ++j)
#pragma unroll
                for (int r = 0; r < 2; ++r) tot[r] += double(lds.tile[j][2 * wave + r][lane]);
            __syncthreads();
        }
        if (col < I.dk) {
            // registers 2 w, 2 w + 1: two consecutive rows
            const int64_t row = row0 + 8 * (wave >> 1) + 4 * lh + 2 * (wave & 1);
            const float v[2] = {float(tot[0]), float(tot[1])};
            if (LAYOUT == LAYOUT_TILES) {
                if (row < ((I.n + 63) & ~int64_t(63)))
                    *reinterpret_cast<float2*>(I.O + ((row >> 6) * I.ld + col) * 64 + (row & 63)) =
                        make_float2(v[0], v[1]);
            } else {
#pragma unroll
                for (int r = 0; r < 2; ++r)
                    if (row + r < I.n)
                        I.O[LAYOUT == LAYOUT_DIMS ? int64_t(col) * I.ld + row + r
                                                  : (row + r) * I.ld + col] = v[r];
            }
        }
    } else {
        constexpr int ROUND = FW * CHAIN_STEPS;
        floatx16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        for (int k0 = 0; k0 < ksteps; k0 += ROUND) {
            Operands o[CHAIN_STEPS];
            const int w0 = k0 + wave * CHAIN_STEPS;
#pragma unroll
            for (int i = 0; i < CHAIN_STEPS; ++i) {
                const int kt = min(w0 + i, ksteps - 1);
                float x[8], c[8];
                load8<VEC>(xrow, kt * SK + 8 * lh, I.D, x);
                load_center<VEC, REF>(crow, kt * SK + 8 * lh, I.D, c);
                load_b(kt, o[i].b);
                split_row(x, c, o[i].a);
            }
            const int turns = min(FW, (ksteps - k0 + CHAIN_STEPS - 1) / CHAIN_STEPS);
            for (int turn = 0; turn < turns; ++turn) {
                if (wave == turn) {
                    if (k0 + turn > 0) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[r] = lds.chain[r][lane];
                    }
#pragma unroll
                    for (int i = 0; i < CHAIN_STEPS; ++i)
                        if (w0 + i < ksteps) acc = step_products(o[i], acc);
#pragma unroll
                    for (int r = 0; r < 16; ++r) lds.chain[r][lane] = acc[r];
                }
                __syncthreads();
            }
        }
        // the block is in LDS: wave w stores registers 4 w .. 4 w + 3, four rows
        if (wave < 4 && col < I.dk) {
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = lds.chain[4 * wave + r][lane];
            store_quad<LAYOUT>(I.O, I.ld, I.n, row0 + 8 * wave + 4 * lh, col, v[0], v[1], v[2], v[3]);
        }
    }
}

// ||x - c||^2 of 32 rows: per row and k half the FP64 chain of project_kernel,
// nacc = fma(d, d, nacc) with d = x - c, over its 8 dims of every k-step, then
// the halves' sum.  All waves prepare the d of NORM_DIMS dims, the first one
// chains them.
template <bool VEC, bool REF>
__device__ __forceinline__ void norm_block(const ProjectItem& I, int rb, FewLds& lds) {
    const int t = threadIdx.x;
    // staging: thread t takes row t / 16 and dims 8 (t % 16) .. + 7 of a round
    const int64_t srow = min(int64_t(rb) * FB + (t >> 4), I.n - 1);
    const float* xrow = I.X + srow * I.D;
    const float* crow;
    center_of<REF>(I, srow, crow);
    float x[8], c[8];
    auto load = [&](int k0) {
        const int kb = k0 + 8 * (t & 15);
        load8<VEC>(xrow, kb, I.D, x);
        load8<VEC>(crow, kb, I.D, c);
    };
    load(0);
    double acc = 0.0;
    int buf = 0;
    for (int k0 = 0; k0 < I.D; k0 += NORM_DIMS, buf ^= 1) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            lds.root[buf][(t >> 4) * NORM_STRIDE + 8 * (t & 15) + e] = double(x[e]) - double(c[e]);
        if (k0 + NORM_DIMS < I.D) load(k0 + NORM_DIMS);
        __syncthreads();
        if (t < 64) {
            const double* d = lds.root[buf] + (t & 31) * NORM_STRIDE + 8 * (t >> 5);
#pragma unroll
            for (int k = 0; k < NORM_DIMS; k += SK)
#pragma unroll
                for (int e = 0; e < 8; ++e) acc = fma(d[k + e], d[k + e], acc);
        }
    }
    if (t < 64) {
        const int lo = __shfl_xor(__double2loint(acc), 32), hi = __shfl_xor(__double2hiint(acc), 32);
        const int64_t row = int64_t(rb) * FB + t;
        const float* cr;
        if (t < 32 && row < I.n)
            I.norm2[row] = center_of<REF>(I, row, cr) ? float(acc + __hiloint2double(hi, lo)) : __builtin_nanf("");
    }
}

template <int LAYOUT, bool VEC, bool REF>
__global__ __launch_bounds__(64 * FW, 1) void project_few_kernel(const ProjectFewArgs args) {
    __shared__ __attribute__((aligned(16))) FewLds lds;
    int d = 0;
    while (d + 1 < args.count && int64_t(blockIdx.x) >= args.first_block[d + 1]) ++d;
    const ProjectItem& I = args.item[d];
    const int b = int(int64_t(blockIdx.x) - args.first_block[d]);
    const int cblocks = (I.dk + FB - 1) / FB;
    const int norms = I.norm2 != nullptr ? 1 : 0;
    const int rb = b / (cblocks + norms), cb = b % (cblocks + norms) - norms;
    if (cb < 0) norm_block<VEC, REF>(I, rb, lds);
    else if (I.acc64) few_block<LAYOUT, VEC, REF, true>(I, rb, cb, lds);
    else few_block<LAYOUT, VEC, REF, false>(I, rb, cb, lds);
}

int64_t item_blocks(const ProjectItem& i) {
    // whole 64-row tiles where the caller asks for the slots past n
    const int64_t rb = i.fill ? (i.n + 63) / 64 * 2 : (i.n + FB - 1) / FB;
    return rb * ((i.dk + FB - 1) / FB + (i.norm2 != nullptr ? 1 : 0));
}

}  // namespace

namespace saq {

// Where the line lies: in rounds of 256 workgroups, one per CU, of which a launch
// takes up to the number that is no slower than project_kernel's tiles.  Those
// take about 3 us and 0.72 per k-step (0.45 in 64 x 64 tiles, 0.82 with FP32
// accumulation), nearly flat while they fit the chip at once; a round here takes
// 5.5 us and 0.13 per k-step.  Measured, us there / here (dims, accumulation,
// workgroups here): D = 64 totals, 40: 6.0 / 7.0; 128, 188: 8.7 / 7.1, 276: 8.8 / 11.9; 768,
// 200: 23 / 13, 500: 26 / 23, 640: 27 / 33; 3072, 308: 97 / 54; FP32 D = 160, 264: 12 / 16;
// 768, 210: 23 / 13, 266: 23 / 23; 960 with references, 450: 35 / 36.
// Rows without 16-byte loads have only the larger tiles there (1.2 us per
// k-step), and here 32 lanes with a row each, whose lines fall together where
// rows are a power of two apart: D = 64, 4: 6.2 / 11.6; 128, 4: 9.9 / 11.7 (one
// row: 9.5 / 6.9); FP32 D = 160, 4: 13 / 19; 333, 225: 23 / 13, 423: 23 / 22; 256, 304: 19 / 22;
// 512, 286: 35 / 26, 532: 35 / 38; 1536, 741: 116 / 111, 975: 115 / 140; 3072, 770: 233 / 216,
// 1155: 233 / 333; FP32 D = 768, 490: 78 / 50, 658: 79 / 69.
int64_t few_blocks(const ProjectItem& it) {
    const int ksteps = it.k_pad / 16;
    const bool vec = it.D % 4 == 0 &&
                     ((reinterpret_cast<uintptr_t>(it.X) | reinterpret_cast<uintptr_t>(it.refs)) & 15) == 0;
    if (ksteps < 6) return 0;
    if (vec) return ksteps < 36 ? 256 : it.acc64 ? 512 : it.refs ? 450 : 256;
    if (ksteps <= 10) return it.n <= 4 ? 256 : 0;
    return ksteps < 20 ? 256 : ksteps < (it.acc64 ? 96 : 48) ? 512 : 768;
}
bool few_rows(const ProjectItem* items, int count) {
    double share = 0.0;
    for (int i = 0; i < count; ++i) {
        const int64_t b = item_blocks(items[i]), most = few_blocks(items[i]);
        if (b > most) return false;
        share += double(b) / double(std::max<int64_t>(most, 1));
    }
    return share > 0.0 && share <= 1.0;
}

saq_status launch_project_few(const ProjectItem* items, int count, int layout, hipStream_t st) {
    ProjectFewArgs a{};
    a.count = count;
    int64_t blocks = 0;
    bool vec = true;
    const bool ref = items[0].refs != nullptr;
    for (int i = 0; i < count; ++i) {
        a.item[i] = items[i];
        a.first_block[i] = blocks;
        blocks += item_blocks(items[i]);
        vec = vec && items[i].D % 4 == 0 && (reinterpret_cast<uintptr_t>(items[i].X) & 15) == 0 &&
              (reinterpret_cast<uintptr_t>(items[i].refs) & 15) == 0;
    }
    const dim3 grid(static_cast<unsigned>(blocks)), block(64 * FW);
#define SAQ_LAUNCH_FEW(L, V, R) hipLaunchKernelGGL((project_few_kernel<L, V, R>), grid, block, 0, st, a)
#define SAQ_LAUNCH_FEW2(L, R) \
    do { if (vec) SAQ_LAUNCH_FEW(L, true, R); else SAQ_LAUNCH_FEW(L, false, R); } while (0)
    if (layout == LAYOUT_TILES) {
        if (ref) SAQ_LAUNCH_FEW2(LAYOUT_TILES, true); else SAQ_LAUNCH_FEW2(LAYOUT_TILES, false);
    } else if (layout == LAYOUT_DIMS) {
        SAQ_LAUNCH_FEW2(LAYOUT_DIMS, false);
    } else {
        if (ref) SAQ_LAUNCH_FEW2(LAYOUT_ROWS, true); else SAQ_LAUNCH_FEW2(LAYOUT_ROWS, false);
    }
#undef SAQ_LAUNCH_FEW2
#undef SAQ_LAUNCH_FEW
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? SAQ_OK : hip_status(e, "project_few_kernel launch");
}

}  // namespace saq
