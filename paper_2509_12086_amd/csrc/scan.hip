// Estimate scan of libsaq.so (gfx950): Section 3.2's estimator over packed
// records, with its C-ABI entry points.
//
//   dist2[q][i] = ||o_i||^2 + ||q - c||^2 - 2 sum_s f_s <u_s(i), q'_s>
//
// The inner products run on the 8-bit integer matrix cores
// (v_mfma_i32_32x32x32_i8) and are exact: a record's codes are at most 8 bits
// per pass as they are stored, so they need no conversion to floating point,
// and a query is written once per scan as four signed 8-bit digits of a
// 31-bit fixed-point number,
//   q'_j = 2^(e - k_s - 30) (2^24 d0 + 2^16 d1 + 2^8 d2 + d3),   2^(e - 1) <= max_j 2^k_s |q'_j| < 2^e,
// with the query's exponent e and shifts k_s of the plan's segments, which
// follow the spread of their dims: components are rounded to at most 2^(3 - 30)
// of the largest, and to 2^-30 of it for queries spread like the data.  As
// independent roundings add up that is 2^-27 ||q - c|| ||o|| at most for an
// orthonormal M, an eighth of FP32's rounding of the estimate.  Plans whose rows of M differ in length run on split bf16 operands
// (even_rows).  The 32-bit integer sums over a segment carry no rounding at
// all; FP32 enters where a segment ends.
//
// Codes as bytes.  A pass covers at most 8 bit planes of one segment.  With
// b < 8 planes the byte holds the code in its top bits, the first plane
// inverted and a one below the last plane, which as a signed number is
//   2^(7 - b) (2c - (2^b - 1)) = 2^(8 - b) (c - h),   h = (2^b - 1)/2,
// so the estimator's c - h itself is the operand.  With 8 planes the byte is
// c - 128 = (c - h) - 1/2, and half the query's sum over the segment is added
// where the pass ends.  More planes than one pass takes are split in groups,
// c - h = sum_g 2^(planes below group g) (c_g - h_g).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <new>
#include <type_traits>
#include <vector>

#include "launch.hpp"

using saq::SegEntry;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x16 __attribute__((ext_vector_type(16)));

namespace {

constexpr int NXCD = 8;         // MI355X: 8 XCDs, workgroups dealt round-robin
constexpr int WR = 32;          // records per wave
constexpr int WAVES = 4;        // waves per workgroup
constexpr int TR = WR * WAVES;  // records per workgroup
constexpr int TQ = 64;          // queries per tile (32 when at most 32 are scanned)
constexpr int SD = 64;          // kept dims per step: one 32-bit plane word per lane half
constexpr int ND = 4;           // 8-bit digits of a query value
constexpr int QEXP = 30;        // a query's largest value is below 2^QEXP in fixed point
// Steps after which the integer sums are folded into the FP32 totals: the
// pairs of digit sums are joined in 32 bits, 256 W 2^14 + W 2^14 < 2^31 with
// W = 384 dims.
constexpr int FOLD_STEPS = 6;
constexpr size_t RES_BYTES = 20480; // most LDS that resident queries take
// 32-byte loads per record and group of passes: MAXNL, or MIN_LOADS where that
// covers every pass; SPAN: the bytes that MAXNL loads cover wherever the first
// one falls in a 16-byte unit
constexpr int MIN_LOADS = 4, MAXNL = 8;
constexpr int SPAN = 32 * MAXNL - 15;
constexpr int OVER = 64;        // a pass's units end less than this past its record

inline __host__ __device__ int seg_steps(int W) { return (W + SD - 1) / SD; }

inline __host__ __device__ int padded_queries(int nq) { return (nq + TQ - 1) / TQ * TQ; }

// Bits of a B-bit segment that the scan reads: all of them, or the first
// `prefix` (progressive approximation, Section 3.2).
inline __host__ __device__ int used_bits(int B, int prefix) {
    return (prefix > 0 && prefix < B) ? prefix : B;
}

// (past 2^e, and NaN: any value in range; see Largest)
__device__ __forceinline__ int fixed_point(float v, int e) {
    constexpr float most = float(1 << QEXP);
    return int(fminf(fmaxf(rintf(ldexpf(v, QEXP - e)), -most), most));
}

// A pass: up to 8 bit planes of up to FOLD_STEPS steps of one segment.
// Consecutive passes whose bytes lie close together in a record form a group,
// whose codes are fetched at once.
struct Pass {
    int off;     // byte offset of its first plane's first step in a record
    int pb;      // bytes per plane
    int b;       // planes
    int steps;   // steps
    int q0;      // query step of its first step
    int s;       // kept segment
    int wexp;    // the pass's sums times 2^wexp are sums of c - h in units of the B-bit code
    int info;    // bit 0: add half the segment's query sum (8 planes, last run of the segment);
                 // where a group starts, bits 8..15: its 32-byte loads per record, bits 16..31:
                 // its passes
};
constexpr int ARG_PASSES = 96;
struct PassArg { Pass p[ARG_PASSES]; };

// The exponent e of a query whose largest weighted component is v.  A pass's
// sums, below 2^46 in units of 2^(e - 30), stay in FP32's range for every e (a
// query with components past 2^111 has an infinite norm, and so the estimate).
__device__ __forceinline__ int query_exponent(float v) {
    if (!(v > 0x1p-97f)) return -96;
    if (v >= 0x1p111f) return 111;
    int k = 0;
    (void)frexpf(v, &k);
    return k;
}

// The largest weighted component of a row, and whether all are finite, over
// `lanes` lanes that start at j0 = 0 .. lanes - 1 (a power of two of a wave's; all
// of them get it).  Fixed point has no infinities: a query with a component
// that is not finite has NaN estimates, as FP32 sums over it would.
struct Largest { float v; bool finite; };
__device__ __forceinline__ Largest largest(const float* __restrict__ row, const float* __restrict__ weight, int dk,
                                           int j0, int lanes) {
    float v = 0.f;
    uint32_t bits = 0;          // of the largest |component|; infinity and NaN are past all finite ones
    auto take = [&](float x, float w) {
        v = fmaxf(v, fabsf(x * w));
        bits = max(bits, __float_as_uint(x) & 0x7fffffffu);
    };
    // clamped addresses instead of a branch per load, which would wait for each
    if ((dk & 3) == 0) {        // rows and weights start at 16-byte addresses
#pragma unroll 4
        for (int i = 0; i < dk; i += 4 * lanes) {
            const int j = min(i + 4 * j0, dk - 4);
            const float4 x = *reinterpret_cast<const float4*>(row + j), w = *reinterpret_cast<const float4*>(weight + j);
            take(x.x, w.x); take(x.y, w.y); take(x.z, w.z); take(x.w, w.w);
        }
    } else {
#pragma unroll 8
        for (int i = 0; i < dk; i += lanes) take(row[min(i + j0, dk - 1)], weight[min(i + j0, dk - 1)]);
    }
    for (int d = 1; d < lanes; d <<= 1) {
        v = fmaxf(v, __shfl_xor(v, d));
        bits = max(bits, uint32_t(__shfl_xor(int(bits), d)));
    }
    return Largest{v, bits < 0x7f800000u};
}

// Further passes of a scan with more than ARG_PASSES.
__global__ __launch_bounds__(64) void write_passes_kernel(const PassArg arg, int count,
                                                          Pass* __restrict__ passes) {
    for (int i = threadIdx.x; i < count; i += 64) passes[i] = arg.p[i];
}

// The queries' digits in the order the scan's matrix operands take them:
// 16-byte groups [query tile][step][digit][half m][lane half lh][query], the
// group holding, for kk = 0..15, dim 32 lh + 8 (kk % 4) + 4 m + kk / 4 of the
// step's 64 (the order in which the scan's bit transposition leaves the codes
// of a plane word); with `few` (scan_few_kernel) [step][digit][quarter 2 m +
// lh][query], dim 16 (2 m + lh) + 8 (kk % 2) + kk / 2.  Dims past the segment
// are zero, so whatever the record side holds there adds nothing.  One
// workgroup per step and DQ queries, which first takes their exponents, then
// one thread per query, m, lh and group of 4 kk.
//
// EXTRA more workgroups per query tile, a wave per query, write the queries'
// exponents qexp and, per segment that has passes of 8 planes, half the sum of
// their fixed-point values (qh [n_kept][padded nq]), copy the last record
// tiles' codes (last_bytes) to `tail`, which has room behind them, and write
// the scan's first passes.
constexpr int EXTRA = TQ / 4;
constexpr int DQ = 16;
__global__ __launch_bounds__(256) void query_digits_kernel(const float* __restrict__ Qp, int nq, int dk,
                                                           const SegEntry* __restrict__ segs, int n_kept,
                                                           const float* __restrict__ weight, int prefix,
                                                           int tq, int few, int steps,
                                                           uint32_t* __restrict__ Qd, int* __restrict__ qexp,
                                                           float* __restrict__ qh, float* __restrict__ qn2,
                                                           const uint8_t* __restrict__ last,
                                                           int last_bytes, uint8_t* __restrict__ tail,
                                                           const PassArg arg, int count,
                                                           Pass* __restrict__ passes) {
    const int parts = tq / DQ, step = blockIdx.x / parts, q0 = blockIdx.y * tq;
    if (step >= steps) {
        const int extra = blockIdx.x - steps * parts, b = extra * gridDim.y + blockIdx.y;
        for (int i = b * 256 + threadIdx.x; i < last_bytes; i += EXTRA * gridDim.y * 256) tail[i] = last[i];
        if (b == 0)
            for (int i = threadIdx.x; i < count; i += 256) passes[i] = arg.p[i];
        const int r = extra * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, q = q0 + r;
        if (r >= tq || q >= nq) return;
        const float* row = Qp + int64_t(q) * dk;
        const Largest most = largest(row, weight, dk, lane, 64);
        const int e = query_exponent(most.v);
        if (lane == 0) {
            qexp[q] = e;
            if (!most.finite) qn2[q] = __builtin_nanf("");
        }
        for (int s = 0; s < n_kept; ++s) {
            const SegEntry g = segs[s];
            if (used_bits(g.bits, prefix) < 8) continue;
            int64_t sum = 0;
            for (int j = lane; j < g.width; j += 64) sum += fixed_point(row[g.col + j] * weight[g.col + j], e);
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
            if (lane == 0) qh[s * padded_queries(nq) + q] = 0.5f * float(sum);
        }
        return;
    }
    const int rows = min(tq, nq - q0);          // queries of this tile
    const int first = blockIdx.x % parts * DQ;  // of this workgroup
    if (first >= rows) return;
    __shared__ int exps[DQ];
    int s = 0, st = step;
    while (st >= seg_steps(segs[s].width)) st -= seg_steps(segs[s++].width);
    const SegEntry g = segs[s];
    const int v = threadIdx.x & 3, lh = (threadIdx.x >> 2) & 1, m = (threadIdx.x >> 3) & 1, q = threadIdx.x >> 4;
    const float* row = Qp + int64_t(q0 + min(first + q, rows - 1)) * dk + g.col;
    const float scale = weight[g.col];          // one weight per segment
    float x4[4];                                // loaded beside the exponents' components
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int j = SD * st + (few ? 16 * (2 * m + lh) + 8 * (k & 1) + 2 * v + (k >> 1)
                                     : 32 * lh + 8 * k + 4 * m + v);
        x4[k] = j < g.width ? row[j] * scale : 0.f;
    }
    {
        // 16 lanes per query; all 64 of a wave where there are at most 4
        const int lanes = rows <= 4 ? 64 : 16, i = threadIdx.x / lanes;
        const Largest most = largest(Qp + int64_t(q0 + min(first + i, rows - 1)) * dk, weight, dk,
                                     threadIdx.x % lanes, lanes);
        if (threadIdx.x % lanes == 0) exps[i] = query_exponent(most.v);
    }
    __syncthreads();
    if (first + q >= rows) return;
    const int e = exps[q];
    uint32_t w[ND] = {};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        int x = fixed_point(x4[k], e);
        // balanced digits, least significant first
#pragma unroll
        for (int d = ND - 1; d >= 0; --d) {
            const int b = int(int8_t(x));
            w[d] |= uint32_t(b & 0xff) << (8 * k);
            x = (x - b) >> 8;
        }
    }
    uint32_t* dst = Qd + 4 * ((int64_t(blockIdx.y) * steps * tq + int64_t(step) * rows) * 4 * ND +
                              (m * 2 + lh) * rows + first + q) + v;
#pragma unroll
    for (int d = 0; d < ND; ++d) dst[d * 16 * rows] = w[d];
}

// Transposes, in each of the four byte lanes, the 8 x 8 bits of w[0..7]: bit
// b of byte k of w[i] becomes bit i of byte k of w[b].  Three rounds of
// masked swaps, each a shift and a bit-field insert per word (the recursive
// block swaps of Warren, Hacker's Delight, section 7-3).
__device__ __forceinline__ void transpose_bits(uint32_t (&w)[8]) {
    auto swap = [&](int a, int b, int s, uint32_t m) {
        const uint32_t x = w[a], y = w[b];
        w[a] = (x & m) | ((y << s) & ~m);
        w[b] = ((x >> s) & m) | (y & ~m);
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) swap(i, i + 4, 4, 0x0f0f0f0fu);
#pragma unroll
    for (int i = 0; i < 8; i += 4) {
        swap(i, i + 2, 2, 0x33333333u);
        swap(i + 1, i + 3, 2, 0x33333333u);
    }
#pragma unroll
    for (int i = 0; i < 8; i += 2) swap(i, i + 1, 1, 0x55555555u);
}

// An LDS offset the compiler computes where it is used: left to itself it
// carries one address per plane and case of the decoding through the loops,
// and spills.
__device__ __forceinline__ int here(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// The bytes of a lane's 32 codes of one step from b plane words, plane p at
// src + p pb (any alignment): byte k of w[i] is the code of dim 8k + i, plane
// p its bit 7 - p (the first one inverted), then a one, then zeros.
template <int B>
__device__ __forceinline__ void decode(const unsigned char* src, int pb, uint32_t (&w)[8]) {
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        w[7 - p] = p == B ? 0xffffffffu : 0u;
        if (p < B) __builtin_memcpy(&w[7 - p], src + p * pb, 4);
    }
    w[7] = ~w[7];
    transpose_bits(w);
}

// The same for 16 dims of two records: the low halves of w are the record at
// sa, the high halves the one at sb.
template <int B>
__device__ __forceinline__ void decode_pair(const unsigned char* sa, const unsigned char* sb, int pb,
                                            uint32_t (&w)[8]) {
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        w[7 - p] = p == B ? 0xffffffffu : 0u;
        if (p < B) {
            uint16_t x, y;
            __builtin_memcpy(&x, sa + p * pb, 2);
            __builtin_memcpy(&y, sb + p * pb, 2);
            w[7 - p] = x | uint32_t(y) << 16;
        }
    }
    w[7] = ~w[7];
    transpose_bits(w);
}

// The codes of a wave's 32 records, one group of passes at a time.  A group is
// a run of bytes of a record; the wave copies it to its own part of LDS as
// 16-byte units, two lanes per record, so each line of the records is read in
// wide pieces.  (Each lane fetching its own planes' pieces took 172 cache
// accesses per load instruction and held the texture addresser busy 82 % of
// the time.)  With a 16-byte aligned code buffer the units are the aligned ones
// around the group's bytes, otherwise they start at its first byte.  They may
// reach a few bytes past the record, so the last record tiles are read from a
// padded copy.
//
// NL: 32-byte loads per record and group; a group that needs fewer points the
// rest at one address.  The loads are unconditional, so that the compiler can
// count them: behind a branch it waits for them at once.
template <int NL>
struct CodeStage {
    // LDS bytes per record: the units, and 16 more so that the rows of a wave
    // spread over the banks
    static constexpr int ROW = 32 * NL + 16;
    struct Regs { u32x4 v[NL]; };
    const uint8_t* base;    // the code buffer, or what stands for it
    const uint8_t* idle;    // an address that can always be read
    int64_t at;             // byte offset of the record this lane loads
    int mask;               // 15: aligned units
    int odd;                // 16 in odd lanes
    unsigned char* dst;     // LDS of its unit

    __device__ __forceinline__ CodeStage(unsigned char* lds, const uint8_t* codes, const uint8_t* tail,
                                         int tail_tile, int rtile, int64_t code_bytes, int64_t n,
                                         int wave, int lane, int align_mask) {
        base = rtile < tail_tile ? codes : tail - int64_t(tail_tile) * TR * code_bytes;
        idle = base + int64_t(rtile) * TR * code_bytes;
        at = min(int64_t(rtile) * TR + wave * WR + (lane >> 1), n - 1) * code_bytes;
        mask = align_mask;
        odd = (lane & 1) * 16;
        dst = lds + (lane >> 1) * ROW + odd;
    }
    __device__ __forceinline__ Regs load(const Pass& P) const {
        const int64_t a = at + P.off;
        const uint8_t* src = base + (a - (int(a) & mask) + odd);
        const int loads = (P.info >> 8) & 0xff;
        Regs c;
#pragma unroll
        for (int k = 0; k < NL; ++k) __builtin_memcpy(&c.v[k], k < loads ? src + 32 * k : idle, 16);
        return c;
    }
    // LDS operations of a wave execute in order, so a group's codes may be
    // written once the wave has read the last plane words of the group before;
    // the fences keep the compiler to that order
    __device__ __forceinline__ void store(const Regs& c) const {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int k = 0; k < NL; ++k) *reinterpret_cast<u32x4*>(dst + 32 * k) = c.v[k];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    // where the group whose first byte is `off` starts in the row of the record
    // at byte offset r
    __device__ __forceinline__ int first(int r, int off) const { return (r + off) & mask; }
};

// The factors of a wave's 32 records: in LDS while a record has at most
// FACTORS of them (read once, wide, and out of the way of the counted loads),
// else where they are.
constexpr int FACTORS = 17;
struct FactorStage {
    float* lds;
    const float* own;       // first wave record's factors
    int nf;
    int64_t last;           // records from the first one of the wave to the last one there is

    __device__ __forceinline__ FactorStage(float* lds_, const float* factors, int n_kept, int64_t first,
                                           int64_t n, int lane) {
        lds = lds_;
        nf = n_kept + 1;
        first = min(first, n - 1);
        last = n - 1 - first;
        own = factors + first * nf;
        if (nf <= FACTORS) {
            const int have = int(min(last + 1, int64_t(WR))) * nf;
            for (int i = lane; i < WR * nf; i += 64) lds[i] = own[min(i, have - 1)];
        }
    }
    // factor s of record r of the wave (r past the last record: any value)
    __device__ __forceinline__ float get(int r, int s) const {
        return nf <= FACTORS ? lds[r * nf + s] : own[min(int64_t(r), last) * nf + s];
    }
};

// The four digit sums of a pair joined, 2^24 s0 + 2^16 s1 + 2^8 s2 + s3: the
// pairs in integers, then in FP32.
__device__ __forceinline__ float join_digits(int s0, int s1, int s2, int s3) {
    return fmaf(float(s0 * 256 + s1), 65536.f, float(s2 * 256 + s3));
}

// The scan.  A workgroup takes 128 records x 32 QB queries, a wave 32 records
// x all queries of the tile.  The query digits are the A operand, the wave's
// own records the B operand, so a lane's 16 sums per query block belong to
// one record, the one whose plane words it transposes, and f_s is the lane's
// own scalar.  Lane half lh takes the plane words of its 32 dims of a 64-dim
// step; the 8 x 8 bit transposition turns the (up to 8) words into the bytes
// of 32 codes, 1.5 VALU operations per code; no conversion follows.  The four
// waves share one step's digits through LDS, double buffered; the digits of the
// step after next are fetched while the next step runs, and a group's codes
// after them, so that waiting for the digits leaves the codes in flight.
//
// Whole calls: 64 queries, 1M records of 768 dims at 4 b/dim 721 us on split bf16
// operands, 513 so; 100 queries, 250,007 records of 3,072 dims at 2 bits 1,121 and
// 514.  In the first the VALU is busy 42 % of the time (half of it where passes
// end), the LDS 33 %, the matrix cores 17 % (27, 46 and 30 % in the second); two
// waves per SIMD do not cover each other's waits.  32-query tiles, with three,
// decode twice: 700 us.
template <int QB, int NL>
__global__ __launch_bounds__(256, 2) void scan_kernel(
    const u32x4* __restrict__ Qd, int nq, const float* __restrict__ qn2, const int* __restrict__ qexp,
    const float* __restrict__ qh, const Pass* __restrict__ passes, int count, int n_kept,
    int steps, const uint8_t* __restrict__ codes, int64_t code_bytes, int align_mask,
    const uint8_t* __restrict__ tail, int tail_tile, const float* __restrict__ factors, int64_t n,
    int rtiles, int qtiles, float* __restrict__ out) {
    constexpr int NQ = 32 * QB;                 // queries of the tile's MFMA blocks
    constexpr int GROUPS = 4 * ND;              // 16-byte groups per query and step
    constexpr int UNITS = GROUPS * NQ / 256;    // groups staged per thread and step
    using Stage = CodeStage<NL>;
    __shared__ __attribute__((aligned(16))) unsigned char clds[WAVES][WR * Stage::ROW];
    __shared__ __attribute__((aligned(16))) u32x4 qlds[2][GROUPS * NQ];
    __shared__ float flds[WAVES][WR * FACTORS];

    // query tiles of one record tile follow each other on one XCD, so the
    // record tile's codes come from its L2 after the first
    const int bid = blockIdx.x, local = bid / NXCD;
    const int rtile = (local / qtiles) * NXCD + bid % NXCD;
    const int qtile = local % qtiles;
    if (rtile >= rtiles) return;
    const int t = threadIdx.x, lane = t & 63, li = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int q0 = qtile * NQ, rows = min(NQ, nq - q0), nqp = padded_queries(nq);
    const u32x4* Qt = Qd + int64_t(qtile) * steps * NQ * GROUPS;
    // records past n read record n - 1 and are never stored
    const int64_t wrec = int64_t(rtile) * TR + wave * WR;       // the wave's first record
    const int low = int(min(wrec + li, n - 1) * code_bytes) & 15;
    const FactorStage fs(flds[wave], factors, n_kept, wrec, n, lane);
    const Stage stage(clds[wave], codes, tail, tail_tile, rtile, code_bytes, n, wave, lane, align_mask);
    const int cl = li * Stage::ROW + 4 * lh;

    // query groups of one step: thread t stages groups i 256 + t (threads of
    // queries past nq stage copies of the last one)
    u32x4 qreg[UNITS];
    const int qg = t / NQ, qq = min(t % NQ, rows - 1);
    auto load_queries = [&](int step) {
        const u32x4* src = Qt + step * rows * GROUPS + (qg * rows + qq);
#pragma unroll
        for (int i = 0; i < UNITS; ++i) qreg[i] = src[i * (256 / NQ) * rows];
    };
    auto store_queries = [&](int buf) {
#pragma unroll
        for (int i = 0; i < UNITS; ++i) qlds[buf][i * 256 + t] = qreg[i];
    };

    float tot[QB][16];
#pragma unroll
    for (int b = 0; b < QB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) tot[b][r] = 0.f;

    if (n_kept > 0) {
        // the queries' steps, two ahead of the products
        int qi = 0, qs = 0;
        Pass Q = passes[0];
        auto next_queries = [&]() {
            load_queries(Q.q0 + qs);
            if (++qs == Q.steps) {          // behind the last pass: the first again, unused
                qi = qi + 1 < count ? qi + 1 : 0;
                Q = passes[qi];
                qs = 0;
            }
        };
        Pass P = passes[0];
        next_queries();
        auto c = stage.load(P);
        store_queries(0);
        stage.store(c);
        next_queries();
        __syncthreads();
        int buf = 0, ip = 0;
        while (ip < count) {
            const int next = ip + (P.info >> 16), goff = P.off;
            const int row0 = cl + stage.first(low, goff);
            // the next group's codes (behind the last group the last pass's, unused)
            c = stage.load(passes[min(next, count - 1)]);
            for (; ip < next; ++ip) {
                const Pass N = passes[min(ip + 1, count - 1)];
                const float f = fs.get(li, P.s);
                const int first = row0 + (P.off - goff);
                i32x16 acc[ND][QB];
                auto step = [&](int st, auto zero) {
                    uint32_t w[8];
                    const int cw = here(first + 8 * st);
                    switch (P.b) {
#define SAQ_DECODE(K) case K: decode<K>(clds[wave] + cw, P.pb, w); break;
                        SAQ_DECODE(1) SAQ_DECODE(2) SAQ_DECODE(3) SAQ_DECODE(4)
                        SAQ_DECODE(5) SAQ_DECODE(6) SAQ_DECODE(7)
                        default: decode<8>(clds[wave] + cw, P.pb, w); break;
#undef SAQ_DECODE
                    }
                    // product u: digit u % 4 with half u / 4 of the codes; its
                    // query operand is read one product ahead
                    const u32x4* A = qlds[buf] + lh * NQ + li;
                    auto operand = [&](int u, int b) {
                        return __builtin_bit_cast(i32x4, A[((u & 3) * 4 + (u >> 2) * 2) * NQ + 32 * b]);
                    };
                    i32x4 a[2][QB];
#pragma unroll
                    for (int b = 0; b < QB; ++b) a[0][b] = operand(0, b);
#pragma unroll
                    for (int u = 0; u < 2 * ND; ++u) {
                        const int m = u >> 2, d = u & 3;
                        const i32x4 B = {int(w[4 * m]), int(w[4 * m + 1]), int(w[4 * m + 2]), int(w[4 * m + 3])};
#pragma unroll
                        for (int b = 0; b < QB; ++b)
                            if (u + 1 < 2 * ND) a[(u + 1) & 1][b] = operand(u + 1, b);
#pragma unroll
                        for (int b = 0; b < QB; ++b) {
                            if (decltype(zero)::value && m == 0)
                                acc[d][b] = i32x16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
                            acc[d][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[u & 1][b], B, acc[d][b], 0, 0, 0);
                        }
                    }
                    store_queries(buf ^ 1);
                    __syncthreads();
                    buf ^= 1;
                    next_queries();
                };
                step(0, std::true_type{});
#pragma unroll 1
                for (int st = 1; st < P.steps; ++st) step(st, std::false_type{});
                // the sums, exact so far, into the FP32 totals
                const float g = ldexpf(f, P.wexp);
                auto fold = [&](auto half) {
#pragma unroll
                    for (int b = 0; b < QB; ++b)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            float T = join_digits(acc[0][b][r], acc[1][b][r], acc[2][b][r], acc[3][b][r]);
                            if (decltype(half)::value) {
                                // rows past nq: never stored
                                T += qh[P.s * nqp + q0 + 32 * b + 8 * (r >> 2) + 4 * lh + (r & 3)];
                            }
                            tot[b][r] = fmaf(g, T, tot[b][r]);
                        }
                };
                if (P.info & 1) fold(std::true_type{});
                else fold(std::false_type{});
                P = N;
            }
            stage.store(c);
        }
    }

    // lane: record rec; register r of block b is query q0 + 32 b + 8 (r/4) +
    // 4 lh + r%4: each store writes 32 consecutive records per lane half
    const float o2 = fs.get(li, n_kept);
    float qn[QB][16];
    int qe[QB][16];
#pragma unroll
    for (int b = 0; b < QB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int q = q0 + 32 * b + 8 * (r >> 2) + 4 * lh + (r & 3);   // padded to a whole tile
            qn[b][r] = qn2[q];
            qe[b][r] = qexp[q];
        }
    const int64_t rec = wrec + li;
    if (rec < n) {
        float* orow = out + (q0 + 4 * lh) * n + rec;
#pragma unroll
        for (int b = 0; b < QB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int q = 32 * b + 8 * (r >> 2) + (r & 3);
                if (q + 4 * lh < rows)
                    orow[q * n] = (o2 + qn[b][r]) - ldexpf(tot[b][r], qe[b][r] - (QEXP - 1));
            }
    }
}

// The scan of at most 16 queries whose digits all fit in RES_BYTES of LDS: no
// barrier after the first, and 16 x 16 x 64 products, which leave a lane 4
// sums per record block instead of 16 (a quarter of the registers and of the
// work where a pass ends), so that three workgroups per CU keep the record stream
// in flight (four with FOUR and 4 loads, two with 8 loads and the queries' 20 KB
// of LDS full).  Lane: records lane % 16 and 16 + lane % 16 of the wave, dims
// 16 (lane / 16) .. + 15 of a step; the two records' 16-bit pieces of a plane
// share a word, are transposed together and parted again.  FOUR: at most four
// queries, each the operand's rows 4 q .. 4 q + 3, so that the first of a lane's
// four sums is query lane / 16's and the others need no work.
//
// One query, 1M records of 1,536 dims at 4 b/dim (820 MB), whole calls: 1,053 us on
// split bf16 operands, 278 so (300 with four sums per lane, whose VALU work is 28 %
// more); the kernel 267.  The VALU is busy 54 % of that time, the LDS 53 %, the
// texture addresser 46 %; the rest is the chain of a step: LDS reads,
// transposition, products.
template <int NL, bool FOUR>
__global__ __launch_bounds__(256, 3) void scan_few_kernel(
    const u32x4* __restrict__ Qd, int nq, const float* __restrict__ qn2, const int* __restrict__ qexp,
    const float* __restrict__ qh, const Pass* __restrict__ passes, int count, int n_kept,
    int steps, const uint8_t* __restrict__ codes, int64_t code_bytes, int align_mask,
    const uint8_t* __restrict__ tail, int tail_tile, const float* __restrict__ factors, int64_t n,
    int rtiles, float* __restrict__ out) {
    using Stage = CodeStage<NL>;
    __shared__ __attribute__((aligned(16))) unsigned char clds[WAVES][WR * Stage::ROW];
    __shared__ float flds[WAVES][WR * FACTORS];
    extern __shared__ __attribute__((aligned(16))) u32x4 qres[];   // [step][digit][quarter][query]
    const int rtile = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63, ri = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t rec0 = int64_t(rtile) * TR + wave * WR + ri;      // and rec0 + 16
    constexpr int R = FOUR ? 1 : 4;                                 // sums used per record
    auto query = [&](int r) { return FOUR ? kg : 4 * kg + r; };
    // rec0 + 16's bytes start at the same place of a 16-byte unit (past the last
    // record: somewhere in its row, never stored)
    const int low = int(min(rec0, n - 1) * code_bytes) & 15;
    const FactorStage fs(flds[wave], factors, n_kept, int64_t(rtile) * TR + wave * WR, n, lane);
    const Stage stage(clds[wave], codes, tail, tail_tile, rtile, code_bytes, n, wave, lane, align_mask);
    const int cl = ri * Stage::ROW + 2 * kg;

    float tot[2][R];
#pragma unroll
    for (int r = 0; r < R; ++r) tot[0][r] = tot[1][r] = 0.f;
    if (n_kept > 0) {
        Pass P = passes[0];
        auto c = stage.load(P);
        for (int u = t; u < steps * 4 * ND * nq; u += 256) qres[u] = Qd[u];
        stage.store(c);
        __syncthreads();
        const u32x4* Abase = qres + kg * nq + min(FOUR ? ri >> 2 : ri, nq - 1);
        int ip = 0;
        while (ip < count) {
            const int next = ip + (P.info >> 16), goff = P.off;
            const int row0 = cl + stage.first(low, goff);
            // the next group's codes (behind the last group the last pass's, unused)
            c = stage.load(passes[min(next, count - 1)]);
            for (; ip < next; ++ip) {
                const Pass N = passes[min(ip + 1, count - 1)];
                const int first = row0 + (P.off - goff);
                i32x4 acc[ND][2];
                auto step = [&](int st, auto zero) {
                    const u32x4* A = Abase + (P.q0 + st) * 4 * ND * nq;
                    i32x4 a[ND];
#pragma unroll
                    for (int d = 0; d < ND; ++d) a[d] = __builtin_bit_cast(i32x4, A[d * 4 * nq]);
                    uint32_t w[8];
                    const unsigned char* src = clds[wave] + here(first + 8 * st);
                    switch (P.b) {
#define SAQ_DECODE(K) case K: decode_pair<K>(src, src + 16 * Stage::ROW, P.pb, w); break;
                        SAQ_DECODE(1) SAQ_DECODE(2) SAQ_DECODE(3) SAQ_DECODE(4)
                        SAQ_DECODE(5) SAQ_DECODE(6) SAQ_DECODE(7)
                        default: decode_pair<8>(src, src + 16 * Stage::ROW, P.pb, w); break;
#undef SAQ_DECODE
                    }
                    // bytes 0, 1 of w[i]: dims i, 8 + i of the first record, bytes
                    // 2, 3 of the second
                    i32x4 B0, B1;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        B0[v] = int(__builtin_amdgcn_perm(w[2 * v + 1], w[2 * v], 0x05040100u));
                        B1[v] = int(__builtin_amdgcn_perm(w[2 * v + 1], w[2 * v], 0x07060302u));
                    }
#pragma unroll
                    for (int d = 0; d < ND; ++d) {
                        if (decltype(zero)::value) acc[d][0] = acc[d][1] = i32x4{0, 0, 0, 0};
                        acc[d][0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[d], B0, acc[d][0], 0, 0, 0);
                        acc[d][1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[d], B1, acc[d][1], 0, 0, 0);
                    }
                };
                step(0, std::true_type{});
#pragma unroll 1
                for (int st = 1; st < P.steps; ++st) step(st, std::false_type{});
                const float ga = ldexpf(fs.get(ri, P.s), P.wexp), gb = ldexpf(fs.get(ri + 16, P.s), P.wexp);
                float h[R];
#pragma unroll
                for (int r = 0; r < R; ++r) h[r] = 0.f;
                if (P.info & 1) {
                    const float* src = qh + P.s * padded_queries(nq) + query(0);
#pragma unroll
                    for (int r = 0; r < R; ++r) h[r] = src[r];
                }
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    tot[0][r] = fmaf(ga, join_digits(acc[0][0][r], acc[1][0][r], acc[2][0][r], acc[3][0][r]) + h[r],
                                     tot[0][r]);
                    tot[1][r] = fmaf(gb, join_digits(acc[0][1][r], acc[1][1][r], acc[2][1][r], acc[3][1][r]) + h[r],
                                     tot[1][r]);
                }
                P = N;
            }
            stage.store(c);
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int q = query(r);
        if (q >= nq) break;
        const float qn = qn2[q];
        const int e = qexp[q] - (QEXP - 1);
        float* orow = out + q * n + rec0;
        if (rec0 < n) orow[0] = (fs.get(ri, n_kept) + qn) - ldexpf(tot[0][r], e);
        if (rec0 + 16 < n) orow[16] = (fs.get(ri + 16, n_kept) + qn) - ldexpf(tot[1][r], e);
    }
}

int total_steps(const saq_plan* p) {
    int s = 0;
    for (const SegEntry& e : p->kept) s += seg_steps(e.width);
    return s;
}

// How a segment read at B bits splits into passes: its planes in groups of at
// most 8, fewer where they would span more bytes than one fetch covers, as
// even as possible, and its steps in runs of FOLD_STEPS.
int plane_groups(int W, int B) {
    const int pb = (W + 7) >> 3, run = std::min(seg_steps(W), FOLD_STEPS);
    const int most = std::min(8, 1 + (SPAN - run * (SD / 8)) / pb);
    return (B + most - 1) / most;
}
int most_passes(const saq_plan* p) {
    int k = 0;
    for (const SegEntry& e : p->kept)
        k += plane_groups(e.width, e.bits) * ((seg_steps(e.width) + FOLD_STEPS - 1) / FOLD_STEPS);
    return k;
}

// The passes of a scan that reads `prefix` bits (0: all).
std::vector<Pass> scan_passes(const saq_plan* p, int prefix) {
    std::vector<Pass> out;
    int q0 = 0;
    for (size_t s = 0; s < p->kept.size(); ++s) {
        const SegEntry& g = p->kept[s];
        const int B = used_bits(g.bits, prefix), pb = (g.width + 7) >> 3, steps = seg_steps(g.width);
        const int parts = plane_groups(g.width, B);
        for (int k = 0, p0 = 0; k < parts; ++k) {
            const int b = B / parts + (k < B % parts ? 1 : 0);
            for (int st0 = 0; st0 < steps; st0 += FOLD_STEPS) {
                Pass P{};
                P.off = g.code_off + p0 * pb + st0 * (SD / 8);
                P.pb = pb;
                P.b = b;
                P.steps = std::min(FOLD_STEPS, steps - st0);
                P.q0 = q0 + st0;
                P.s = int(s);
                P.wexp = g.bits - p0 - b + (b < 8 ? b - 8 : 0) - p->shift[s];
                P.info = b == 8 && st0 + P.steps == steps;
                out.push_back(P);
            }
            p0 += b;
        }
        q0 += steps;
    }
    return out;
}

// 32-byte loads that cover bytes first .. first + len - 1 of a record wherever
// the first one falls in a 16-byte unit
int span_loads(int len) { return (15 + len + 31) / 32; }
int pass_end(const Pass& P) { return P.off + (P.b - 1) * P.pb + P.steps * (SD / 8); }

// Joins passes to groups of at most nl loads.
void group_passes(std::vector<Pass>& v, int nl) {
    for (size_t i = 0; i < v.size();) {
        int end = pass_end(v[i]);
        size_t j = i + 1;
        for (; j < v.size() && v[j].off >= v[i].off; ++j) {
            const int e = std::max(end, pass_end(v[j]));
            if (span_loads(e - v[i].off) > nl) break;
            end = e;
        }
        v[i].info |= span_loads(end - v[i].off) << 8 | int(j - i) << 16;
        i = j;
    }
}

// Scans of narrow segments that scan_few_kernel does not take run on split bf16
// operands instead (estimate_kernel), where f_s is part of the operand: in
// scan_kernel every pass costs a 64-dim step and 6 VALU operations per pair
// whatever its width.  Measured, us in scan_kernel / there: D = 128 (16-dim
// segments) 68 / 60 at 16 queries and 300,000 records, 319 / 213 at 64 and 1M;
// D = 200 84 / 71 at 9 to 16 queries and 300,000; D = 333 (mostly 32-dim segments)
// 87 / 73 at 9 to 16 and 200,000, 174 / 146 at 130 and 100,001.  The line: 64
// queries, 100,000 records, 32-dim segments 98 there, 118 at the commit before
// this kernel; 40-dim segments 84 and 48-dim 74 here, 162 and 113 at that commit.
// scan_few_kernel's passes cost a quarter: D = 128 and 12 queries 52 us, 62 there.
bool narrow_passes(const saq_plan* p, const std::vector<Pass>& v) {
    return int64_t(p->D_kept) < 40 * int64_t(v.size());
}

// Few queries, all digits resident in LDS (scan_few_kernel).
size_t digit_bytes(const saq_plan* p, int nq) { return size_t(nq) * total_steps(p) * SD * ND; }
bool few_queries(const saq_plan* p, int nq) { return nq <= 16 && digit_bytes(p, nq) <= RES_BYTES; }

int64_t align16(int64_t v) { return (v + 15) & ~int64_t(15); }

// workspace of a scan: Qp [nq x D_kept], ||q - c||^2 and the fixed-point
// exponents [nq padded to whole query tiles], half sums [n_kept x padded nq],
// the digits, the last record tiles' codes, the passes
struct ScanLayout {
    int64_t off_n2, off_exp, off_qh, off_qd, off_tail, off_pass, bytes;
    ScanLayout(const saq_plan* p, int32_t nq) {
        const int64_t q = std::max(nq, 1);
        off_n2 = align16(q * std::max(p->D_kept, 1) * 4);
        off_exp = off_n2 + int64_t(padded_queries(int(q))) * 4;
        off_qh = off_exp + int64_t(padded_queries(int(q))) * 4;
        off_qd = off_qh + align16(int64_t(padded_queries(int(q))) * std::max(p->n_kept, 1) * 4);
        off_tail = off_qd + q * total_steps(p) * SD * ND;
        off_pass = off_tail + align16(TR * p->code_bytes + OVER + OVER);
        bytes = off_pass + most_passes(p) * int64_t(sizeof(Pass)) + 256;
    }
};

saq_status scan_impl(const saq_plan* p, const float* Q, int32_t nq, const float* ref,
                     const uint8_t* codes, const float* factors, int64_t n, int32_t prefix_bits,
                     float* out, void* ws, int64_t ws_bytes, void* stream) try {
    if (saq_status st = saq::check_uploaded(p, "plan"); st != SAQ_OK) return st;
    if (nq < 0 || n < 0) return saq::fail(SAQ_EINVAL, "bad sizes");
    if (prefix_bits < 0) return saq::fail(SAQ_EINVAL, "prefix_bits < 0");
    if (nq == 0 || n == 0) return SAQ_OK;
    if (!Q || !codes || !factors || !out || !ws) return saq::fail(SAQ_EINVAL, "null buffer");
    if (ws_bytes < saq_estimate_workspace_bytes(p, nq)) return saq::fail(SAQ_EINVAL, "workspace too small");
    hipStream_t st = static_cast<hipStream_t>(stream);
    std::vector<Pass> pv = scan_passes(p, prefix_bits);
    // rows of M of different lengths: the operands that hold every component to 24 bits
    const bool few = few_queries(p, nq);
    if (!p->even_rows || (!few && narrow_passes(p, pv)))
        return saq::scan_split(p, Q, nq, ref, codes, factors, n, prefix_bits, out, ws, st);
    char* base = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255));
    const ScanLayout L(p, nq);
    float* Qp = reinterpret_cast<float*>(base);
    float* qn2 = reinterpret_cast<float*>(base + L.off_n2);
    int* qexp = reinterpret_cast<int*>(base + L.off_exp);
    float* qh = reinterpret_cast<float*>(base + L.off_qh);
    u32x4* Qd = reinterpret_cast<u32x4*>(base + L.off_qd);
    uint8_t* tail = reinterpret_cast<uint8_t*>(base + L.off_tail);
    Pass* passes = reinterpret_cast<Pass*>(base + L.off_pass);
    const SegEntry* segs = saq::device_segments(p);
    saq_status s = saq::project_queries(p, Q, nq, ref, Qp, qn2, st);
    if (s != SAQ_OK) return s;
    const int dk = p->D_kept, steps = total_steps(p);
    const int tq = nq <= TQ / 2 ? TQ / 2 : TQ;
    const int qtiles = (nq + tq - 1) / tq;
    const size_t resident = digit_bytes(p, nq);
    // loads per group: what the longest pass needs, and where that is little
    // enough to cover several passes, so that a group's codes are in flight
    // for more than a step or two
    int nl = MIN_LOADS;
    for (const Pass& P : pv) nl = std::max(nl, span_loads(pass_end(P) - P.off));
    if (nl > MIN_LOADS) nl = MAXNL;
    group_passes(pv, nl);
    const int64_t rtiles = (n + TR - 1) / TR;
    // the copied tiles: the last one, two when it holds less than a pass's
    // units can reach past a record
    int64_t tail_tile = rtiles - 1;
    if (tail_tile > 0 && (n - tail_tile * TR) * p->code_bytes < OVER) --tail_tile;
    const uint8_t* last = codes + tail_tile * TR * p->code_bytes;
    const int last_bytes = int((n - tail_tile * TR) * p->code_bytes);
    const int align_mask = (reinterpret_cast<uintptr_t>(codes) & 15) == 0 ? 15 : 0;
    for (size_t i = 0; i < pv.size() || i == 0; i += ARG_PASSES) {
        PassArg arg;
        const int k = int(std::min<size_t>(ARG_PASSES, pv.size() - i));
        std::copy(pv.begin() + i, pv.begin() + i + k, arg.p);
        if (i == 0)
            hipLaunchKernelGGL(query_digits_kernel, dim3(unsigned(steps * (tq / DQ) + EXTRA), unsigned(qtiles)),
                               dim3(256), 0, st, Qp, nq, dk, segs, p->n_kept, saq::device_weights(p),
                               int(prefix_bits), tq, few ? 1 : 0, steps, reinterpret_cast<uint32_t*>(Qd), qexp,
                               qh, qn2, last, last_bytes, tail, arg, k, passes);
        else
            hipLaunchKernelGGL(write_passes_kernel, dim3(1), dim3(64), 0, st, arg, k, passes + i);
    }
    const dim3 grid(unsigned((rtiles + NXCD - 1) / NXCD * NXCD * qtiles));
#define SAQ_LAUNCH_SCAN(QB, NL)                                                                      \
    hipLaunchKernelGGL((scan_kernel<QB, NL>), grid, dim3(256), 0, st, Qd, nq, qn2, qexp, qh, passes, \
                       int(pv.size()), p->n_kept, steps, codes, p->code_bytes, align_mask, tail,              \
                       int(tail_tile), factors, n, int(rtiles), qtiles, out)
#define SAQ_LAUNCH_FEW(NL, FOUR)                                                                     \
    hipLaunchKernelGGL((scan_few_kernel<NL, FOUR>), dim3(unsigned(rtiles)), dim3(256), resident, st, Qd,   \
                       nq, qn2, qexp, qh, passes, int(pv.size()), p->n_kept, steps, codes, p->code_bytes,     \
                       align_mask, tail, int(tail_tile), factors, n, int(rtiles), out)
#define SAQ_BY_LOADS(LAUNCH)                                                                         \
    do {                                                                                             \
        if (nl == MIN_LOADS) LAUNCH(MIN_LOADS);                                                      \
        else LAUNCH(MAXNL);                                                                          \
    } while (0)
#define SAQ_LAUNCH_FEW4(NL) SAQ_LAUNCH_FEW(NL, true)
#define SAQ_LAUNCH_FEW16(NL) SAQ_LAUNCH_FEW(NL, false)
#define SAQ_LAUNCH_SCAN1(NL) SAQ_LAUNCH_SCAN(1, NL)
#define SAQ_LAUNCH_SCAN2(NL) SAQ_LAUNCH_SCAN(2, NL)
    if (few && nq <= 4) SAQ_BY_LOADS(SAQ_LAUNCH_FEW4);
    else if (few) SAQ_BY_LOADS(SAQ_LAUNCH_FEW16);
    else if (tq == TQ / 2) SAQ_BY_LOADS(SAQ_LAUNCH_SCAN1);
    else SAQ_BY_LOADS(SAQ_LAUNCH_SCAN2);
#undef SAQ_LAUNCH_SCAN
#undef SAQ_LAUNCH_SCAN1
#undef SAQ_LAUNCH_SCAN2
#undef SAQ_LAUNCH_FEW
#undef SAQ_LAUNCH_FEW4
#undef SAQ_LAUNCH_FEW16
#undef SAQ_BY_LOADS
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? SAQ_OK : saq::hip_status(e, "scan_kernel launch");
} catch (const std::bad_alloc&) {
    return saq::fail(SAQ_ENOMEM, "out of host memory");
}

}  // namespace

namespace saq {
int64_t scan_workspace_bytes(const saq_plan* p, int32_t nq) { return ScanLayout(p, nq).bytes; }
}  // namespace saq

extern "C" {

saq_status saq_estimate_dist_prefix(const saq_plan* p, const float* Q_dev, int32_t nq,
                                    const uint8_t* codes_dev, const float* factors_dev, int64_t n,
                                    int32_t prefix_bits, float* dist2_dev, void* ws_dev,
                                    int64_t ws_bytes, void* stream) {
    return scan_impl(p, Q_dev, nq, nullptr, codes_dev, factors_dev, n, prefix_bits, dist2_dev, ws_dev,
                     ws_bytes, stream);
}

saq_status saq_estimate_dist(const saq_plan* p, const float* Q_dev, int32_t nq,
                             const uint8_t* codes_dev, const float* factors_dev, int64_t n,
                             float* dist2_dev, void* ws_dev, int64_t ws_bytes, void* stream) {
    return scan_impl(p, Q_dev, nq, nullptr, codes_dev, factors_dev, n, 0, dist2_dev, ws_dev, ws_bytes,
                     stream);
}

saq_status saq_estimate_dist_ref(const saq_plan* p, const float* Q_dev, int32_t nq,
                                 const float* ref_dev, const uint8_t* codes_dev,
                                 const float* factors_dev, int64_t n, float* dist2_dev, void* ws_dev,
                                 int64_t ws_bytes, void* stream) {
    if (!ref_dev && nq > 0 && n > 0) return saq::fail(SAQ_EINVAL, "null reference");
    return scan_impl(p, Q_dev, nq, ref_dev, codes_dev, factors_dev, n, 0, dist2_dev, ws_dev, ws_bytes,
                     stream);
}

}  // extern "C"
