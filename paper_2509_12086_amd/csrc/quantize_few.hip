// Quantize, adjust and pack for few vectors (gfx950): one wave per vector and
// kept segment, one dim per lane.
//
// quantize_kernel (device.hip) gives every lane a vector and walks its dims in
// a chain; that fills the chip only with tens of thousands of vectors, and one
// vector takes as long as 64.  Here the 64 lanes hold 64 dims of one vector.
// Algorithm 1 is sequential over the dims, but few dims move (2.9, 1.8, 0.9
// and 0.5 % of them in rounds 1 to 4 on the 1M x 960 workload): all lanes
// evaluate their moves with the current state, the first lane that accepts one
// commits it, and the lanes behind it evaluate again.  The lanes before it saw
// the state that the sequential order gives them, so the moves, and every
// FP64 operation behind them, are quantize_kernel's own: same codes, factors
// and bytes.  The sums that start the state, ip = sum u o and sum o o, depend
// on their order; one lane per vector takes them in the order of the dims,
// from LDS, while nn = sum u u is exact in any order.
//
// Bound: latency.  A chunk of 64 dims takes 1 + (accepted moves) passes per
// round, about 8 in 4 rounds, where the chain of quantize_kernel takes 64 dims
// x 4 rounds.  One vector of 768 dims at 4 b/dim: 160 us before, 7 now; 517 at
// 6 b/dim: 340 before, 20 now.  The instructions per vector and dim are 2.5
// times the chain's, so with many vectors quantize_kernel is the faster one
// (few_vectors below).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "launch.hpp"

using saq::QuantItem;
using saq::SegEntry;

namespace {

constexpr int VECTORS = 8;              // vectors (waves) per workgroup
constexpr int CHUNKS = 8;               // 64-dim chunks a wave can hold
constexpr int MAXW = 64 * CHUNKS;       // widest segment

struct QuantFewArgs {
    QuantItem item[SAQ_BATCH_MAX];
    int64_t first_block[SAQ_BATCH_MAX];
    int count, rounds, lds_w;
};

__device__ __forceinline__ double lane_value(double x, int lane) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(x), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(x), lane);
    return __hiloint2double(hi, lo);
}

__global__ __launch_bounds__(64 * VECTORS) void quantize_few_kernel(const QuantFewArgs args) {
    extern __shared__ __attribute__((aligned(16))) float smem[];   // [vector][o | u][lds_w]
    __shared__ double sums[2 * VECTORS];                           // ip, oo
    int d = 0;
    while (d + 1 < args.count && int64_t(blockIdx.x) >= args.first_block[d + 1]) ++d;
    const QuantItem& I = args.item[d];
    const int64_t b = int64_t(blockIdx.x) - args.first_block[d];
    const int s = int(b % I.n_kept);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t v = (b / I.n_kept) * VECTORS + wave;
    const bool live = v < I.n;
    const int64_t vv = live ? v : I.n - 1;
    const SegEntry e = I.segs[s];
    const int W = e.width, B = e.bits, cmax = (1 << B) - 1;
    const float* src;
    int64_t sd;
    if (I.layout == SAQ_LAYOUT_TILES) {
        sd = 64;
        src = I.O + ((vv >> 6) * I.ld + e.col) * 64 + (vv & 63);
    } else if (I.layout == SAQ_LAYOUT_DIMS) {
        sd = I.ld;
        src = I.O + e.col * I.ld + vv;
    } else {
        sd = 1;
        src = I.O + vv * I.ld + e.col;
    }
    float o[CHUNKS];
    int c[CHUNKS];
    float vmax = 0.f;
#pragma unroll
    for (int k = 0; k < CHUNKS; ++k) {
        o[k] = 0.f;
        if (64 * k < W && 64 * k + lane < W) o[k] = src[int64_t(64 * k + lane) * sd];
    }
#pragma unroll
    for (int k = 0; k < CHUNKS; ++k) vmax = fmaxf(vmax, fabsf(o[k]));
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) vmax = fmaxf(vmax, __shfl_xor(vmax, m));
    const bool zero = !(vmax > 0.f);

    // initial codes, as in quantize_kernel
    const double vd = zero ? ldexp(1.0, B - 1) : double(vmax);
    const double delta = zero ? 1.0 : ldexp(2.0 * vd, -B);
    const double inv = zero ? 1.0 : ldexp(0.5 / vd, B);
    const double half = 0.5 * double(cmax);
    float* lo = smem + wave * 2 * args.lds_w;
    float* lu = lo + args.lds_w;
    double nn = 0.0;
#pragma unroll
    for (int k = 0; k < CHUNKS; ++k) {
        c[k] = 0;
        if (64 * k >= W) continue;
        const double av = double(o[k]) + vd;
        const double q = floor(av * inv);
        const double r = fma(-q, delta, av);
        int code = int(q) + (r >= delta ? 1 : 0) - (r < 0.0 ? 1 : 0);
        code = min(max(code, 0), cmax);
        const bool in = 64 * k + lane < W;
        const double u = in ? double(code) - half : 0.0;
        c[k] = in ? code : 0;
        nn = fma(u, u, nn);
        lo[64 * k + lane] = in ? o[k] : 0.f;
        lu[64 * k + lane] = float(u);          // exact: a half-integer below 2^16
    }
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) {
        const int xl = __shfl_xor(__double2loint(nn), m), xh = __shfl_xor(__double2hiint(nn), m);
        nn += __hiloint2double(xh, xl);        // multiples of 1/4 below 2^41: exact
    }
    __syncthreads();
    if (threadIdx.x < 2 * VECTORS) {
        // the sums in the order of the dims (zeros behind the last one)
        const int w = threadIdx.x & (VECTORS - 1);
        const float4* a = reinterpret_cast<const float4*>(smem + (2 * w + (threadIdx.x < VECTORS ? 1 : 0)) * args.lds_w);
        const float4* bb = reinterpret_cast<const float4*>(smem + 2 * w * args.lds_w);
        double acc = 0.0;
        for (int j = 0; 4 * j < W; ++j) {
            const float4 x = a[j], y = bb[j];
            acc = fma(double(x.x), double(y.x), acc);
            acc = fma(double(x.y), double(y.y), acc);
            acc = fma(double(x.z), double(y.z), acc);
            acc = fma(double(x.w), double(y.w), acc);
        }
        sums[threadIdx.x] = acc;
    }
    __syncthreads();
    if (!live) return;
    double ip = sums[wave];
    const double oo = sums[VECTORS + wave];

    // Algorithm 1
    if (B >= 2 && args.rounds > 0) {
        const double cmd = double(cmax);
        double P = 2.0 * ip, nS = -(ip * ip);
        for (int rd = 0; rd < args.rounds; ++rd) {
            bool moved = false;
#pragma unroll
            for (int k = 0; k < CHUNKS; ++k) {
                if (64 * k >= W) break;
                const double x = double(o[k]);
                const int width = min(64, W - 64 * k);
                uint64_t pending = width == 64 ? ~0ull : (1ull << width) - 1;
                for (;;) {
                    const double w = fma(2.0, double(c[k]), -cmd);
                    const double no = nn * x;
                    const double A = fma(no, x, nS);
                    const double Bv = fma(no, P, nS * w);
                    const bool up = c[k] < cmax && Bv > -A;
                    const bool dn = c[k] > 0 && A > Bv;
                    const uint64_t take = __ballot(up || dn) & pending;
                    if (take == 0) break;
                    const int f = __builtin_ctzll(take);
                    // what the move makes of the state, in every lane for its own dim
                    const double sg = up ? 1.0 : -1.0;
                    const double nn1 = nn + fma(sg, w, 1.0);
                    const double ip1 = fma(sg, x, ip);
                    nn = lane_value(nn1, f);
                    ip = lane_value(ip1, f);
                    P = 2.0 * ip;
                    nS = -(ip * ip);
                    if (lane == f) c[k] += up ? 1 : -1;
                    moved = true;
                    pending &= f == 63 ? 0ull : ~0ull << (f + 1);
                    if (pending == 0) break;
                }
            }
            if (!moved) break;
        }
    }

    if (lane == 0) {
        I.factors[v * (I.n_kept + 1) + s] = zero ? 0.f : float(oo / ip);
        if (s == 0) I.factors[v * (I.n_kept + 1) + I.n_kept] = I.norm2[v];
    }
    // bit planes, most significant first: lane q takes plane q's 8 bytes of a
    // 64-dim chunk
    const int pb = (W + 7) >> 3;
    uint8_t* dst = I.codes + v * I.code_bytes + e.code_off;
#pragma unroll
    for (int k = 0; k < CHUNKS; ++k) {
        if (64 * k >= W) break;
        uint64_t mine = 0;
        for (int q = 0; q < B; ++q) {
            const uint64_t m = __ballot((c[k] >> (B - 1 - q)) & 1);
            if (lane == q) mine = m;
        }
        if (lane < B) {
            uint8_t* p = dst + int64_t(lane) * pb + 8 * k;
            const int left = pb - 8 * k;
            if (left >= 8) {
                __builtin_memcpy(p, &mine, 8);
            } else {
                for (int i = 0; i < left; ++i) p[i] = uint8_t(mine >> (8 * i));
            }
        }
    }
}

}  // namespace

namespace saq {

// Where the line lies.  quantize_kernel with a workgroup per segment takes
// about 0.3 to 0.5 us per dim of the widest segment however few the vectors;
// this kernel's time grows with vectors x (dims + about 60 per segment).
// Measured, us here / there: D = 768, 4 b/dim (widest segment 80) 22 / 46 at
// 1,000 vectors, 63 / 50 at 4,000; 6 b/dim (240) 78 / 114 at 4,000, 141 / 118
// at 8,000; D = 1536 (144) 32 / 74 and 98 / 82; D = 3072, 2 b/dim (512) 48 /
// 121 and 135 / 133; D = 128 (16) 11 / 17 and 31 / 17.
bool few_vectors(const QuantItem* items, int count) {
    int64_t work = 0, widest = 0;
    for (int i = 0; i < count; ++i) {
        if (items[i].n_kept <= 0 || items[i].max_w > MAXW || items[i].norm2 == nullptr) return false;
        work += items[i].n * (items[i].dk + 60 * items[i].n_kept);
        widest = std::max<int64_t>(widest, items[i].max_w);
    }
    return work <= 32768 * widest;
}

saq_status launch_quantize_few(const QuantItem* items, int count, int rounds, hipStream_t st) {
    QuantFewArgs a{};
    a.count = count;
    a.rounds = rounds;
    int w = 64;
    int64_t blocks = 0;
    for (int i = 0; i < count; ++i) {
        a.item[i] = items[i];
        a.first_block[i] = blocks;
        blocks += (items[i].n + VECTORS - 1) / VECTORS * items[i].n_kept;
        w = std::max(w, (items[i].max_w + 63) / 64 * 64);
    }
    a.lds_w = w;
    hipLaunchKernelGGL(quantize_few_kernel, dim3(unsigned(blocks)), dim3(64 * VECTORS),
                       size_t(VECTORS) * 2 * w * sizeof(float), st, a);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? SAQ_OK : hip_status(e, "quantize_few_kernel launch");
}

}  // namespace saq
