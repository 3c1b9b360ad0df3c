// libsaq device fit: mean and covariance of the fit sample on the GPU
// (Section 4.1), for saq_covariance and saq_fit_plan_device.
//
//   mean_part_kernel / mean_reduce_kernel
//       FP64 column sums over fixed blocks of 4,096 sample rows, added in
//       block order: the same order as the host fit, so the mean is the
//       host fit's bit for bit.
//   cov_kernel
//       (1/m) sum_r (x_r - c)(x_r - c)^T as an FP64 matrix-core contraction
//       (v_mfma_f64_16x16x4_f64): one 64 x 64 output tile of the upper
//       triangle per workgroup, over one slice of the sample rows; rows are
//       staged in LDS as FP64 x - c, 32 rows per step, the next step's raw
//       FP32 values loaded during the current step's MFMAs.
//   cov_reduce_kernel
//       adds the row slices of each element in slice order, divides by m and
//       writes both triangles.
//   jacobi_*_kernel
//       the covariance's eigen-decomposition (the PCA basis of Section 4.1)
//       by the cyclic Jacobi method with a parallel ordering: in each round
//       the indices form n/2 disjoint pairs (the round-robin tournament
//       schedule), one plane rotation per pair zeroes that pair's
//       off-diagonal entry, and the rotations of a round commute, so
//       A <- J^T A J is applied at once: each 2 x 2 block (pair P rows, pair
//       Q columns) of A, B' = R_P^T B R_Q, goes from one buffer into the
//       other.  The rounds' rotations are kept, and V <- V J is applied for a
//       whole sweep, its rows being independent.
//       n - 1 rounds make a sweep; sweeps repeat until the off-diagonal
//       mass is below FP64 rounding of the diagonal (Jacobi 1846; the
//       parallel ordering of Brent and Luk 1985; the rotation formulas of
//       Rutishauser, Numer. Math. 9, 1966).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <string>
#include <vector>

#include "plan.hpp"

typedef double doublex4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int MEAN_ROWS = 4096;   // rows per partial mean (the host fit's block)
constexpr int CT = 64;            // covariance output tile
constexpr int CK = 32;            // sample rows per k-step
constexpr int CSTR = CT + 2;      // doubles per LDS row

__device__ __forceinline__ int64_t sample_row(int64_t i, int64_t n, int64_t m) {
    return m == n ? i : (i * n) / m;
}

// One lane per column and 4,096-row block.  The sum is one chain in row order
// (the host's), so what counts is loads in flight: MEAN_AHEAD rows are loaded
// while the ones before them are added.  65,536 x 960: 1,665 us with one load
// at a time, 265 us so.
constexpr int MEAN_AHEAD = 32;
__global__ __launch_bounds__(64) void mean_part_kernel(const float* __restrict__ X, int64_t n, int D,
                                                       int64_t m, double* __restrict__ part) {
    const int k = blockIdx.x * 64 + threadIdx.x;
    const int64_t b = blockIdx.y;
    if (k >= D) return;
    double s = 0.0;
    const int64_t i0 = b * MEAN_ROWS, i1 = std::min<int64_t>(m, i0 + MEAN_ROWS);
    float cur[MEAN_AHEAD], nxt[MEAN_AHEAD];
    auto load = [&](int64_t i, float (&v)[MEAN_AHEAD]) {
#pragma unroll
        for (int e = 0; e < MEAN_AHEAD; ++e) v[e] = X[sample_row(std::min(i + e, i1 - 1), n, m) * D + k];
    };
    load(i0, cur);
    int64_t i = i0;
    for (; i + MEAN_AHEAD <= i1; i += MEAN_AHEAD) {
        load(std::min(i + MEAN_AHEAD, i1 - 1), nxt);
#pragma unroll
        for (int e = 0; e < MEAN_AHEAD; ++e) s += double(cur[e]);
#pragma unroll
        for (int e = 0; e < MEAN_AHEAD; ++e) cur[e] = nxt[e];
    }
#pragma unroll
    for (int e = 0; e < MEAN_AHEAD; ++e)
        if (i + e < i1) s += double(cur[e]);
    part[b * D + k] = s;
}

__global__ __launch_bounds__(256) void mean_reduce_kernel(const double* __restrict__ part, int64_t nb,
                                                          int D, int64_t m, double* __restrict__ mu) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= D) return;
    double s = 0.0;
    for (int64_t b = 0; b < nb; ++b) s += part[b * D + k];
    mu[k] = s / double(m);
}

// Upper-triangle tile t (row block I <= column block J) of an nt x nt grid.
__device__ __forceinline__ void tile_of(int t, int nt, int& I, int& J) {
    I = 0;
    while (t >= nt - I) { t -= nt - I; ++I; }
    J = I + t;
}

// grid: (upper tiles, row slices).  part: [slices][D][D], only the upper
// tiles' elements written.  Wave w computes rows 32 (w/2) .. +31 and columns
// 32 (w%2) .. +31 of the tile as 2 x 2 blocks of 16 x 16.
__global__ __launch_bounds__(256) void cov_kernel(const float* __restrict__ X, int64_t n, int D,
                                                  int64_t m, const double* __restrict__ mu,
                                                  int64_t slice_rows, int vec,
                                                  double* __restrict__ part) {
    __shared__ __attribute__((aligned(16))) double Ya[2][CK * CSTR];
    __shared__ __attribute__((aligned(16))) double Yb[2][CK * CSTR];
    const int nt = (D + CT - 1) / CT;
    int I, J;
    tile_of(blockIdx.x, nt, I, J);
    const int i0 = I * CT, j0 = J * CT;
    const int64_t r_begin = int64_t(blockIdx.y) * slice_rows;
    const int64_t r_end = std::min<int64_t>(m, r_begin + slice_rows);
    const int t = threadIdx.x;
    const int wave = t >> 6, lane = t & 63;
    const int wi = wave >> 1, wj = wave & 1;
    const int li = lane & 15, lk = lane >> 4;

    // staging: thread t loads row t/8 of the step, columns 8 (t%8) .. +7 of
    // both column blocks
    const int sr = t >> 3, sc = (t & 7) * 8;
    double ma[8], mb[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        ma[e] = (i0 + sc + e < D) ? mu[i0 + sc + e] : 0.0;
        mb[e] = (j0 + sc + e < D) ? mu[j0 + sc + e] : 0.0;
    }
    float ra[8], rb[8];
    // 8 consecutive floats of one row per column block: two 16-byte loads
    // when rows are 16-byte aligned and the 8 columns are inside D
    auto load8 = [&](const float* x, int c0, bool live, float (&r)[8]) {
        if (vec && live && c0 + 8 <= D) {
            const float4 u = *reinterpret_cast<const float4*>(x + c0);
            const float4 v = *reinterpret_cast<const float4*>(x + c0 + 4);
            r[0] = u.x; r[1] = u.y; r[2] = u.z; r[3] = u.w;
            r[4] = v.x; r[5] = v.y; r[6] = v.z; r[7] = v.w;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) r[e] = (live && c0 + e < D) ? x[c0 + e] : 0.f;
        }
    };
    auto load = [&](int64_t r0) {
        const int64_t r = r0 + sr;
        const bool live = r < r_end;
        const float* x = X + (live ? sample_row(r, n, m) : 0) * int64_t(D);
        load8(x, i0 + sc, live, ra);
        load8(x, j0 + sc, live, rb);
    };
    auto store = [&](int64_t r0, int buf) {
        const bool live = r0 + sr < r_end;
        // x - c in FP64 (exact for FP32 x); rows past the slice and columns
        // past D are 0 and add nothing.  Stored as pairs (16-byte LDS writes).
        double2* ya = reinterpret_cast<double2*>(&Ya[buf][sr * CSTR + sc]);
        double2* yb = reinterpret_cast<double2*>(&Yb[buf][sr * CSTR + sc]);
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            double2 va, vb;
            va.x = (live && i0 + sc + e < D) ? double(ra[e]) - ma[e] : 0.0;
            va.y = (live && i0 + sc + e + 1 < D) ? double(ra[e + 1]) - ma[e + 1] : 0.0;
            vb.x = (live && j0 + sc + e < D) ? double(rb[e]) - mb[e] : 0.0;
            vb.y = (live && j0 + sc + e + 1 < D) ? double(rb[e + 1]) - mb[e + 1] : 0.0;
            ya[e / 2] = va;
            yb[e / 2] = vb;
        }
    };

    doublex4 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = doublex4{0.0, 0.0, 0.0, 0.0};

    if (r_begin < r_end) {
        load(r_begin);
        store(r_begin, 0);
        __syncthreads();
        for (int64_t r0 = r_begin, step = 0; r0 < r_end; r0 += CK, ++step) {
            const int buf = int(step & 1);
            const bool more = r0 + CK < r_end;
            if (more) load(r0 + CK);
            const double* A = Ya[buf];
            const double* B = Yb[buf];
#pragma unroll
            for (int k = 0; k < CK; k += 4) {
                // A[i][kk] = y_{r0+k+kk}[i0 + i], B[kk][j] = y_{r0+k+kk}[j0 + j]
                const double a0 = A[(k + lk) * CSTR + wi * 32 + li];
                const double a1 = A[(k + lk) * CSTR + wi * 32 + 16 + li];
                const double b0 = B[(k + lk) * CSTR + wj * 32 + li];
                const double b1 = B[(k + lk) * CSTR + wj * 32 + 16 + li];
                acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
                acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
                acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
                acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
            }
            if (more) store(r0 + CK, buf ^ 1);
            __syncthreads();
        }
    }
    // the FP64 16 x 16 result is row-interleaved: lane holds, for register
    // q, row 4 q + lane/16 and column lane%16 of each block
    double* P = part + int64_t(blockIdx.y) * D * D;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int col = j0 + wj * 32 + b * 16 + li;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int row = i0 + wi * 32 + a * 16 + 4 * q + lk;
                if (row < D && col < D) P[int64_t(row) * D + col] = acc[a][b][q];
            }
        }
}

// cov[i][j] = cov[j][i] = (sum over slices, in order) / m for i <= j
__global__ __launch_bounds__(256) void cov_reduce_kernel(const double* __restrict__ part, int slices,
                                                         int D, int64_t m, double* __restrict__ cov) {
    const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (e >= int64_t(D) * D) return;
    const int i = int(e / D), j = int(e % D);
    if (i > j) return;
    double s = 0.0;
    for (int sl = 0; sl < slices; ++sl) s += part[int64_t(sl) * D * D + e];
    const double v = s / double(m);
    cov[int64_t(i) * D + j] = v;
    cov[int64_t(j) * D + i] = v;
}

// ---------------------------------------------------------------------------
// Cyclic Jacobi on the device.  N is n rounded up to even; a padded index
// has a zero row and column, so its rotations are the identity and its
// column of V stays a unit vector outside the first n rows and columns.
// ---------------------------------------------------------------------------
// the pair k (k < N/2) of round r of the round-robin schedule on N players:
// player N - 1 stays, the others rotate
__device__ __forceinline__ void jacobi_pair(int N, int r, int k, int& a, int& b) {
    if (k == 0) {
        a = r;
        b = N - 1;
    } else {
        const int m = N - 1;         // 0 <= r < m, 0 < k < m
        a = r + k < m ? r + k : r + k - m;
        b = r >= k ? r - k : r - k + m;
    }
    if (a > b) {
        const int t = a;
        a = b;
        b = t;
    }
}

// (c, s) of R = [[c, s], [-s, c]] with (R^T [[app, apq], [apq, aqq]] R)[0][1] = 0,
// the smaller of the two angles
__device__ __forceinline__ void jacobi_rotation(double app, double aqq, double apq, double& c,
                                                double& s) {
    if (apq == 0.0) {
        c = 1.0;
        s = 0.0;
        return;
    }
    const double th = (aqq - app) / (2.0 * apq);
    double t;
    if (fabs(th) > 1e150) {
        t = 0.5 / th;
    } else {
        t = 1.0 / (fabs(th) + sqrt(th * th + 1.0));
        if (th < 0.0) t = -t;
    }
    c = 1.0 / sqrt(t * t + 1.0);
    s = t * c;
}

// (x, y) -> (c x - s y, s x + c y).  The roundings are spelled out: the sign
// and order of the eigenvectors follow from them (a rotation of two nearly
// equal diagonal entries may turn either way).
__device__ __forceinline__ void rotate2(double x, double y, double c, double s, double& x1, double& y1) {
    x1 = fma(c, x, -(s * y));
    y1 = fma(s, x, c * y);
}

// R_P^T B R_Q of the block of a row pair and a column pair, rows first; own: the
// pair's own block, whose off-diagonal entries are zero by construction
struct Block { double v[2][2]; };
__device__ __forceinline__ Block rotate_block(const Block& b, double2 p, double2 q, bool own) {
    double r00, r01, r10, r11;
    Block n;
    rotate2(b.v[0][0], b.v[1][0], p.x, p.y, r00, r10);
    rotate2(b.v[0][1], b.v[1][1], p.x, p.y, r01, r11);
    rotate2(r00, r01, q.x, q.y, n.v[0][0], n.v[0][1]);
    rotate2(r10, r11, q.x, q.y, n.v[1][0], n.v[1][1]);
    if (own) n.v[0][1] = n.v[1][0] = 0.0;
    return n;
}

__global__ __launch_bounds__(256) void jacobi_init_kernel(const double* __restrict__ C, int n, int N,
                                                          double* __restrict__ A,
                                                          double* __restrict__ V) {
    const int64_t idx = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (idx >= int64_t(N) * N) return;
    const int i = int(idx / N), j = int(idx % N);
    A[idx] = (i < n && j < n) ? C[int64_t(i) * n + j] : 0.0;
    V[idx] = i == j ? 1.0 : 0.0;
}

// One round on A (the last one of a sweep, jacobi_two_kernel taking the others
// in twos): a workgroup takes the 2 x 2 blocks of JP row pairs and JQ
// column pairs of Ain into Aout.  The rotations of its pairs are computed once,
// by one thread each, while the blocks load (every thread computing both of
// its block's rotations, each two FP64 divisions and two square roots, was most
// of the round's work); the round's rotations also go to rot [pair], for the
// eigenvectors.  A round moves A once through the caches and waits for two
// loads in a row, with n - 1 launches a sweep: 12.5 us per round at n = 960
// with V and a thread per block, 5.7 so (5.6 / 6.0 / 7.3 at 4 / 16 / 32 row
// pairs).
constexpr int JP = 8, JQ = 64;
__global__ __launch_bounds__(256) void jacobi_round_kernel(const double* __restrict__ Ain,
                                                           double* __restrict__ Aout,
                                                           double2* __restrict__ rot, int N, int r) {
    __shared__ double2 cs[JQ + JP];
    const int h = N / 2, t = threadIdx.x;
    const int q_first = blockIdx.x * JQ, p_first = blockIdx.y * JP;
    const int kq = q_first + (t & (JQ - 1));
    auto at = [&](int i, int j) { return Ain[int64_t(i) * N + j]; };
    int q0 = 0, q1 = 0;
    if (kq < h) jacobi_pair(N, r, kq, q0, q1);
    double B[JP / 4][4];
#pragma unroll
    for (int e = 0; e < JP / 4; ++e) {
        const int kp = p_first + t / JQ + 4 * e;
        if (kq >= h || kp >= h) continue;
        int p0, p1;
        jacobi_pair(N, r, kp, p0, p1);
        B[e][0] = at(p0, q0); B[e][1] = at(p0, q1);
        B[e][2] = at(p1, q0); B[e][3] = at(p1, q1);
    }
    if (t < JQ + JP) {
        const int k = t < JQ ? q_first + t : p_first + t - JQ;
        if (k < h) {
            int a, b;
            jacobi_pair(N, r, k, a, b);
            double c, s;
            jacobi_rotation(at(a, a), at(b, b), at(a, b), c, s);
            cs[t] = make_double2(c, s);
            if (blockIdx.y == 0 && t < JQ) rot[k] = make_double2(c, s);
        }
    }
    __syncthreads();
    if (kq >= h) return;
    const double cq = cs[t & (JQ - 1)].x, sq = cs[t & (JQ - 1)].y;
#pragma unroll
    for (int e = 0; e < JP / 4; ++e) {
        const int kp = p_first + t / JQ + 4 * e;
        if (kp >= h) continue;
        int p0, p1;
        jacobi_pair(N, r, kp, p0, p1);
        const double cp = cs[JQ + kp - p_first].x, sp = cs[JQ + kp - p_first].y;
        const Block b{{{B[e][0], B[e][1]}, {B[e][2], B[e][3]}}};
        const Block n = rotate_block(b, make_double2(cp, sp), make_double2(cq, sq), kp == kq);
        Aout[int64_t(p0) * N + q0] = n.v[0][0];
        Aout[int64_t(p0) * N + q1] = n.v[0][1];
        Aout[int64_t(p1) * N + q0] = n.v[1][0];
        Aout[int64_t(p1) * N + q1] = n.v[1][1];
    }
}

// Rounds r and r + 1 on A in one pass over it (r + 2 < N).  A player's partner
// changes to that of a neighbouring pair, so pair k of round r + 1 is made of
// players of round r's pairs k - 1 .. k + 1: a workgroup that loads SP x SQ
// blocks of round r has what it needs for the (SP - 2) x (SQ - 2) inside them in
// round r + 1.  The rotations of round r + 1 need three entries of A after round
// r, which one thread per pair works out from the blocks that hold them.  Every
// entry sees the operations of two single rounds.  What bounds it is the chain of
// loads, two rotations and barriers: n = 960, two rounds 11.5 us one by one, 7.5
// so (8.7 with 16 x 32 blocks and 256 threads, 7.7 with 32 x 32 and 1,024).
constexpr int SP = 32, SQ = 64, IP = SP - 2, IQ = SQ - 2, TWO_T = 1024;
__global__ __launch_bounds__(TWO_T) void jacobi_two_kernel(const double* __restrict__ Ain,
                                                           double* __restrict__ Aout,
                                                           double2* __restrict__ rot, int N, int r) {
    __shared__ double2 T[2 * SP][SQ + 1];      // A after round r: [2 row slot + side][column slot]
    __shared__ double2 cs0[SQ + SP];           // rotations of round r: column slots, row slots
    __shared__ double2 cs1[IQ + IP];           // of round r + 1
    __shared__ int2 loc[IQ + IP];              // its players as 2 slot + side
    const int h = N / 2, t = threadIdx.x;
    const int q_first = int(blockIdx.x) * IQ - 1, p_first = int(blockIdx.y) * IP - 1;   // pairs of slot 0
    auto at = [&](int i, int j) { return Ain[int64_t(i) * N + j]; };
    auto load = [&](int kp, int kq) {
        int p0, p1, q0, q1;
        jacobi_pair(N, r, kp, p0, p1);
        jacobi_pair(N, r, kq, q0, q1);
        return Block{{{at(p0, q0), at(p0, q1)}, {at(p1, q0), at(p1, q1)}}};
    };
    auto inside = [&](int k) { return min(max(k, 0), h - 1); };   // slots past the pairs: never used
    constexpr int BLOCKS = SP * SQ / TWO_T;
    Block B[BLOCKS];
#pragma unroll
    for (int e = 0; e < BLOCKS; ++e)
        B[e] = load(inside(p_first + t / SQ + TWO_T / SQ * e), inside(q_first + t % SQ));
    // round r + 1's pairs, threads TWO_T - IQ - IP on: columns, then rows
    const int nx = t - (TWO_T - IQ - IP);
    const int first = nx < IQ ? q_first : p_first, k1 = first + 1 + (nx < IQ ? nx : nx - IQ);
    const bool next = nx >= 0 && k1 < h;
    Block X{}, Y{}, Z{};
    int ka = 0, kb = 0, sa = 0, sb = 0;
    if (next) {
        // player x in round r: its pair, and its side of it
        auto player = [&](int x, int& k, int& side) {
            const int m = N - 1, d = x >= r ? x - r : x - r + m;
            k = x == m ? 0 : d < h ? d : m - d;
            int a, b;
            jacobi_pair(N, r, k, a, b);
            side = x == b;
        };
        int a, b;
        jacobi_pair(N, r + 1, k1, a, b);
        player(a, ka, sa);
        player(b, kb, sb);
        X = load(ka, ka);
        Y = load(kb, kb);
        Z = load(ka, kb);
        loc[nx] = make_int2(2 * (ka - first) + sa, 2 * (kb - first) + sb);
    }
    if (t < SQ + SP) {
        const int k = t < SQ ? q_first + t : p_first + t - SQ;
        if (k >= 0 && k < h) {
            int a, b;
            jacobi_pair(N, r, k, a, b);
            double c, s;
            jacobi_rotation(at(a, a), at(b, b), at(a, b), c, s);
            cs0[t] = make_double2(c, s);
            if (blockIdx.y == 0 && t >= 1 && t <= IQ) rot[k] = make_double2(c, s);
        }
    }
    __syncthreads();
    if (next) {
        const double2* c0 = cs0 + (nx < IQ ? 0 : SQ) - first;
        X = rotate_block(X, c0[ka], c0[ka], true);
        Y = rotate_block(Y, c0[kb], c0[kb], true);
        Z = rotate_block(Z, c0[ka], c0[kb], false);
        auto side = [](const Block& b, int i, int j) {
            const double x = j ? b.v[0][1] : b.v[0][0], y = j ? b.v[1][1] : b.v[1][0];
            return i ? y : x;
        };
        double c, s;
        jacobi_rotation(side(X, sa, sa), side(Y, sb, sb), side(Z, sa, sb), c, s);
        cs1[nx] = make_double2(c, s);
        if (blockIdx.y == 0 && nx < IQ) rot[h + k1] = make_double2(c, s);
    }
#pragma unroll
    for (int e = 0; e < BLOCKS; ++e) {
        const int ip = t / SQ + TWO_T / SQ * e, iq = t % SQ;
        const Block n = rotate_block(B[e], cs0[SQ + ip], cs0[iq], p_first + ip == q_first + iq);
        T[2 * ip][iq] = make_double2(n.v[0][0], n.v[0][1]);
        T[2 * ip + 1][iq] = make_double2(n.v[1][0], n.v[1][1]);
    }
    __syncthreads();
    for (int i = t; i < IP * IQ; i += TWO_T) {
        const int ip = i / IQ, iq = i % IQ, kp = p_first + 1 + ip, kq = q_first + 1 + iq;
        if (kp >= h || kq >= h) continue;
        const int2 lp = loc[IQ + ip], lq = loc[iq];
        const double *row0 = reinterpret_cast<const double*>(T[lp.x]), *row1 = reinterpret_cast<const double*>(T[lp.y]);
        const Block n = rotate_block({{{row0[lq.x], row0[lq.y]}, {row1[lq.x], row1[lq.y]}}}, cs1[IQ + ip], cs1[iq],
                                     kp == kq);
        int p0, p1, q0, q1;
        jacobi_pair(N, r + 1, kp, p0, p1);
        jacobi_pair(N, r + 1, kq, q0, q1);
        Aout[int64_t(p0) * N + q0] = n.v[0][0];
        Aout[int64_t(p0) * N + q1] = n.v[0][1];
        Aout[int64_t(p1) * N + q0] = n.v[1][0];
        Aout[int64_t(p1) * N + q1] = n.v[1][1];
    }
}

// V <- V J for `rounds` rounds from r0 on, a sweep as a rule: the rows of V are
// independent, so a workgroup keeps ROWS of them in LDS and applies the rounds'
// rotations, one barrier per round and the next round's rotations in flight, instead of V
// passing through memory in every round.  KM: pairs per thread.  ROWS = 0: one
// row, in memory, for matrices whose rows LDS does not hold.  What bounds it is
// the chain of a round: two LDS reads, four products, two writes, a barrier.
template <int ROWS, int KM>
__global__ __launch_bounds__(256) void jacobi_vectors_kernel(const double2* __restrict__ rot,
                                                             double* __restrict__ V, int N, int r0,
                                                             int rounds) {
    extern __shared__ double lv[];
    constexpr int R = ROWS ? ROWS : 1;
    const int h = N / 2, t = threadIdx.x;
    const int64_t row0 = int64_t(blockIdx.x) * R;
    const int live = int(std::min<int64_t>(R, N - row0));
    double* rows = ROWS ? lv : V + row0 * N;
    if (ROWS)
        for (int i = t; i < live * N; i += 256) lv[i] = V[row0 * N + i];
    // pair k of round r, rotated by cs
    auto rotate = [&](int r, int k, double2 cs) {
        int a, b;
        jacobi_pair(N, r, k, a, b);
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if (i >= live) break;
            const double v0 = rows[int64_t(i) * N + a], v1 = rows[int64_t(i) * N + b];
            double w0, w1;
            rotate2(v0, v1, cs.x, cs.y, w0, w1);
            rows[int64_t(i) * N + a] = w0;
            rows[int64_t(i) * N + b] = w1;
        }
    };
    if constexpr (ROWS == 0) {
        for (int r = 0; r < rounds; ++r) {
            for (int k = t; k < h; k += 256) rotate(r0 + r, k, rot[int64_t(r) * h + k]);
            __syncthreads();
        }
        return;
    }
    double2 cur[KM], nxt[KM];
    auto load = [&](int r, double2 (&c)[KM]) {
#pragma unroll
        for (int e = 0; e < KM; ++e) c[e] = rot[int64_t(r) * h + std::min(t + 256 * e, h - 1)];
    };
    load(0, cur);
    __syncthreads();
    for (int r = 0; r < rounds; ++r) {
        load(std::min(r + 1, rounds - 1), nxt);
#pragma unroll
        for (int e = 0; e < KM; ++e)
            if (t + 256 * e < h) rotate(r0 + r, t + 256 * e, cur[e]);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < KM; ++e) cur[e] = nxt[e];
    }
    if (ROWS)
        for (int i = t; i < live * N; i += 256) V[row0 * N + i] = lv[i];
}

// per-block sums of squares: off-diagonal entries, diagonal entries
__global__ __launch_bounds__(256) void jacobi_off_kernel(const double* __restrict__ A, int N,
                                                         double* __restrict__ part) {
    __shared__ double so[256], sd[256];
    double off = 0.0, dg = 0.0;
    for (int64_t idx = int64_t(blockIdx.x) * 256 + threadIdx.x; idx < int64_t(N) * N;
         idx += int64_t(gridDim.x) * 256) {
        const double a = A[idx];
        if (idx / N == idx % N) dg += a * a;
        else off += a * a;
    }
    so[threadIdx.x] = off;
    sd[threadIdx.x] = dg;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (int(threadIdx.x) < w) {
            so[threadIdx.x] += so[threadIdx.x + w];
            sd[threadIdx.x] += sd[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = so[0];
        part[2 * blockIdx.x + 1] = sd[0];
    }
}

// w[j] = A[j][j], Vout = the first n rows and columns of V
__global__ __launch_bounds__(256) void jacobi_finish_kernel(const double* __restrict__ A,
                                                            const double* __restrict__ V, int n,
                                                            int N, double* __restrict__ w,
                                                            double* __restrict__ Vout) {
    const int64_t idx = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (idx >= int64_t(n) * n) return;
    const int i = int(idx / n), j = int(idx % n);
    Vout[idx] = V[int64_t(i) * N + j];
    if (i == j) w[i] = A[int64_t(i) * N + i];
}

constexpr int JACOBI_OFF_BLOCKS = 256;
constexpr int JACOBI_MAX_SWEEPS = 40;

struct CovShape {
    int64_t m = 0, nb = 0, slice_rows = 0;
    int nt = 0, tiles = 0, slices = 0;
    int64_t off_mpart = 0, off_part = 0, bytes = 0;
};

int64_t align256(int64_t v) { return (v + 255) & ~int64_t(255); }

CovShape cov_shape(int64_t n, int32_t D, int64_t fit_sample) {
    CovShape S;
    S.m = (fit_sample > 0 && fit_sample < n) ? fit_sample : n;
    S.nb = (S.m + MEAN_ROWS - 1) / MEAN_ROWS;
    S.nt = (D + CT - 1) / CT;
    S.tiles = S.nt * (S.nt + 1) / 2;
    // enough row slices to give the chip about 2,048 workgroups, each slice
    // at least 1,024 rows
    const int64_t want = std::max<int64_t>(1, (2048 + S.tiles - 1) / S.tiles);
    const int64_t most = std::max<int64_t>(1, S.m / 1024);
    S.slices = int(std::min<int64_t>(std::min<int64_t>(want, most), 64));
    S.slice_rows = ((S.m + S.slices - 1) / S.slices + CK - 1) / CK * CK;
    S.slices = int((S.m + S.slice_rows - 1) / S.slice_rows);
    S.off_mpart = 0;
    S.off_part = align256(S.nb * D * 8);
    S.bytes = S.off_part + int64_t(S.slices) * D * D * 8 + 256;
    return S;
}

saq_status hip_err(hipError_t e, const char* what) {
    return saq::fail(SAQ_EDEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

saq_status run_covariance(const float* X, int64_t n, int32_t D, int64_t fit_sample, double* mu,
                          double* cov, void* ws, int64_t ws_bytes, hipStream_t st) {
    const CovShape S = cov_shape(n, D, fit_sample);
    if (ws_bytes < S.bytes) return saq::fail(SAQ_EINVAL, "workspace too small");
    char* base = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255));
    double* mpart = reinterpret_cast<double*>(base + S.off_mpart);
    double* part = reinterpret_cast<double*>(base + S.off_part);
    const unsigned cb = unsigned((D + 255) / 256);
    hipLaunchKernelGGL(mean_part_kernel, dim3(unsigned((D + 63) / 64), unsigned(S.nb)), dim3(64), 0, st, X, n, D, S.m, mpart);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_err(e, "mean_part_kernel launch");
    hipLaunchKernelGGL(mean_reduce_kernel, dim3(cb), dim3(256), 0, st, mpart, S.nb, D, S.m, mu);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_err(e, "mean_reduce_kernel launch");
    const int vec = (D % 4 == 0) && ((reinterpret_cast<uintptr_t>(X) & 15) == 0);
    hipLaunchKernelGGL(cov_kernel, dim3(unsigned(S.tiles), unsigned(S.slices)), dim3(256), 0, st, X, n, D,
                       S.m, mu, S.slice_rows, vec, part);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_err(e, "cov_kernel launch");
    const int64_t el = int64_t(D) * D;
    hipLaunchKernelGGL(cov_reduce_kernel, dim3(unsigned((el + 255) / 256)), dim3(256), 0, st, part,
                       S.slices, D, S.m, cov);
    e = hipGetLastError();
    return e == hipSuccess ? SAQ_OK : hip_err(e, "cov_reduce_kernel launch");
}

// two buffers of A, V; the rotations go to the caller's V until it is written
int64_t jacobi_bytes(int32_t n) {
    const int64_t N = n + (n & 1);
    return 3 * align256(N * N * 8) + align256(int64_t(JACOBI_OFF_BLOCKS) * 2 * 8) + 256;
}

// V <- V J of rounds r0 .. r0 + rounds - 1
void launch_vectors(const double2* rot, double* V, int N, int r0, int rounds, hipStream_t st) {
    const size_t row = size_t(N) * 8;
#define SAQ_LAUNCH_V(ROWS, KM)                                                                      \
    hipLaunchKernelGGL((jacobi_vectors_kernel<ROWS, KM>),                                           \
                       dim3(unsigned((N + (ROWS ? ROWS : 1) - 1) / (ROWS ? ROWS : 1))), dim3(256),  \
                       ROWS * row, st, rot, V, N, r0, rounds)
    // ROWS rows within 64 KB.  Few rows: a round's chain hardly depends on
    // them, and rows spread over more CUs (n = 960, a sweep: 693 us with 4,
    // 520 with 2, 477 with 1; 2 halves the reads of the rotations).
    if (N <= 512) SAQ_LAUNCH_V(2, 1);
    else if (N <= 1024) SAQ_LAUNCH_V(2, 2);
    else if (N <= 2048) SAQ_LAUNCH_V(2, 4);
    else if (N <= 4096) SAQ_LAUNCH_V(2, 8);
    else if (N <= 8192) SAQ_LAUNCH_V(1, 16);
    else SAQ_LAUNCH_V(0, 1);
#undef SAQ_LAUNCH_V
}

// eigen-decomposition of the symmetric C [n x n] (device): w [n] in the
// Jacobi order, V [n x n] row-major with eigenvector j in column j; waits
// for `st` once per sweep (the convergence test)
saq_status run_jacobi(const double* C, int32_t n, double* w, double* V, void* ws, int64_t ws_bytes,
                      hipStream_t st) {
    if (ws_bytes < jacobi_bytes(n)) return saq::fail(SAQ_EINVAL, "workspace too small");
    const int N = n + (n & 1);
    const int64_t el = int64_t(N) * N;
    char* base = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255));
    double* A[2] = {reinterpret_cast<double*>(base), reinterpret_cast<double*>(base + align256(el * 8))};
    double* Vw = reinterpret_cast<double*>(base + 2 * align256(el * 8));
    double* part = reinterpret_cast<double*>(base + 3 * align256(el * 8));
    // The rotations of a sweep, N - 1 rounds of N doubles, wait in V, which is
    // written at the end only: all of them for an even n, all but the last round
    // for an odd one (or a V that is 8 bytes off).  A small n's fit in `part`, which
    // is written and read after them.
    double2* rot = reinterpret_cast<double2*>(part);
    int64_t room = int64_t(JACOBI_OFF_BLOCKS) * 2 / N;
    if (room < N - 1) {
        const int64_t off = (reinterpret_cast<uintptr_t>(V) & 15) ? 1 : 0;
        rot = reinterpret_cast<double2*>(V + off);
        room = (int64_t(n) * n - off) / N;
    }
    const unsigned gel = unsigned((el + 255) / 256);
    const dim3 gpair(unsigned((N / 2 + JQ - 1) / JQ), unsigned((N / 2 + JP - 1) / JP));
    const dim3 gtwo(unsigned((N / 2 + IQ - 1) / IQ), unsigned((N / 2 + IP - 1) / IP));
    hipLaunchKernelGGL(jacobi_init_kernel, dim3(gel), dim3(256), 0, st, C, n, N, A[0], Vw);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_err(e, "jacobi_init_kernel launch");
    std::vector<double> hp(size_t(JACOBI_OFF_BLOCKS) * 2);
    int cur = 0;
    bool converged = false;
    for (int sweep = 0; sweep < JACOBI_MAX_SWEEPS && !converged; ++sweep) {
        // an odd number of rounds: two at a time, then the last
        int r0 = 0;
        for (int r = 0; r + 1 < N; r += 2) {
            const int rounds = r + 2 < N ? 2 : 1;
            if (r + rounds - r0 > room) {
                launch_vectors(rot, Vw, N, r0, r - r0, st);
                r0 = r;
            }
            double2* rr = rot + int64_t(r - r0) * (N / 2);
            if (rounds == 2) hipLaunchKernelGGL(jacobi_two_kernel, gtwo, dim3(TWO_T), 0, st, A[cur], A[cur ^ 1], rr, N, r);
            else hipLaunchKernelGGL(jacobi_round_kernel, gpair, dim3(256), 0, st, A[cur], A[cur ^ 1], rr, N, r);
            cur ^= 1;
        }
        launch_vectors(rot, Vw, N, r0, N - 1 - r0, st);
        e = hipGetLastError();
        if (e != hipSuccess) return hip_err(e, "jacobi_round_kernel launch");
        hipLaunchKernelGGL(jacobi_off_kernel, dim3(JACOBI_OFF_BLOCKS), dim3(256), 0, st, A[cur], N, part);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipMemcpyAsync(hp.data(), part, hp.size() * 8, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return hip_err(e, "jacobi convergence test");
        double off = 0.0, dg = 0.0;
        for (int b = 0; b < JACOBI_OFF_BLOCKS; ++b) {
            off += hp[2 * b];
            dg += hp[2 * b + 1];
        }
        // below FP64 rounding of the diagonal: further rotations change
        // nothing in the eigenvalues' leading 15 digits
        converged = off <= 1e-30 * dg;
    }
    if (!converged) return saq::fail(SAQ_EINVAL, "Jacobi eigen-decomposition did not converge");
    hipLaunchKernelGGL(jacobi_finish_kernel, dim3(unsigned((int64_t(n) * n + 255) / 256)), dim3(256), 0,
                       st, A[cur], Vw, n, N, w, V);
    e = hipGetLastError();
    return e == hipSuccess ? SAQ_OK : hip_err(e, "jacobi_finish_kernel launch");
}

// the fit's own buffers ahead of the covariance workspace: mean,
// covariance, eigenvalues, eigenvectors, then the Jacobi workspace
int64_t fit_extra(int32_t D) {
    return align256(int64_t(D) * 8) + align256(int64_t(D) * D * 8) + align256(int64_t(D) * 8) +
           align256(int64_t(D) * D * 8) + jacobi_bytes(D);
}

}  // namespace

extern "C" {

int64_t saq_covariance_workspace_bytes(int64_t n, int32_t D, int64_t fit_sample) {
    if (n <= 0 || D <= 0 || fit_sample < 0) return -1;
    return cov_shape(n, D, fit_sample).bytes;
}

saq_status saq_covariance(const float* X_dev, int64_t n, int32_t D, int64_t fit_sample,
                          double* mean_dev, double* cov_dev, void* ws_dev, int64_t ws_bytes,
                          void* stream) {
    if (n <= 0 || D <= 0 || fit_sample < 0) return saq::fail(SAQ_EINVAL, "bad sizes");
    if (!X_dev || !mean_dev || !cov_dev || !ws_dev) return saq::fail(SAQ_EINVAL, "null buffer");
    return run_covariance(X_dev, n, D, fit_sample, mean_dev, cov_dev, ws_dev, ws_bytes,
                          static_cast<hipStream_t>(stream));
}

int64_t saq_sym_eigen_workspace_bytes(int32_t n) {
    if (n <= 0) return -1;
    return jacobi_bytes(n);
}

saq_status saq_sym_eigen_device(const double* A_dev, int32_t n, double* w_dev, double* V_dev,
                                void* ws_dev, int64_t ws_bytes, void* stream) {
    if (n <= 0) return saq::fail(SAQ_EINVAL, "bad size");
    if (!A_dev || !w_dev || !V_dev || !ws_dev) return saq::fail(SAQ_EINVAL, "null buffer");
    return run_jacobi(A_dev, n, w_dev, V_dev, ws_dev, ws_bytes, static_cast<hipStream_t>(stream));
}

int64_t saq_fit_workspace_bytes(int64_t n, int32_t D, const saq_plan_params* p) {
    if (!p || n <= 0 || D <= 0 || p->fit_sample < 0) return -1;
    return fit_extra(D) + cov_shape(n, D, p->fit_sample).bytes + 256;
}

saq_status saq_fit_plan_device(const float* X_dev, int64_t n, int32_t D, const saq_plan_params* p,
                               void* ws_dev, int64_t ws_bytes, void* stream, saq_plan** out) {
    if (!X_dev || !p || !out || !ws_dev || n <= 0 || D <= 0 || p->fit_sample < 0)
        return saq::fail(SAQ_EINVAL, "bad arguments");
    if (ws_bytes < saq_fit_workspace_bytes(n, D, p)) return saq::fail(SAQ_EINVAL, "workspace too small");
    hipStream_t st = static_cast<hipStream_t>(stream);
    char* base = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws_dev) + 255) & ~uintptr_t(255));
    const int64_t dv = align256(int64_t(D) * 8), dm = align256(int64_t(D) * D * 8);
    double* mu = reinterpret_cast<double*>(base);
    double* cov = reinterpret_cast<double*>(base + dv);
    double* w = reinterpret_cast<double*>(base + dv + dm);
    double* V = reinterpret_cast<double*>(base + 2 * dv + dm);
    char* jws = base + 2 * dv + 2 * dm;
    char* rest = base + fit_extra(D);
    const int64_t rest_bytes = ws_bytes - (rest - static_cast<char*>(ws_dev));
    saq_status s = run_covariance(X_dev, n, D, p->fit_sample, mu, cov, rest, rest_bytes, st);
    if (s != SAQ_OK) return s;
    s = run_jacobi(cov, D, w, V, jws, jacobi_bytes(D), st);
    if (s != SAQ_OK) return s;
    try {
        std::vector<double> hm(static_cast<size_t>(D)), hw(static_cast<size_t>(D)),
            hv(static_cast<size_t>(D) * D);
        hipError_t e = hipMemcpyAsync(hm.data(), mu, size_t(D) * 8, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipMemcpyAsync(hw.data(), w, size_t(D) * 8, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess)
            e = hipMemcpyAsync(hv.data(), V, size_t(D) * D * 8, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return hip_err(e, "copying the basis to the host");
        // the plan search on the host, from the device's basis (sorted there)
        return saq_plan_from_basis(hm.data(), hv.data(), hw.data(), D, p, out);
    } catch (const std::bad_alloc&) {
        return saq::fail(SAQ_ENOMEM, "out of host memory");
    }
}

}  // extern "C"
