// resample.hip -- the steps after the k-distribution (§2.6, eq. 5):
// least-squares Chebyshev coefficients of ln kappa(y) per bin, and the
// transmission function T(m) = int_0^1 exp(-kappa(y) m) dy.
//
// The design matrix A[i][c] = T_c(t_i), t_i = 2 (i + 1/2)/M - 1, is the same
// for every bin of M points, so its QR factors (A = QR, made once: here for
// bins of at least kMfmaRows points, on the host by Householder for smaller
// ones) are shared: per bin the kernels form Q^T d
// (d_i = ln kappa_i of the sorted bin) and solve R C = Q^T d.  Over all bins
// Q^T d is one matrix product, taken by the matrix cores for bins of at least
// kMfmaRows points.
#include <algorithm>

#include "hk_internal.h"

namespace hk {
namespace {

constexpr int kThreads = 256;

__device__ inline double key_to_double(const double* s, int64_t i) { return s[i]; }
__device__ inline double key_to_double(const float* s, int64_t i) { return (double)s[i]; }

// Bins of few points, and calls without scratch: one workgroup per bin.  Q:
// row-major [M][nc]; R: row-major [nc][nc], upper triangular.  The last bin may
// use its own factors (Ql, Rl, ml).
template <typename K>
__global__ __launch_bounds__(kThreads) void resample_kernel(const K* __restrict__ sorted, int64_t n_points,
                                                            int64_t ppb, int nc, const double* __restrict__ Q,
                                                            const double* __restrict__ Rm, const double* __restrict__ Ql,
                                                            const double* __restrict__ Rl, double* __restrict__ coef)
{
    __shared__ double part[kThreads / 64][kMaxCoef];
    __shared__ double qd[kMaxCoef];
    const int64_t b = blockIdx.x;
    const int64_t b0 = b * ppb;
    const int64_t m = min(ppb, n_points - b0);
    const bool last = m != ppb;
    const double* q = last ? Ql : Q;
    const double* r = last ? Rl : Rm;
    double acc[kMaxCoef];
#pragma unroll
    for (int c = 0; c < kMaxCoef; ++c) acc[c] = 0.0;
    for (int64_t i = threadIdx.x; i < m; i += kThreads) {
        const double d = log(fmax(key_to_double(sorted, b0 + i), 2.2250738585072014e-308));
        const double* qi = q + i * nc;
#pragma unroll
        for (int c = 0; c < kMaxCoef; ++c)
            if (c < nc) acc[c] = fma(qi[c], d, acc[c]);
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < kMaxCoef; ++c) {
        double v = acc[c];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (lane == 0) part[wave][c] = v;
    }
    __syncthreads();
    if ((int)threadIdx.x < nc) {
        double v = 0.0;
        for (int w = 0; w < kThreads / 64; ++w) v += part[w][threadIdx.x];
        qd[threadIdx.x] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {  // back substitution R C = Q^T d
        double x[kMaxCoef];
        for (int c = nc - 1; c >= 0; --c) {
            double s = qd[c];
            for (int k = c + 1; k < nc; ++k) s -= r[c * nc + k] * x[k];
            x[c] = s / r[c * nc + c];
        }
        for (int c = 0; c < nc; ++c) coef[b * nc + c] = x[c];
    }
}

// ---- Q^T d on the matrix cores ----
//
// Sixteen bins form a group: their Q^T d is the product of Q^T (32 x M, two
// tiles of 16 coefficients) and the 16 columns d, by v_mfma_f64_16x16x4.  A
// workgroup takes kChunkRows rows of one group, kWaveRows per wavefront; the
// partial products of its wavefronts are added in LDS and its sum goes to
// part; resample_solve_kernel adds a bin's parts in chunk order and solves.
// Bound: the logarithms (one per point) and reading the bins once; Q (1.6 MB
// for bins of 1e4 points, 20 coefficients) is read once per group from L2.
// One workgroup per bin with a dot product per coefficient read Q once per
// bin and solved the triangle with one lane: 300 bins of 1e4 points took 229
// us, 37 us (27 + 10) now.
constexpr int64_t kMfmaRows = 512;  // bins from this size (smaller ones: a workgroup per bin)
constexpr int kWaveRows = 64, kChunkRows = kWaveRows * kThreads / 64;
constexpr int kGroupBins = 16;
typedef double doublex4 __attribute__((ext_vector_type(4)));

// The bins of one size: n_bins of m rows from `sorted` on, ppb points apart,
// their factors and their coefficients.
template <typename K>
struct BinSet {
    const K* sorted;
    int64_t n_bins, m;
    const double *Q, *R;
    double* coef;
};

// Group blockIdx.x (of the whole bins, or the last, shorter bin's own), chunk
// blockIdx.y; part: [group][chunk][32 coefficients][16 bins].
template <typename K>
__global__ __launch_bounds__(kThreads) void resample_product_kernel(BinSet<K> whole, BinSet<K> last, int64_t groups,
                                                                    int64_t ppb, int nc, double* __restrict__ part)
{
    __shared__ double sum[kThreads / 64][32 * kGroupBins];
    const bool is_last = blockIdx.x >= groups;
    const BinSet<K>& B = is_last ? last : whole;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 15, kk = lane >> 4;
    const int64_t bin = (is_last ? 0 : (int64_t)blockIdx.x * kGroupBins) + col;
    const bool have = bin < B.n_bins;
    const K* __restrict__ d = B.sorted + (have ? bin : 0) * ppb;
    const double* __restrict__ Q = B.Q;
    const bool two = nc > 16;
    const int64_t r0 = (int64_t)blockIdx.y * kChunkRows + wave * kWaveRows;
    const int64_t r1 = min(r0 + kWaveRows, B.m);
    doublex4 c0 = {0.0, 0.0, 0.0, 0.0}, c1 = {0.0, 0.0, 0.0, 0.0};
    // 16 rows at a time, the next 16 loaded while these are taken; lane (col,
    // kk) takes rows 4 kk .. 4 kk + 3 of its bin's column and of Q's (any
    // order of the rows will do, as long as both operands have the same)
    double v[4], q0[4], q1[4], vn[4], q0n[4], q1n[4];
    auto load = [&](int64_t r, double (&a)[4], double (&x)[4], double (&y)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t i = r + 4 * kk + e;
            const bool in = i < r1;
            a[e] = in && have ? key_to_double(d, i) : 1.0;
            x[e] = in && col < nc ? Q[i * nc + col] : 0.0;
            y[e] = two && in && col + 16 < nc ? Q[i * nc + col + 16] : 0.0;
        }
    };
    load(r0, v, q0, q1);
    for (int64_t r = r0; r < r1; r += 16) {
        load(r + 16, vn, q0n, q1n);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double lv = log(fmax(v[e], 2.2250738585072014e-308));
            c0 = __builtin_amdgcn_mfma_f64_16x16x4f64(q0[e], lv, c0, 0, 0, 0);
            if (two) c1 = __builtin_amdgcn_mfma_f64_16x16x4f64(q1[e], lv, c1, 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = vn[e];
            q0[e] = q0n[e];
            q1[e] = q1n[e];
        }
    }
    // lane (col, kk) holds coefficients kk + 4 e of bin col
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        sum[wave][(kk + 4 * e) * kGroupBins + col] = c0[e];
        sum[wave][(16 + kk + 4 * e) * kGroupBins + col] = c1[e];
    }
    __syncthreads();
    double* out = part + ((int64_t)blockIdx.x * gridDim.y + blockIdx.y) * 32 * kGroupBins;
    for (int t = threadIdx.x; t < 32 * kGroupBins; t += kThreads) {
        double w = 0.0;
#pragma unroll
        for (int k = 0; k < kThreads / 64; ++k) w += sum[k][t];
        out[t] = w;
    }
}

// R C = Q^T d, a wavefront per bin (the last, shorter bin in a workgroup of
// its own, past `blocks`): lane c adds its coefficient's parts in chunk order;
// then back substitution by columns, lane c holding row c's right-hand side.
template <typename K>
__global__ __launch_bounds__(kThreads) void resample_solve_kernel(BinSet<K> whole, BinSet<K> last, int64_t blocks,
                                                                  int64_t groups, int chunks, int nc,
                                                                  const double* __restrict__ part)
{
    __shared__ double R[kMaxCoef * kMaxCoef];
    const bool is_last = blockIdx.x >= blocks;
    const BinSet<K>& B = is_last ? last : whole;
    for (int t = threadIdx.x; t < nc * nc; t += kThreads) R[t] = B.R[t];
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t bin = (is_last ? 0 : (int64_t)blockIdx.x * (kThreads / 64)) + wave;
    if (bin >= B.n_bins) return;
    const int c = min(lane, nc - 1);
    const int n_parts = (int)((B.m + kChunkRows - 1) / kChunkRows);  // the other chunks of a shorter bin are empty
    const double* p = part + ((is_last ? groups : bin / kGroupBins) * chunks * 32 + c) * kGroupBins + bin % kGroupBins;
    double s = 0.0;
#pragma unroll 8
    for (int k = 0; k < n_parts; ++k) s += p[(int64_t)k * 32 * kGroupBins];
    double x = 0.0;
    for (int k = nc - 1; k >= 0; --k) {
        const double xk = __shfl(s, k, 64) / R[k * nc + k];
        if (lane == k) x = xk;
        if (lane < k) s = fma(-R[lane * nc + k], xk, s);
    }
    if (lane < nc) B.coef[bin * nc + lane] = x;
}

// ---- the factors of the design matrix ----
//
// Cholesky QR: A^T A = R^T R, Q = A R^-1.  For M >= 512 the columns T_c on the
// equispaced t_i are close to orthogonal (condition number at most 7.01, for 32
// coefficients), so forming A^T A loses at most a factor 50; it, its Cholesky
// factor, the inverse and Q's sums are taken in pairs of binary64 numbers
// (106 bits), so that Q and R are A's factors rounded once.  Below 512 points
// the condition number rises (it is unbounded as M nears the number of
// coefficients).  A's rows are formed where they are needed.  Bound: the
// serial chain of the Cholesky factor and the launches.  Bins of 1e4 points,
// 20 coefficients: 9 ms on the host, column by column, now 67 us (48 of them the Cholesky
// factor).
constexpr int kQrTile = 64, kQrMaxChunks = 256;
constexpr int kQrThreads = kMaxCoef * kMaxCoef;
static_assert(kMaxCoef == 32 && kQrThreads == 1024, "a thread per pair of coefficients");

// A sum h + l of two binary64 numbers, |l| <= half an ulp of h (Dekker 1971,
// Knuth's two-sum; products by FMA).
struct Pair {
    double h, l;
};
__device__ inline Pair fast_pair(double a, double b)
{
    const double s = a + b;
    return {s, b - (s - a)};
}
__device__ inline Pair add(Pair a, Pair b)
{
    const double s = a.h + b.h, v = s - a.h;
    return fast_pair(s, ((a.h - (s - v)) + (b.h - v)) + (a.l + b.l));
}
__device__ inline Pair mul(Pair a, Pair b)
{
    const double p = a.h * b.h;
    return fast_pair(p, fma(a.h, b.h, -p) + fma(a.h, b.l, a.l * b.h));
}
__device__ inline Pair neg(Pair a) { return {-a.h, -a.l}; }
__device__ inline Pair div(Pair a, Pair b)
{
    const double q = a.h / b.h;
    const Pair r = add(a, neg(mul({q, 0.0}, b)));
    return fast_pair(q, r.h / b.h);
}
__device__ inline Pair root(Pair a)
{
    const double q = sqrt(a.h);
    const Pair r = add(a, neg(mul({q, 0.0}, {q, 0.0})));
    return fast_pair(q, r.h / (2.0 * q));
}

// Rows [r0, r0 + kQrTile) of A (0 from r1 on) into a; all threads take part.
__device__ inline void design_rows(int64_t r0, int64_t r1, int64_t m, int nc, double (*a)[kMaxCoef + 1])
{
    if (threadIdx.x < kQrTile) {
        const int64_t i = r0 + threadIdx.x;
        double* row = a[threadIdx.x];
        const bool in = i < r1;
        const double t = 2.0 * ((double)i + 0.5) / (double)m - 1.0;
        double tm = in ? 1.0 : 0.0, tc = in ? t : 0.0;
        for (int c = 0; c < nc; ++c) {
            row[c] = tm;
            const double tn = 2.0 * t * tc - tm;
            tm = tc;
            tc = tn;
        }
    }
    __syncthreads();
}

// part[chunk][a][b] = sum over the chunk's rows of A_a A_b
__global__ __launch_bounds__(kQrThreads) void gram_kernel(int64_t m, int nc, int64_t rows, Pair* __restrict__ part)
{
    __shared__ double a[kQrTile][kMaxCoef + 1];
    const int i = threadIdx.x / kMaxCoef, j = threadIdx.x % kMaxCoef;
    const int64_t r1 = min(m, (int64_t)(blockIdx.x + 1) * rows);
    Pair acc = {0.0, 0.0};
    for (int64_t r0 = (int64_t)blockIdx.x * rows; r0 < r1; r0 += kQrTile) {
        design_rows(r0, r1, m, nc, a);
        if (i < nc && j < nc) {
#pragma unroll 4
            for (int r = 0; r < kQrTile; ++r) acc = add(acc, mul({a[r][i], 0.0}, {a[r][j], 0.0}));
        }
        __syncthreads();
    }
    part[(int64_t)blockIdx.x * kQrThreads + threadIdx.x] = acc;
}

// One workgroup: R (nc columns, rounded), the Cholesky factor of the summed
// parts, and W = R^-1 (kMaxCoef columns).
__global__ __launch_bounds__(kQrThreads) void cholesky_kernel(const Pair* __restrict__ part, int chunks, int nc,
                                                              Pair* __restrict__ W, double* __restrict__ R)
{
    __shared__ Pair g[kMaxCoef][kMaxCoef + 1], f[kMaxCoef][kMaxCoef + 1], x[kMaxCoef][kMaxCoef + 1];
    const int i = threadIdx.x / kMaxCoef, j = threadIdx.x % kMaxCoef;
    Pair s = {0.0, 0.0};
#pragma unroll 4
    for (int k = 0; k < chunks; ++k) s = add(s, part[(int64_t)k * kQrThreads + threadIdx.x]);
    g[i][j] = s;
    f[i][j] = x[i][j] = {0.0, 0.0};
    __syncthreads();
    for (int k = 0; k < nc; ++k) {
        if (i == k && j >= k && j < nc) f[k][j] = div(g[k][j], root(g[k][k]));
        __syncthreads();
        if (i > k && j >= i && j < nc) g[i][j] = add(g[i][j], neg(mul(f[k][i], f[k][j])));
        __syncthreads();
    }
    // row p of F^-1 from the rows below it, a thread per column:
    // x_pc = (1_pc - sum_k f_pk x_kc) / f_pp
    for (int p = nc - 1; p >= 0; --p) {
        if (i == 0 && j >= p && j < nc) {
            Pair v = {j == p ? 1.0 : 0.0, 0.0};
            for (int k = p + 1; k <= j; ++k) v = add(v, neg(mul(f[p][k], x[k][j])));
            x[p][j] = div(v, f[p][p]);
        }
        __syncthreads();
    }
    W[threadIdx.x] = x[i][j];
    if (i < nc && j < nc) R[i * nc + j] = f[i][j].h;
}

__global__ __launch_bounds__(kQrThreads) void design_q_kernel(int64_t m, int nc, const Pair* __restrict__ W,
                                                              double* __restrict__ Q)
{
    __shared__ Pair w[kMaxCoef][kMaxCoef + 1];
    __shared__ double a[kQrTile][kMaxCoef + 1];
    w[threadIdx.x / kMaxCoef][threadIdx.x % kMaxCoef] = W[threadIdx.x];
    // (tiles in turn: a grid of one each would pass 2^32 threads from 2^28 rows)
    for (int64_t r0 = (int64_t)blockIdx.x * kQrTile; r0 < m; r0 += (int64_t)gridDim.x * kQrTile) {
        const int64_t n = min((int64_t)kQrTile, m - r0) * nc;
        design_rows(r0, m, m, nc, a);
        for (int e = threadIdx.x; e < n; e += kQrThreads) {
            const int r = e / nc, c = e % nc;
            Pair s = {0.0, 0.0};
            for (int k = 0; k <= c; ++k) s = add(s, mul({a[r][k], 0.0}, w[k][c]));
            Q[r0 * nc + e] = s.h;
        }
        __syncthreads();
    }
}

// ---- transmission ----

// e^{-t} for 0 <= t <= kExpMost (there 0): t = -n ln 2 - r, |r| <= ln 2 / 2, e^r
// by the polynomial through the function at Chebyshev nodes (within 2e-17).  18
// instructions; the library's exp, for any argument, 22.
constexpr double kExpMost = 800.0;
__device__ inline double exp_neg(double t)
{
    const double n = rint(t * -1.4426950408889634);
    const double r = fma(n, -7.371002565167799e-13, fma(n, -0.6931471805592082, -t));
    double p = fma(2.5110049204818658e-08, r, 2.763265472252779e-07);
    p = fma(p, r, 2.755724088722987e-06);
    p = fma(p, r, 2.4801485441561313e-05);
    p = fma(p, r, 0.00019841269890076403);
    p = fma(p, r, 0.0013888888952352863);
    p = fma(p, r, 0.008333333333319589);
    p = fma(p, r, 0.04166666666648795);
    p = fma(p, r, 0.1666666666666668);
    p = fma(p, r, 0.5000000000000019);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return ldexp(p, (int)n);
}
// e^{-t} is exactly 0 in binary64 above kExpZero and rounds to 1 below
// kExpOne.
constexpr double kExpZero = 746.0, kExpOne = 5.5511151231257827e-17;  // 2^-54
constexpr double kHuge = 1.7976931348623157e308;

// T(m_j) = sum_q w_q exp(-exp(P(t_q)) m_j), P the bin's Chebyshev sum, at the
// quadrature nodes y_q (t_q = 2 y_q - 1).  A wavefront per bin and 64 column
// masses: the nodes' exp(P) a node per lane, kept in LDS, then a mass per lane.
// kStep nodes whose exponentials are all 0, or all 1, for every lane need none
// of them: on column masses over many decades most are. (300 bins x 1000
// masses: 23 us, 44 with a workgroup per bin and the library's exp throughout;
// 1e5 bins x 10 masses 415 and 500.)
constexpr int kStep = 4;
__global__ __launch_bounds__(kThreads) void transmission_fit_kernel(const double* __restrict__ coef, int64_t n_bins,
                                                                    int nc, const double* __restrict__ yq,
                                                                    const double* __restrict__ wq, int nq,
                                                                    const double* __restrict__ mcol, int n_m,
                                                                    double* __restrict__ T)
{
    __shared__ double2 node[kThreads / 64][kMaxQuad];  // exp(P(t_q)), w_q
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t b = (int64_t)blockIdx.x * (kThreads / 64) + wave;
    if (b >= n_bins) return;
    double2* nd = node[wave];
    const double* c = coef + b * nc;
    const int j = blockIdx.y * 64 + lane;
    const double mj = mcol[min(j, n_m - 1)];
    bool fine = mj >= 0.0 && mj <= kHuge;
    for (int q = lane; q < nq; q += 64) {
        const double t = 2.0 * yq[q] - 1.0;
        double tm = 1.0, tc = t, s = c[0];
        if (nc > 1) s = fma(c[1], t, s);
        for (int k = 2; k < nc; ++k) {
            const double tn = fma(2.0 * t, tc, -tm);
            tm = tc;
            tc = tn;
            s = fma(c[k], tc, s);
        }
        const double v = exp(s);
        nd[q] = make_double2(v, wq[q]);
        fine = fine && v <= kHuge;  // finite (>= 0, an exponential), not NaN
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    double s = 0.0;
    if (!__ballot(!fine)) {
        int q = 0;
        for (; q + kStep <= nq; q += kStep) {  // independent chains
            double t[kStep], w[kStep], e[kStep];
#pragma unroll
            for (int u = 0; u < kStep; ++u) {
                const double2 n = nd[q + u];
                t[u] = fmin(n.x * mj, kExpMost);
                w[u] = n.y;
            }
            double lo = t[0], hi = t[0];
#pragma unroll
            for (int u = 1; u < kStep; ++u) {
                lo = fmin(lo, t[u]);
                hi = fmax(hi, t[u]);
            }
            if (!__ballot(lo < kExpZero)) continue;
            if (__ballot(hi >= kExpOne)) {
#pragma unroll
                for (int u = 0; u < kStep; ++u) e[u] = exp_neg(t[u]);
#pragma unroll
                for (int u = 0; u < kStep; ++u) s = fma(w[u], e[u], s);
            } else {
#pragma unroll
                for (int u = 0; u < kStep; ++u) s += w[u];
            }
        }
        for (; q < nq; ++q) s = fma(nd[q].y, exp_neg(fmin(nd[q].x * mj, kExpMost)), s);
    } else {
        for (int q = 0; q < nq; ++q) s = fma(nd[q].y, exp(-nd[q].x * mj), s);
    }
    if (j < n_m) T[b * n_m + j] = s;
}

// T(m_j) = (1/M) sum_i exp(-kappa_i m_j) over a bin's values, by two kernels.
//
// Bins of up to kShortBin values, and of up to kMidBin where there are at least
// 4 m^2 outputs for m values: a thread per bin and mass, over all outputs in
// turn, so that lanes stay full whatever the counts are.  Bound: the
// exponentials.  (Against the kernel below, whose wavefronts take 64 values of
// a bin each: 1e6 bins of 1 x 10 masses 30 / 3700 us, 15625 of 64 x 200 133 /
// 640, 3000 of 100 x 300 62 / 156, 1560 of 192 x 300 69 / 94, 1170 of 256 x 300
// 70 / 75.  Fewer outputs leave a thread's chain of m exponentials bare: 656 of
// 100 x 100 12.6 / 19.3, but 640 of 250 x 106 30 / 19 and 30 of 100 x 100 10.9 /
// 7.4.  A workgroup of 256 masses per bin, with the library's exp: 620, 171,
// 104, 108, 112, 16.6, 38 and 8.9 us.)
constexpr int64_t kShortBin = 64, kMidBin = 256;
template <typename K>
__global__ __launch_bounds__(kThreads) void transmission_short_kernel(const K* __restrict__ sorted, int64_t n_points,
                                                                      int ppb, uint32_t n_out,
                                                                      const double* __restrict__ mcol, uint32_t n_m,
                                                                      double* __restrict__ T)
{
    const uint32_t o = blockIdx.x * kThreads + threadIdx.x;
    if (o >= n_out) return;
    const uint32_t b = o / n_m, j = o - b * n_m;
    const K* __restrict__ k = sorted + (int64_t)b * ppb;
    const int m = (int)min((int64_t)ppb, n_points - (int64_t)b * ppb);
    const double mj = mcol[j];
    double s = 0.0;
    int i = 0;
    for (; i + 4 <= m; i += 4) {  // four independent chains
        double t[4], c[4], e[4];
        uint64_t other = 0;  // lanes with a negative t, or NaN
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            t[u] = key_to_double(k, i + u) * mj;
            c[u] = fmin(t[u], kExpMost);
            other |= __ballot(!(t[u] >= 0.0));
        }
        if (!other) {
#pragma unroll
            for (int u = 0; u < 4; ++u) e[u] = exp_neg(c[u]);
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) e[u] = exp(-t[u]);
        }
        s += (e[0] + e[1]) + (e[2] + e[3]);
    }
    for (; i < m; ++i) {
        const double t = key_to_double(k, i) * mj, c = fmin(t, kExpMost);
        s += __ballot(!(t >= 0.0)) ? exp(-t) : exp_neg(c);
    }
    T[o] = s / (double)m;
}

// Longer bins: block (bin, 64 column masses, segment of the bin), a mass per
// lane; its wavefronts take the segment's values 64 at a time in turn, each
// finding the least and the largest of its 64.  Where those and the wavefront's
// own least and largest mass put all of the 64 values' exponentials at 0, or at
// 1, none is evaluated.  The wavefronts' sums are added in LDS in order; with
// more than one segment (few bins and masses would leave the chip idle) the
// segments' go to part and are added by transmission_sum_kernel.  Bound: the
// VALU work of the exponentials left.  (100 bins of 1e4 x 500 masses over 48
// decades: 680 us with a mass per thread over the whole bin and the library's
// exp throughout, 230 us; 3 bins of 2.7e4 x 37 masses 1790 -> 29 us.)
constexpr int kDirectWaves = 8;
template <typename K>
__global__ __launch_bounds__(64 * kDirectWaves) void transmission_direct_kernel(const K* __restrict__ sorted,
                                                                                int64_t n_points, int64_t ppb,
                                                                                const double* __restrict__ mcol,
                                                                                int n_m, double* __restrict__ part,
                                                                                double* __restrict__ T)
{
    __shared__ double kb[kDirectWaves][64], sums[kDirectWaves][64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t b = blockIdx.x;
    const int j = blockIdx.y * 64 + lane;
    const int64_t b0 = b * ppb;
    const int64_t m = min(ppb, n_points - b0);
    const double mj = mcol[min(j, n_m - 1)];
    double mlo = mj, mhi = mj;
    const bool fine_m = !__ballot(!(mj >= 0.0 && mj <= kHuge));
    for (int o = 32; o > 0; o >>= 1) {
        mlo = fmin(mlo, __shfl_xor(mlo, o, 64));
        mhi = fmax(mhi, __shfl_xor(mhi, o, 64));
    }
    double s = 0.0;
    const int64_t step = 64ll * kDirectWaves * gridDim.z;
    for (int64_t i0 = 64ll * ((int64_t)blockIdx.z * kDirectWaves + wave); i0 < m; i0 += step) {
        const int64_t i = i0 + lane;
        const int cnt = (int)min((int64_t)64, m - i0);
        const double v = i < m ? key_to_double(sorted, b0 + i) : 0.0;
        const bool fine = !__ballot(!(v >= 0.0 && v <= kHuge));
        double vlo = i < m ? v : kHuge, vhi = v;
        for (int o = 32; o > 0; o >>= 1) {
            vlo = fmin(vlo, __shfl_xor(vlo, o, 64));
            vhi = fmax(vhi, __shfl_xor(vhi, o, 64));
        }
        double* k64 = kb[wave];
        k64[lane] = v;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (!fine_m || !fine) {
            for (int k = 0; k < cnt; ++k) s += exp(-k64[k] * mj);
        } else if (vlo * mlo > kExpZero) {
            // all 0
        } else if (vhi * mhi < kExpOne) {
            s += (double)cnt;
        } else {
            int k = 0;
            for (; k + 4 <= cnt; k += 4) {  // four independent chains
                double e[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) e[u] = exp_neg(fmin(k64[k + u] * mj, kExpMost));
                s += (e[0] + e[1]) + (e[2] + e[3]);
            }
            for (; k < cnt; ++k) s += exp_neg(fmin(k64[k] * mj, kExpMost));
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    sums[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && j < n_m) {
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < kDirectWaves; ++w) v += sums[w][lane];
        if (gridDim.z == 1)
            T[b * n_m + j] = v / (double)m;
        else
            part[((int64_t)blockIdx.z * gridDim.x + b) * n_m + j] = v;
    }
}

// The segments' sums, in order.
__global__ __launch_bounds__(256) void transmission_sum_kernel(const double* __restrict__ part, int segs,
                                                              int64_t n_bins, int64_t n_points, int64_t ppb, int n_m,
                                                              double* __restrict__ T)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= n_bins * n_m) return;
    double v = 0.0;
    for (int k = 0; k < segs; ++k) v += part[k * n_bins * n_m + t];
    const int64_t b = t / n_m;
    T[t] = v / (double)min(ppb, n_points - b * ppb);
}

// Segments of each bin: enough for four wavefronts per SIMD, of at least one
// round of the workgroup's wavefronts each.
int direct_segments(int64_t n_points, int64_t ppb, int n_m)
{
    const int64_t n_bins = (n_points + ppb - 1) / ppb, blocks = n_bins * ((n_m + 63) / 64);
    const int64_t m = std::min(ppb, n_points);
    return (int)std::max<int64_t>(1, std::min<int64_t>(512 / blocks, m / (64 * kDirectWaves)));
}

}  // namespace

namespace {

template <typename K>
hipError_t run_resample(const K* sorted, int64_t n_points, int64_t ppb, int nc, const double* Q, const double* R,
                        const double* Ql, const double* Rl, double* part, double* coef, hipStream_t s)
{
    const int64_t n_bins = (n_points + ppb - 1) / ppb;
    const int64_t m = std::min(ppb, n_points), last = n_points - (n_bins - 1) * ppb;
    if (!part || !resample_scratch_bytes(n_points, ppb)) {
        constexpr int64_t most = (int64_t)1 << 23;  // (a launch holds less than 2^32 threads)
        for (int64_t b = 0; b < n_bins; b += most)
            resample_kernel<K><<<dim3((unsigned)std::min(most, n_bins - b)), dim3(kThreads), 0, s>>>(
                sorted + b * ppb, n_points - b * ppb, ppb, nc, Q, R, Ql, Rl, coef + b * nc);
        return hipGetLastError();
    }
    // the whole bins, and a shorter last one with its own factors
    const int64_t n_whole = last < m ? n_bins - 1 : n_bins, n_last = n_bins - n_whole;
    const BinSet<K> whole{sorted, n_whole, m, Q, R, coef};
    const BinSet<K> short_bin{sorted + n_whole * ppb, n_last, last, Ql, Rl, coef + n_whole * nc};
    const int64_t groups = (n_whole + kGroupBins - 1) / kGroupBins;
    const int64_t chunks = (m + kChunkRows - 1) / kChunkRows;
    if (groups + n_last > (int64_t)INT32_MAX) return hipErrorInvalidValue;
    resample_product_kernel<K><<<dim3((unsigned)(groups + n_last), (unsigned)chunks), dim3(kThreads), 0, s>>>(
        whole, short_bin, groups, ppb, nc, part);
    const int64_t blocks = (n_whole + kThreads / 64 - 1) / (kThreads / 64);
    resample_solve_kernel<K><<<dim3((unsigned)(blocks + n_last)), dim3(kThreads), 0, s>>>(whole, short_bin, blocks,
                                                                                         groups, (int)chunks, nc, part);
    return hipGetLastError();
}

}  // namespace

// (Bins whose rows would need more than 65535 chunks, 1.6e7 points, also go
// one workgroup per bin.)
int64_t design_factor_min_rows() { return kMfmaRows; }

size_t design_factor_scratch_bytes() { return (size_t)(kQrMaxChunks + 1) * kQrThreads * sizeof(Pair); }

hipError_t launch_design_factors(int64_t m, int nc, double* Q, double* R, void* scratch, hipStream_t s)
{
    if (m < kMfmaRows || nc < 1 || nc > kMaxCoef) return hipErrorInvalidValue;
    const int64_t per = (m + kQrMaxChunks - 1) / kQrMaxChunks;
    const int64_t rows = (per + kQrTile - 1) / kQrTile * kQrTile;
    const int chunks = (int)((m + rows - 1) / rows);
    const int64_t tiles = std::min<int64_t>((m + kQrTile - 1) / kQrTile, (int64_t)1 << 16);
    Pair* W = static_cast<Pair*>(scratch);
    Pair* part = W + kQrThreads;
    gram_kernel<<<dim3((unsigned)chunks), dim3(kQrThreads), 0, s>>>(m, nc, rows, part);
    cholesky_kernel<<<dim3(1), dim3(kQrThreads), 0, s>>>(part, chunks, nc, W, R);
    design_q_kernel<<<dim3((unsigned)tiles), dim3(kQrThreads), 0, s>>>(m, nc, W, Q);
    return hipGetLastError();
}

size_t resample_scratch_bytes(int64_t n_points, int64_t ppb)
{
    const int64_t m = std::min(ppb, n_points);
    const int64_t chunks = (m + kChunkRows - 1) / kChunkRows;
    if (m < kMfmaRows || chunks > 65535) return 0;
    const int64_t groups = ((n_points + ppb - 1) / ppb + kGroupBins - 1) / kGroupBins + 1;
    return (size_t)(groups * chunks) * 32 * kGroupBins * sizeof(double);
}

hipError_t launch_resample(const void* sorted, int key_bytes, int64_t n_points, int64_t ppb, int nc,
                           const double* Q, const double* R, const double* Ql, const double* Rl, double* part,
                           double* coef, hipStream_t s)
{
    if (n_points == 0) return hipSuccess;
    if (key_bytes == 8)
        return run_resample(static_cast<const double*>(sorted), n_points, ppb, nc, Q, R, Ql, Rl, part, coef, s);
    return run_resample(static_cast<const float*>(sorted), n_points, ppb, nc, Q, R, Ql, Rl, part, coef, s);
}

hipError_t launch_transmission_fit(const double* coef, int64_t n_bins, int nc, const double* yq, const double* wq,
                                   int nq, const double* m, int n_m, double* T, hipStream_t s)
{
    if (n_bins == 0 || n_m == 0) return hipSuccess;
    constexpr int64_t per_block = kThreads / 64;
    // (a launch holds less than 2^32 threads along its blocks)
    const int64_t most = ((int64_t)1 << 23) * per_block;
    for (int64_t b = 0; b < n_bins; b += most) {
        const int64_t nb = std::min(most, n_bins - b);
        const dim3 grid((unsigned)((nb + per_block - 1) / per_block), (unsigned)((n_m + 63) / 64));
        transmission_fit_kernel<<<grid, dim3(kThreads), 0, s>>>(coef + b * nc, nb, nc, yq, wq, nq, m, n_m,
                                                                T + b * n_m);
    }
    return hipGetLastError();
}

size_t transmission_direct_scratch_bytes(int64_t n_points, int64_t ppb, int n_m)
{
    if (n_points <= 0 || n_m <= 0) return 0;
    const int segs = direct_segments(n_points, ppb, n_m);
    return segs == 1 ? 0 : (size_t)segs * (size_t)((n_points + ppb - 1) / ppb) * (size_t)n_m * sizeof(double);
}

hipError_t launch_transmission_direct(const void* sorted, int key_bytes, int64_t n_points, int64_t ppb,
                                      const double* m, int n_m, double* part, double* T, hipStream_t s)
{
    const int64_t n_bins = (n_points + ppb - 1) / ppb;
    if (n_bins == 0 || n_m == 0) return hipSuccess;
    const int64_t span = std::min(ppb, n_points);
    if (span <= kShortBin || (span <= kMidBin && n_bins * n_m >= 4 * span * span)) {
        // (outputs of a launch counted in 32 bits; less than 2^32 threads)
        const int64_t most = std::max<int64_t>(1, ((int64_t)1 << 30) / n_m);
        for (int64_t b = 0; b < n_bins; b += most) {
            const int64_t n_out = std::min(most, n_bins - b) * n_m, o = b * ppb;
            const dim3 grid((unsigned)((n_out + kThreads - 1) / kThreads));
            if (key_bytes == 8)
                transmission_short_kernel<double><<<grid, dim3(kThreads), 0, s>>>(
                    static_cast<const double*>(sorted) + o, n_points - o, (int)span, (uint32_t)n_out, m, (uint32_t)n_m,
                    T + b * n_m);
            else
                transmission_short_kernel<float><<<grid, dim3(kThreads), 0, s>>>(
                    static_cast<const float*>(sorted) + o, n_points - o, (int)span, (uint32_t)n_out, m, (uint32_t)n_m,
                    T + b * n_m);
        }
        return hipGetLastError();
    }
    const int segs = part ? direct_segments(n_points, ppb, n_m) : 1;
    const dim3 grid((unsigned)n_bins, (unsigned)((n_m + 63) / 64), (unsigned)segs);
    if (key_bytes == 8)
        transmission_direct_kernel<double><<<grid, dim3(64 * kDirectWaves), 0, s>>>(
            static_cast<const double*>(sorted), n_points, ppb, m, n_m, part, T);
    else
        transmission_direct_kernel<float><<<grid, dim3(64 * kDirectWaves), 0, s>>>(static_cast<const float*>(sorted),
                                                                                   n_points, ppb, m, n_m, part, T);
    if (segs > 1)
        transmission_sum_kernel<<<dim3((unsigned)((n_bins * n_m + 255) / 256)), dim3(256), 0, s>>>(
            part, segs, n_bins, n_points, ppb, n_m, T);
    return hipGetLastError();
}

}  // namespace hk
