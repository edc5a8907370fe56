// opacity_f64.hip -- the "kappa(nu)" stage in binary64 (§2.4, §2.5).
//
// The paper's GPU scheme is a serial loop over lines with the grid spread
// over threads, kappa held in a register (§2.5).  Here a workgroup owns a
// block of consecutive grid points and the lines (sorted by wavenumber) that
// reach it.
//
// Two kernels per call:
//  wing: the 3-node and 1-node Gauss-Hermite rules (a^2+u^2 >= 100) for
//        every line and point; it writes kappa (over the work items of
//        work_plan.hip: a block, or the part of its lines in one segment,
//        whose partial sums a reduction adds in segment order).  Most lines
//        are far from most blocks and smooth there, and are evaluated at a
//        few nodes per tile instead of at every point.
//  core: the series for a^2+u^2 < 100, a few hundred times rarer but ~30
//        times dearer per point and heavy in registers; it writes its own
//        ordered sums into a grid of their own (so the two kernels can run
//        at the same time, on two streams), added to kappa afterwards.
// So kappa_j = sum_wing + sum_core, each in an order fixed by the lines and
// the grid alone, without atomics: reproducible bit for bit.
#include <algorithm>
#include <cmath>

#include "hk_internal.h"

namespace hk {
namespace {

constexpr int kWaves = 4;            // wavefronts per workgroup
constexpr int kMaxTerms = 32;  // series terms: n = 1 .. 2 x + 12, x < 10
constexpr int kTermStride = kMaxTerms + 2;  // between tables in LDS (other banks)
static_assert(kMaxTerms <= 64, "one lane per series term builds the tables");

// num / den to about 2^-48 relative: the hardware reciprocal (relative
// error below 2^-24 on gfx950) and one Newton correction of the quotient,
// which is none where num is infinite.  Callers discard the result (by select)
// wherever den may be 0.
__device__ inline double qdiv(double num, double den)
{
    const double r = __builtin_amdgcn_rcp(den);
    const double q = num * r;
    const double e = fma(-den, q, num);
    return e == e ? fma(e, r, q) : q;
}

// 1 / den to about 2^-48 relative (one Newton step on the reciprocal).
__device__ inline double qrcp(double den)
{
    const double r = __builtin_amdgcn_rcp(den);
    return fma(r, fma(-den, r, 1.0), r);
}

// Work items run dearest tile first (high wavenumber: wider Doppler cores,
// more 3-node points), so cheap tiles fill the launch's tail, and are dealt
// to the 8 XCDs (each with its own L2) in chunks of consecutive tiles
// (xcd_rank), so an XCD's neighbouring tiles, which read mostly the same
// lines, share its L2 while every XCD gets a mix of dear and cheap chunks.

// ---- the wing: far lines at Chebyshev nodes, near lines point by point ----
//
// A line's wing over a tile of points that it covers whole, on one rule and
// far enough away, is smooth there: its value at every point of the tile
// follows from its values at kFarNodes Chebyshev nodes of the tile.  So such
// a line is evaluated at the nodes only, the nodes' sums over all such lines
// are kept per tile, and one polynomial per tile gives the sums at its
// points.  The tiles form three levels (a work item's block of 4 kSub points,
// its four wavefronts' kSub, their four kLeaf) or, with kSub = kLeaf, two; a
// line is taken at the largest tile that admits it (a tile inside an admitting
// one admits the line too), and point by point only in the leaves that do not:
// those near its centre, or where its window, or its boundary between the
// two rules or with the series, ends inside the leaf.  Items of few lines are
// taken point by point throughout.
//
// The error of interpolating 1/(x - p) at the roots of T_N is
// T_N(x)/T_N(p) of the value, pointwise.  The rules' poles (nu0 -+ i Gamma_L,
// and for the 3-node rule nu0 -+ sqrt(3/2) alpha -+ i Gamma_L) lie at least
// kFarRatio half-widths of the tile from its centre, where
// |1/T_24| <= 2 (3 + sqrt 8)^-24 = 8.5e-19; a Lorentzian is a difference of
// two such terms over Gamma_L, which costs a factor up to ~1.5 N: below
// 4e-17 of each line's value in every case.
//
// Bound: VALU (binary64; 81% of its cycles busy).  On 1e6 lines x 3e6 points
// with 2e4 points per window a line costs ~1000 node evaluations and ~500
// point evaluations in place of 2e4, and the kernel alone takes 1.22 ms
// against 6.9 ms with every line at every point; 3e6 lines x 1e6 points with
// 5e3 points per window 2.6 against 9.7 ms, 1e5 lines x 4e5 points 0.16
// against 0.49 ms.  More than 128 registers cost a wavefront per SIMD: what is
// added here is checked against that (131: 3e6 lines x 1e6 points 3590 -> 3690
// us a step, in 128 with spills).
constexpr int kFarNodes = kWingNodes;  // 24
constexpr int kFarRatio = 3;
constexpr int kLeaf = 64;
static_assert(kFarNodes == 24, "far_eval and wave_reduce are written for 24 nodes");
// Lines of a work item up to which all of them are taken point by point, in
// blocks of 1024 and of 256 points: there a block's fixed cost (clearing and
// reducing the node sums, the interpolation) is more than the points'.  (Steps
// with 24 lines, through the leaves' lists / with 48, a run of 256 points at a
// time: 1e4 lines x 3e6 points 182 / 130 us, 10 x 1e7 without a cutoff 356 /
// 192, 24 x 1e7 477 / 242; with 64 lines 64 x 1e7 330 / 391.  Blocks of 256:
// tables of 300 states of 300 lines x 6e4 points 2130 / 1616 us; with 96 lines
// in place of 64 1e3 x 6e4 2424 / 2344, with 192 1e4 x 3e5 74 / 91.)
constexpr int kFewLines = 48, kFewLinesSmall = 96;
// Lists whose centres lie on up to this many grid points take blocks of 256
// points (two levels of tiles): a quarter of the serial work per wavefront,
// four times the workgroups; wider lists fill the chip with blocks of 1024,
// which take far lines at fewer nodes.  (500 lines x 6e3 points: 16 us in
// blocks of 256, 47 in blocks of 1024; 1e5 lines x 4e5 points 0.20 against
// 0.26 ms; whole steps of 1.2e5 lines x 6e5 points 255 against 248 us, 1.25e5
// x 1e6 283 / 239, 8 times 1.25e5 lines on an eighth each of 1e6 points 2.8 /
// 4.0 ms; 1e6 lines x 3e6 points 2.1 / 1.4 ms.)
constexpr int64_t kSmallGrid = 400000;
// (a thread per point of the blocks, up to 6 items a block: 2^32 threads are
// more than a launch holds)
constexpr int64_t kSmallTiles = (int64_t)1 << 29;
// Entries of a wavefront's list of lines that its sub-tile does not admit.
constexpr int kNearCap = 768;
// A rest of up to this many lines of a leaf's is taken with a point per lane:
// ~27 issue slots a line, against ~1900 for a batch of a line per lane.
constexpr int kFewDirect = 48;
// Marks a ring's entry (a line's offset from lo, below 2^31) as 3-node.
constexpr uint32_t kThree = 0x80000000u;
// Points of a leaf evaluated at a time.
constexpr int kPoints = 16;

// cos((2k + 1) pi / 48), k = 0 .. 11; node 23 - k is the negative of node k
constexpr double kNode[kFarNodes / 2] = {
    0.99785892323860348, 0.98078528040323043, 0.94693012949510569, 0.89687274153268826,
    0.83146961230254524, 0.75183980747897738, 0.65934581510006884, 0.55557023301960218,
    0.44228869021900125, 0.32143946530316159, 0.19509032201612828, 0.065403129230143055};

// 1 / den to full precision: the hardware reciprocal (relative error e below
// 2^-24) times 1 + e + e^2.
__device__ inline double qrcp3(double den)
{
    const double r = __builtin_amdgcn_rcp(den);
    const double e = fma(-den, r, 1.0);
    return fma(r, fma(e, e, e), r);
}

// 3-node rule of one point, S Phi = Lg n / m (WingRec): six operations.
__device__ inline void gh3_nm(double dv, double X, double a2, double c, double p, double r, double& n, double& m)
{
    const double x = fma(dv, dv, X);
    n = fma(x, fma(0.5, a2, x), c);
    m = fma(fma(x, x, p), x, r);
}

// How a line meets the tile of W points from t0 (t1: its last point on the
// grid).  touches: its window does.  far: the tile admits it at its nodes --
// the window covers the tile, one rule serves all of it (three: the 3-node
// rule) and no series point lies in it, the poles are kFarRatio half-widths
// from its centre (in whole points: jc is the grid point nearest nu0, the
// slack sqrt(3/2) alpha in points, rounded up, plus one), and the products
// of four denominators stay in range.  Each condition holds for every tile
// inside one for which it holds, in these integers exactly.
struct Meets {
    bool touches, far, three;
};
__device__ inline Meets meets(const WingIdx& r, int32_t t0, int32_t t1, int32_t W, bool far_ok)
{
    Meets m;
    m.touches = t0 <= t1 && r.whi >= t0 && r.wlo <= t1;
    const bool full = r.wlo <= t0 && r.whi >= t1;
    const bool nocore = t1 < r.clo || t0 > r.chi;
    const bool out3 = t1 < r.g3lo || t0 > r.g3hi;  // wholly 1-node
    m.three = r.g3lo <= t0 && r.g3hi >= t1;        // wholly 3-node
    const bool away = abs(t0 + W / 2 - r.jc) >= kFarRatio * (W / 2) + (r.flags >> kSlackShift);
    m.far = m.touches && full && nocore && (out3 || m.three) && away && far_ok && (r.flags & kGroupSafe);
    return m;
}

// acc[k] += the line (one per lane) at the nodes dvc + h kNode[k] (dvc: the
// tile's centre less nu0).  Lanes without a line have Lg = 0.  The 3-node
// rule's coefficients are those of WingRec, from G2 and alpha^2; with
// alpha^2 = 0 it is the 1-node rule, so lanes of both rules share a call (a
// path of its own for 1-node lines made the compiler hold the sums twice: 208
// registers).  Four nodes share one reciprocal (the binary64 reciprocal issues at a quarter of
// the FMA rate): with P01 = d_0 d_1, P23 = d_2 d_3, c = Lg / (P01 P23),
// Lg/d_0 = (c P23) d_1 and so on.
__device__ __forceinline__ void far_eval(double (&acc)[kFarNodes], double dvc, double h, double Lg, double G2,
                                         double a2)
{
    const double X = G2 - a2, cc = a2 * fma(4.0, G2, a2), p = a2 * fma(6.0, G2, -0.75 * a2);
    const double r = a2 * a2 * fma(6.0, G2, 0.25 * a2);
#pragma unroll
    for (int g = 0; g < kFarNodes / 4; ++g) {
        double nn[4], mm[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double t = (e & 2) ? -kNode[2 * g + (e & 1)] : kNode[2 * g + (e & 1)];
            gh3_nm(fma(t, h, dvc), X, a2, cc, p, r, nn[e], mm[e]);
        }
        const double P01 = mm[0] * mm[1], P23 = mm[2] * mm[3];
        const double c = qrcp3(P01 * P23);
        const double c01 = (c * P23) * Lg, c23 = (c * P01) * Lg;
        acc[2 * g] = fma(c01 * mm[1], nn[0], acc[2 * g]);
        acc[2 * g + 1] = fma(c01 * mm[0], nn[1], acc[2 * g + 1]);
        acc[23 - 2 * g] = fma(c23 * mm[3], nn[2], acc[23 - 2 * g]);
        acc[22 - 2 * g] = fma(c23 * mm[2], nn[3], acc[22 - 2 * g]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// x and y with the upper half of x and the lower half of y exchanged (kHalf
// 32: 32-lane halves; 16: odd and even rows of 16), added.
template <int kHalf>
__device__ inline double swap_add(double x, double y)
{
    const uint64_t a = (uint64_t)__double_as_longlong(x), b = (uint64_t)__double_as_longlong(y);
    u32x2 lo, hi;
    if constexpr (kHalf == 32) {
        lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
        hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    } else {
        lo = __builtin_amdgcn_permlane16_swap((uint32_t)a, (uint32_t)b, false, false);
        hi = __builtin_amdgcn_permlane16_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    }
    const double p = __longlong_as_double((long long)(((uint64_t)hi.x << 32) | lo.x));
    const double q = __longlong_as_double((long long)(((uint64_t)hi.y << 32) | lo.y));
    return p + q;
}

// v plus v rotated by kRor lanes within each row of 16.
template <int kRor>
__device__ inline double row_add(double v)
{
    const uint64_t a = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)a, 0x120 | kRor, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(a >> 32), 0x120 | kRor, 0xf, 0xf, false);
    return v + __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Adds a row's (16 lanes') values; every lane of the row holds the sum.
__device__ inline double row_sum(double v) { return row_add<1>(row_add<2>(row_add<4>(row_add<8>(v)))); }

// dst[k] += the wavefront's sum of acc[k].  Two halving steps leave
// row r of 16 lanes with the partial sums of nodes 6 r .. 6 r + 5.
__device__ __forceinline__ void wave_reduce(double (&acc)[kFarNodes], double* dst, int lane)
{
    double a[12], b[6];
#pragma unroll
    for (int i = 0; i < 12; ++i) a[i] = swap_add<32>(acc[i], acc[i + 12]);
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        b[i] = row_sum(swap_add<16>(a[i], a[i + 6]));
    }
    if ((lane & 15) == 0) {
        double* d = dst + 6 * (lane >> 4);
#pragma unroll
        for (int i = 0; i < 6; ++i) d[i] += b[i];
    }
}

__device__ inline void clear(double (&acc)[kFarNodes])
{
#pragma unroll
    for (int i = 0; i < kFarNodes; ++i) acc[i] = 0.0;
}

// A value that every lane holds alike, in scalar registers.
__device__ inline uint64_t uniform_bits(uint64_t a)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
    return ((uint64_t)hi << 32) | lo;
}
__device__ inline double uniform(double v)
{
    return __longlong_as_double((long long)uniform_bits((uint64_t)__double_as_longlong(v)));
}

// The points of the closed index interval [lo, hi] (empty: lo > hi) among the
// kPoints from q0, or the kLeaf from q0, as bits.
__device__ inline uint32_t point_bits(int32_t lo, int32_t hi, int32_t q0)
{
    const int32_t a = max(lo, q0), b = min(hi, q0 + kPoints - 1);
    return a > b ? 0u : (0xffffffffu >> (31 - (b - a))) << (a - q0);
}
__device__ inline uint64_t leaf_bits(int32_t lo, int32_t hi, int32_t q0)
{
    const int32_t a = max(lo, q0), b = min(hi, q0 + kLeaf - 1);
    return a > b ? 0ull : (~0ull >> (63 - (b - a))) << (a - q0);
}

__device__ inline uint64_t readlane64(uint64_t v, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

// dacc += four lines at this lane's point x of a leaf: line e's record by
// uniform (scalar) loads, take[e] the points that its window holds outside
// the series, one[e] the points of the 1-node rule (uniform masks over the
// leaf's points).  Points not taken have numerator 0 and denominator 1.
__device__ __forceinline__ double direct_four(const WingRec* const (&r)[4], const uint64_t (&take)[4],
                                              const uint64_t (&one)[4], double x, double dacc)
{
    double num[4], den[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const bool tk = __builtin_amdgcn_inverse_ballot_w64(take[e]);
        const bool on = __builtin_amdgcn_inverse_ballot_w64(one[e]);
        const double dv = x - r[e]->nu0;
        double n, m;
        gh3_nm(dv, r[e]->X, r[e]->a2, r[e]->c, r[e]->p, r[e]->r, n, m);
        m = on ? fma(dv, dv, r[e]->G2) : m;
        n = (on ? 1.0 : n) * r[e]->Lg;
        num[e] = tk ? n : 0.0;
        den[e] = tk ? m : 1.0;
    }
    const double P01 = den[0] * den[1], P23 = den[2] * den[3];
    const double c = qrcp3(P01 * P23);
    const double c01 = c * P23, c23 = c * P01;
    dacc = fma(c01 * den[1], num[0], dacc);
    dacc = fma(c01 * den[0], num[1], dacc);
    dacc = fma(c23 * den[3], num[2], dacc);
    return fma(c23 * den[2], num[3], dacc);
}

// v where m is all ones, 0 where it is 0.
__device__ inline double masked(double v, int32_t m)
{
    return __longlong_as_double(__double_as_longlong(v) & (int64_t)m);
}
// v where m is all ones, a value in [1, 2) where it is 0 (v's low word under
// the exponent of 1).
__device__ inline double one_to_two(double v, int32_t m)
{
    const uint64_t a = (uint64_t)__double_as_longlong(v);
    const uint32_t hi = ((uint32_t)(a >> 32) & (uint32_t)m) | (0x3ff00000u & ~(uint32_t)m);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | (uint32_t)a));
}

// acc[p] += the line (one per lane) at points x[p] of a leaf where bit p of
// tk is set (its window holds the point outside the series); bit p of on:
// the 1-node rule, else the 3-node rule.  Points not taken have numerator 0
// and a denominator of about 1 (a series point's may be 0 or negative).  kOne, kGh3: some lane takes points of that rule.
// Four points share one reciprocal, as at the nodes.
template <bool kOne, bool kGh3>
__device__ __forceinline__ void point_eval(double (&acc)[kPoints], const double (&x)[kPoints], uint32_t tk,
                                           uint32_t on, const WingRec& l)
{
#pragma unroll
    for (int g = 0; g < kPoints; g += 4) {
        double num[4], den[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int p = g + e;
            const int32_t take = (int32_t)(tk << (31 - p)) >> 31;  // all ones where the point is taken
            const double dv = x[p] - l.nu0;
            double nn, dd;
            if constexpr (kGh3) gh3_nm(dv, l.X, l.a2, l.c, l.p, l.r, nn, dd);
            if constexpr (kOne) {
                const bool one = !kGh3 || ((on >> p) & 1u);
                dd = one ? fma(dv, dv, l.G2) : dd;
                nn = one ? 1.0 : nn;
            }
            num[e] = masked(nn, take);
            den[e] = one_to_two(dd, take);
        }
        const double P01 = den[0] * den[1], P23 = den[2] * den[3];
        const double c = qrcp3(P01 * P23) * l.Lg;
        const double c01 = c * P23, c23 = c * P01;
        acc[g] = fma(c01 * den[1], num[0], acc[g]);
        acc[g + 1] = fma(c01 * den[0], num[1], acc[g + 1]);
        acc[g + 2] = fma(c23 * den[3], num[2], acc[g + 2]);
        acc[g + 3] = fma(c23 * den[2], num[3], acc[g + 3]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The same with a division per point, for lines outside the grouping range.
__device__ __forceinline__ void point_eval_single(double (&acc)[kPoints], const double (&x)[kPoints], uint32_t tk,
                                                  uint32_t on, const WingRec& l)
{
#pragma unroll
    for (int p = 0; p < kPoints; ++p) {
        const double dv = x[p] - l.nu0;
        double nn, mm;
        gh3_nm(dv, l.X, l.a2, l.c, l.p, l.r, nn, mm);
        const bool one = (on >> p) & 1u;
        const double v = qdiv(l.Lg * (one ? 1.0 : nn), one ? fma(dv, dv, l.G2) : mm);
        acc[p] += (tk >> p) & 1u ? v : 0.0;
    }
}

// The node sums of one work item: of the block per wavefront (summed at the
// end), of each sub-tile and of each leaf, then each leaf's polynomial.
template <int kSub>
struct WingLds {
    double block[kWaves][kFarNodes], sub[kWaves][kFarNodes];
    double leaf[kWaves * kSub / kLeaf][kFarNodes], coef[kWaves * kSub / kLeaf][kFarNodes];
    double point[kWaves][kSub];        // the lines taken point by point
    uint32_t near[kWaves][kNearCap];   // lines (offsets from lo) the sub-tile does not admit
    uint16_t direct[kWaves][kNearCap]; // of those, the ones the current leaf does not admit either
    uint32_t queue[kWaves][2][128];    // rings of lines (with kThree) for the nodes of the sub-tile, of a leaf
    uint64_t done[kWaves];             // bit b: batch 4 b + wave needs nothing below the block
};

__device__ inline void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// acc[e] += the line at this lane's points x[e] (index j0 + 64 e): a run of 256
// points, four a lane, that share one reciprocal.  The line's window, rules and
// series intervals are the same for the wavefront.
__device__ __forceinline__ void run_eval(double (&acc)[4], const double (&x)[4], int32_t run0, int32_t j0,
                                         const WingIdx& w, const WingRec& l)
{
    const int32_t run1 = run0 + 255;
    const bool inside = w.wlo <= run0 && w.whi >= run1 && (run1 < w.clo || run0 > w.chi);
    const bool out3 = run1 < w.g3lo || run0 > w.g3hi;
    double num[4], den[4];
    if (inside && out3 && (w.flags & kGroupSafe)) {  // the window covers the run, on the 1-node rule
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double dv = x[e] - l.nu0;
            num[e] = 1.0;
            den[e] = fma(dv, dv, l.G2);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int32_t j = j0 + 64 * e;
            const bool take = j >= w.wlo && j <= w.whi && !(j >= w.clo && j <= w.chi);
            const bool one = j < w.g3lo || j > w.g3hi;
            const double dv = x[e] - l.nu0;
            double nn, mm;
            gh3_nm(dv, l.X, l.a2, l.c, l.p, l.r, nn, mm);
            mm = one ? fma(dv, dv, l.G2) : mm;
            nn = one ? 1.0 : nn;
            if (!(w.flags & kGroupSafe)) {
                const double v = qdiv(l.Lg * nn, mm);
                acc[e] += take ? v : 0.0;
            }
            num[e] = take ? nn : 0.0;
            den[e] = take ? mm : 1.0;
        }
        if (!(w.flags & kGroupSafe)) return;
    }
    const double P01 = den[0] * den[1], P23 = den[2] * den[3];
    const double c = qrcp3(P01 * P23) * l.Lg;
    const double c01 = c * P23, c23 = c * P01;
    acc[0] = fma(c01 * den[1], num[0], acc[0]);
    acc[1] = fma(c01 * den[0], num[1], acc[1]);
    acc[2] = fma(c23 * den[3], num[2], acc[2]);
    acc[3] = fma(c23 * den[2], num[3], acc[3]);
}

// The run's sums over every kStep-th of the nl lines from the first on.
template <int kStep>
__device__ __forceinline__ void run_lines(double (&acc)[4], int32_t first, int32_t nl, int32_t run0, double nu_min,
                                          double dnu, const WingRec* __restrict__ wing,
                                          const WingIdx* __restrict__ idx)
{
    const int32_t j0 = run0 + (int32_t)(threadIdx.x & 63);
    double x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        x[e] = fma((double)(j0 + 64 * e), dnu, nu_min);
        acc[e] = 0.0;
    }
    if (first >= nl) return;
    WingIdx w = idx[first];
    WingRec l = wing[first];
    for (int32_t i = first; i < nl; i += kStep) {
        // (the next line's records on their way meanwhile)
        const int32_t next = min(i + kStep, nl - 1);
        const WingIdx wn = idx[next];
        const WingRec ln = wing[next];
        if (w.whi >= run0 && w.wlo <= run0 + 255) run_eval(acc, x, run0, j0, w, l);
        w = wn;
        l = ln;
    }
}

// Lines [L0, L1) at the points of block t of one state (record pointers
// already offset to the state): out[j - obase] = the sum, or += it with
// accumulate.  Each wavefront takes every fourth batch of 64 lines (one per
// lane) for the block's nodes, then walks all batches for its own sub-tile:
// admitted lines go through a ring to full 64-lane evaluations, the others
// to a list that is walked once per leaf in the same way, and lines that a
// leaf does not admit are evaluated at its points.  A lane holds one line
// throughout, so the records are read by coalesced vector loads; its sums
// are added across the wavefront at the end.  The order of every sum is
// fixed by (L0, L1) and the lines alone.
template <int kSub>
__device__ __forceinline__ void wing_f64_tile(int64_t t, int64_t L0, int64_t L1, const WingRec* __restrict__ wing,
                                              const WingIdx* __restrict__ idx, const WingTables* __restrict__ tab,
                                              double nu_min, double dnu, int32_t n, double* __restrict__ out,
                                              int64_t obase, int accumulate, bool far_ok)
{
    constexpr int kBlock = kWaves * kSub, kLeaves = kSub / kLeaf;  // leaves per wavefront
    constexpr bool kThreeLevels = kLeaves > 1;
    static_assert(kLeaves == 1 || kLeaves == 4, "tiles have four children each");
    __shared__ WingLds<kSub> S;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int32_t b0 = (int32_t)(t * kBlock);
    const int32_t s0 = b0 + wave * kSub;
    const int32_t b1 = min(b0 + kBlock, n) - 1, s1 = min(s0 + kSub, n) - 1;
    const double xref = fma((double)b0, dnu, nu_min);  // positions are taken relative to the block's first point
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    wing += L0;
    idx += L0;
    const int32_t nl = (int32_t)(L1 - L0);
    if (nl <= (kThreeLevels ? kFewLines : kFewLinesSmall)) {
        double acc[4];
        if constexpr (kThreeLevels) {  // each wavefront its points
            run_lines<1>(acc, 0, nl, s0, nu_min, dnu, wing, idx);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int32_t j = s0 + 64 * e + lane;
                if (j < n) out[j - obase] = accumulate ? out[j - obase] + acc[e] : acc[e];
            }
        } else {  // each wavefront every fourth line at all points
            double* part = reinterpret_cast<double*>(&S.near[0][0]);
            run_lines<kWaves>(acc, wave, nl, b0, nu_min, dnu, wing, idx);
#pragma unroll
            for (int e = 0; e < 4; ++e) part[wave * kBlock + 64 * e + lane] = acc[e];
            __syncthreads();
            const int32_t j = b0 + (int32_t)threadIdx.x;
            if (j < n) {
                double v = 0.0;
#pragma unroll
                for (int q = 0; q < kWaves; ++q) v += part[q * kBlock + threadIdx.x];
                out[j - obase] = accumulate ? out[j - obase] + v : v;
            }
        }
        return;
    }

    for (int k = threadIdx.x; k < kWaves * kFarNodes; k += 64 * kWaves) (&S.sub[0][0])[k] = (&S.block[0][0])[k] = 0.0;
    for (int k = threadIdx.x; k < kLeaves * kWaves * kFarNodes; k += 64 * kWaves) (&S.leaf[0][0])[k] = 0.0;
    for (int k = threadIdx.x; k < kBlock; k += 64 * kWaves) (&S.point[0][0])[k] = 0.0;
    __syncthreads();

    // ---- the block's nodes ----
    const double hs = 0.5 * (double)kSub * dnu, hl = 0.5 * (double)kLeaf * dnu, hb = 0.5 * (double)kBlock * dnu;
    if (far_ok) {
        double acc[kFarNodes];
        clear(acc);
        bool any_block = false;
        uint64_t done = 0;  // (of the first 64 batches: longer items test the others twice)
        for (int32_t base = 64 * wave, b = 0; base < nl; base += 64 * kWaves, ++b) {
            const int32_t i = base + lane;
            bool far = false, three = false, rest = false;
            if (i < nl) {
                const Meets m = meets(idx[i], b0, b1, kBlock, true);
                far = m.far;
                three = m.far && m.three;
                rest = m.touches && !m.far;
            }
            if (b < 64 && !__ballot(rest)) done |= 1ull << b;
            if (!__ballot(far)) continue;
            any_block = true;
            double dvc = 1.0, Lg = 0.0, G2 = 1.0, a2 = 0.0;
            if (far) {
                const WingRec& r = wing[i];
                dvc = (xref - r.nu0) + hb;
                Lg = r.Lg;
                G2 = r.G2;
                a2 = three ? r.a2 : 0.0;
            }
            far_eval(acc, dvc, hb, Lg, G2, a2);
        }
        if (any_block) wave_reduce(acc, S.block[wave], lane);
        if (lane == 0) S.done[wave] = done;
        __syncthreads();
    }

    // ---- the sub-tile ----
    if (s0 <= s1) {
        uint32_t* near = S.near[wave];
        uint32_t* qs = S.queue[wave][0];
        uint32_t* ql = S.queue[wave][1];
        uint16_t* dir = S.direct[wave];
        const double cs = (double)(wave * kSub + kSub / 2) * dnu;  // the sub-tile's centre from xref
        int n_near = 0, q_head = 0, q_n = 0;
        double acc[kFarNodes];  // of the sub-tile's nodes
        clear(acc);
        uint64_t done[kWaves] = {};
        if (far_ok) {
#pragma unroll
            for (int w = 0; w < kWaves; ++w) done[w] = uniform_bits(S.done[w]);
        }
        for (int32_t base = 0, b = 0;; base += 64, ++b) {
            const bool last = base >= nl;
            if (!last && b < 64 * kWaves) {
                const uint64_t dn = (b & 3) == 0 ? done[0] : (b & 3) == 1 ? done[1] : (b & 3) == 2 ? done[2] : done[3];
                if ((dn >> (b >> 2)) & 1) continue;
            }
            if (!last) {
                const int32_t i = base + lane;
                bool far = false, keep = false, three = false;
                if (i < nl) {
                    const WingIdx r = idx[i];
                    const Meets m = meets(r, s0, s1, kSub, far_ok);
                    const bool up = meets(r, b0, b1, kBlock, far_ok).far;
                    far = kThreeLevels && m.far && !up;
                    three = m.three;
                    keep = m.touches && !far && !up;
                }
                const uint64_t fm = __ballot(far), km = __ballot(keep);
                if (far) qs[(q_head + q_n + __builtin_popcountll(fm & below)) & 127] = (uint32_t)i | (three ? kThree : 0u);
                if (keep) near[n_near + __builtin_popcountll(km & below)] = (uint32_t)i;
                q_n += __builtin_popcountll(fm);
                n_near += __builtin_popcountll(km);
                wave_fence();
            }
            while (q_n >= (last ? 1 : 64)) {  // full batches; what is left at the end
                double dvc = 1.0, Lg = 0.0, G2 = 1.0, a2 = 0.0;
                if (lane < q_n) {
                    const uint32_t e = qs[(q_head + lane) & 127];
                    const WingRec& r = wing[e & ~kThree];
                    dvc = (xref - r.nu0) + cs;
                    Lg = r.Lg;
                    G2 = r.G2;
                    a2 = (e & kThree) ? r.a2 : 0.0;
                }
                far_eval(acc, dvc, hs, Lg, G2, a2);
                const int done = min(q_n, 64);
                q_head = (q_head + done) & 127;
                q_n -= done;
            }
            if (n_near > kNearCap - 64 || (last && n_near > 0)) {
                // the list is full, or complete: walk it once per leaf
                if constexpr (kThreeLevels) wave_reduce(acc, S.sub[wave], lane);
                for (int lf = 0; lf < kLeaves; ++lf) {
                    const int32_t l0 = s0 + lf * kLeaf, l1 = min(l0 + kLeaf, n) - 1;
                    if (l0 > l1) break;
                    const double cl = (double)(l0 - b0 + kLeaf / 2) * dnu;
                    int h_l = 0, n_l = 0, n_d = 0;
                    bool any_leaf = false;
                    double la[kFarNodes];
                    clear(la);
                    for (int k = 0;; k += 64) {
                        const bool lastk = k >= n_near;
                        if (!lastk) {
                            bool far = false, direct = false, three = false;
                            uint32_t i = 0;
                            if (k + lane < n_near) {
                                i = near[k + lane];
                                const WingIdx w = idx[i];
                                const Meets m = meets(w, l0, l1, kLeaf, far_ok);
                                far = m.far;
                                three = m.three;
                                // (a leaf wholly inside the series is the series kernel's)
                                direct = m.touches && !m.far && !(w.clo <= l0 && w.chi >= l1);
                            }
                            const uint64_t fm = __ballot(far), dm = __ballot(direct);
                            if (far) ql[(h_l + n_l + __builtin_popcountll(fm & below)) & 127] = i | (three ? kThree : 0u);
                            if (direct) dir[n_d + __builtin_popcountll(dm & below)] = (uint16_t)(k + lane);
                            n_l += __builtin_popcountll(fm);
                            n_d += __builtin_popcountll(dm);
                            wave_fence();
                        }
                        while (n_l >= (lastk ? 1 : 64)) {
                            double dvc = 1.0, Lg = 0.0, G2 = 1.0, a2 = 0.0;
                            if (lane < n_l) {
                                const uint32_t e = ql[(h_l + lane) & 127];
                                const WingRec& r = wing[e & ~kThree];
                                dvc = (xref - r.nu0) + cl;
                                Lg = r.Lg;
                                G2 = r.G2;
                                a2 = (e & kThree) ? r.a2 : 0.0;
                            }
                            far_eval(la, dvc, hl, Lg, G2, a2);
                            any_leaf = true;
                            const int done = min(n_l, 64);
                            h_l = (h_l + done) & 127;
                            n_l -= done;
                        }
                        if (lastk) break;
                    }
                    if (any_leaf) wave_reduce(la, S.leaf[wave * kLeaves + lf], lane);
                    // the others point by point: whole batches of 64 with a
                    // line per lane, kPoints points at a time, and a rest of
                    // up to kFewDirect with a point per lane, four lines at a
                    // time (a batch costs the same whatever its lanes hold)
                    const int rest = n_d & 63;
                    const int n_few = rest <= kFewDirect ? rest : 0;
                    const int n_batch = n_d - n_few;
                    if (n_few) {
                        const double x = fma((double)(l0 + lane), dnu, nu_min);
                        double dacc = 0.0;
                        uint32_t i = 0;
                        uint64_t take = 0, one = 0;
                        bool safe = true;
                        if (lane < n_few) {
                            i = near[dir[n_batch + lane]];
                            const WingIdx w = idx[i];
                            take = leaf_bits(w.wlo, w.whi, l0) & ~leaf_bits(w.clo, w.chi, l0);
                            one = ~leaf_bits(w.g3lo, w.g3hi, l0);
                            safe = (w.flags & kGroupSafe) != 0;
                        }
                        for (uint64_t m = __ballot(take != 0 && safe); m;) {
                            const WingRec* r4[4];
                            uint64_t t4[4], o4[4];
                            const int e0 = (int)__builtin_ctzll(m);
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const int at = m ? (int)__builtin_ctzll(m) : e0;
                                r4[e] = wing + (uint32_t)__builtin_amdgcn_readlane((int)i, at);
                                t4[e] = m ? readlane64(take, at) : 0ull;
                                o4[e] = readlane64(one, at);
                                m &= m - 1;
                            }
                            dacc = direct_four(r4, t4, o4, x, dacc);
                        }
                        for (uint64_t m = __ballot(take != 0 && !safe); m; m &= m - 1) {
                            const int at = (int)__builtin_ctzll(m);
                            const WingRec* r = wing + (uint32_t)__builtin_amdgcn_readlane((int)i, at);
                            const bool tk = __builtin_amdgcn_inverse_ballot_w64(readlane64(take, at));
                            const bool on = __builtin_amdgcn_inverse_ballot_w64(readlane64(one, at));
                            const double dv = x - r->nu0;
                            double nn, mm;
                            gh3_nm(dv, r->X, r->a2, r->c, r->p, r->r, nn, mm);
                            const double v = qdiv(r->Lg * (on ? 1.0 : nn), on ? fma(dv, dv, r->G2) : mm);
                            dacc += tk ? v : 0.0;
                        }
                        S.point[wave][lf * kLeaf + lane] += dacc;
                        wave_fence();  // (other lanes add to these below)
                    }
                    for (int p0 = 0; n_batch > 0 && p0 < kLeaf; p0 += kPoints) {
                        double x[kPoints], pa[kPoints];
#pragma unroll
                        for (int p = 0; p < kPoints; ++p) {
                            x[p] = uniform(fma((double)(l0 + p0 + p), dnu, nu_min));
                            pa[p] = 0.0;
                        }
                        for (int k = 0; k < n_batch; k += 64) {
                            uint32_t tk = 0, on = 0;
                            bool safe = true;
                            WingRec r = {};
                            if (k + lane < n_batch) {
                                const uint32_t i = near[dir[k + lane]];
                                const WingIdx w = idx[i];
                                const int32_t q0 = l0 + p0;
                                tk = point_bits(w.wlo, w.whi, q0) & ~point_bits(w.clo, w.chi, q0);
                                on = ~point_bits(w.g3lo, w.g3hi, q0);
                                safe = (w.flags & kGroupSafe) != 0;
                                r = wing[i];
                            }
                            if (!__ballot(tk != 0)) continue;
                            const bool any1 = __ballot((tk & on) != 0) != 0, any3 = __ballot((tk & ~on) != 0) != 0;
                            if (__ballot(!safe))
                                point_eval_single(pa, x, tk, on, r);
                            else if (!any1)
                                point_eval<false, true>(pa, x, tk, on, r);
                            else if (!any3)
                                point_eval<true, false>(pa, x, tk, on, r);
                            else
                                point_eval<true, true>(pa, x, tk, on, r);
                        }
                        double* dst = &S.point[wave][lf * kLeaf + p0 + 4 * (lane >> 4)];
                        double h8[8];
#pragma unroll
                        for (int q = 0; q < 8; ++q) h8[q] = swap_add<32>(pa[q], pa[q + 8]);
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const double v = row_sum(swap_add<16>(h8[q], h8[q + 4]));
                            if ((lane & 15) == 0) dst[q] += v;
                        }
                    }
                }
                n_near = 0;
                clear(acc);
            }
            if (last) break;
        }
        if constexpr (kThreeLevels) wave_reduce(acc, S.sub[wave], lane);
    }

    // ---- down the levels, then each leaf's polynomial at its points ----
    wave_fence();
    if (far_ok) {
        __syncthreads();
        // the parent's sums at this wavefront's nodes: the block's (two
        // levels), or the block's interpolated and added to the sub-tile's
        if (lane < kFarNodes) {
            double v = 0.0;
            if constexpr (kThreeLevels) {
                v = S.sub[wave][lane];
#pragma unroll
                for (int m = 0; m < kFarNodes; ++m) {
                    double b = S.block[0][m];
#pragma unroll
                    for (int w = 1; w < kWaves; ++w) b += S.block[w][m];
                    v = fma(tab->child[wave][m][lane], b, v);
                }
            } else {
#pragma unroll
                for (int w = 0; w < kWaves; ++w) v += S.block[w][lane];
            }
            S.sub[wave][lane] = v;
        }
        wave_fence();
        for (int o = lane; o < kLeaves * kFarNodes; o += 64) {  // Chebyshev coefficients of the leaves
            const int lf = o / kFarNodes, k = o % kFarNodes, c = kThreeLevels ? lf : wave;
            double v = 0.0;
#pragma unroll
            for (int m = 0; m < kFarNodes; ++m) v = fma(tab->cheb[m][k], S.leaf[wave * kLeaves + lf][m], v);
#pragma unroll
            for (int m = 0; m < kFarNodes; ++m) v = fma(tab->child_cheb[c][m][k], S.sub[wave][m], v);
            S.coef[wave * kLeaves + lf][k] = v;
        }
        wave_fence();
    }
#pragma unroll
    for (int lf = 0; lf < kLeaves; ++lf) {
        const int32_t j = s0 + lf * kLeaf + lane;
        if (j < n) {
            double v = S.point[wave][lf * kLeaf + lane];
            if (far_ok) {  // Clenshaw's recurrence
                const double x = fma((double)j, dnu, nu_min) - xref;
                const double tt = (x - (double)(wave * kSub + lf * kLeaf + kLeaf / 2) * dnu) / hl;
                const double* c = S.coef[wave * kLeaves + lf];
                double u1 = 0.0, u2 = 0.0;
#pragma unroll
                for (int k = kFarNodes - 1; k >= 1; --k) {
                    const double u = fma(2.0 * tt, u1, c[k] - u2);
                    u2 = u1;
                    u1 = u;
                }
                v += fma(tt, u1, c[0] - u2);
            }
            out[j - obase] = accumulate ? out[j - obase] + v : v;
        }
    }
}

// One workgroup per work item (a block of a state, or its lines in one
// segment), wp.launch_items of them (the plan's item count or its bound:
// workgroups past the last item exit at once).  Per-state arrays lie n_lines
// records, 2 n_tiles ranges and n points apart; a cut item writes its slot of
// partial (kBlock values).
template <int kSub>
__global__ __launch_bounds__(64 * kWaves) void wing_f64_kernel(
    const WingRec* __restrict__ wing, const WingIdx* __restrict__ idx, const int64_t* __restrict__ ranges,
    int64_t n_lines, int64_t n_tiles, int32_t n_states, WorkPlan wp, const WingTables* __restrict__ tab,
    double nu_min, double dnu, int32_t n, double* __restrict__ kappa, double* __restrict__ partial, int accumulate,
    int far_ok)
{
    constexpr int64_t kBlock = kWaves * kSub;
    WorkItem it;
    if (work_item(xcd_rank(blockIdx.x), wp, ranges, n_tiles, n_states, it)) {
        const int64_t o = it.st * n_lines;
        const bool direct = it.slot < 0;
        double* out = direct ? kappa + it.st * (int64_t)n : partial + it.slot * kBlock;
        wing_f64_tile<kSub>(it.tile, it.lo, it.hi, wing + o, idx + o, tab, nu_min, dnu, n, out,
                      direct ? 0 : it.tile * kBlock, direct ? accumulate : 0, far_ok != 0);
    }
}

// H_V(a, u) for a^2 + u^2 < 100 by the series form of the Faddeeva function
// (Abramowitz & Stegun 7.1.29 applied to w(z) = e^{-z^2} erfc(-iz), step
// 1/2), the three exponential series summed in one loop (§2.4):
//   H = e^{-x^2} [erfcx(y) cos 2xy + sin(xy) (sin(xy)/y) / pi]
//     + (y/pi) [ -cos(2xy) e^{-x^2} T1 + (S2 + S3)/2 ],
// x = |u|, y = a, T1 = sum_n e^{-n^2/4}/(n^2/4+y^2) (per line), and
// S2 + S3 = sum_n (e^{-(n/2+x)^2} + e^{-(n/2-x)^2}) / (n^2/4 + y^2)
//         = 2 e^{-x^2} sum_n w_n cosh(n x),  w_n = e^{-n^2/4} / (n^2/4 + y^2),
// so that H = e^{-x^2} [erfcx(y) cos 2xy + sin^2(xy)/(pi y)
//                        + (y/pi) (sum_n w_n cosh(nx) - cos(2xy) T1)].
// The powers of e^x and of e^-x are summed by Horner's rule (at most e^{320},
// x < 10, n <= 32); w[n-1] is the line's table (same y for all its points),
// read from LDS.
// e^{-n^2/4}, n = 1 .. kMaxTerms
__constant__ double kGauss[kMaxTerms] = {
    0.77880078307140488,
    0.36787944117144233,
    0.10539922456186433,
    0.018315638888734179,
    0.0019304541362277093,
    0.00012340980408667956,
    4.7851173921290088e-06,
    1.1253517471925912e-07,
    1.6052280551856116e-09,
    1.3887943864964021e-11,
    7.2877240958196922e-14,
    2.3195228302435696e-16,
    4.4777324417183015e-19,
    5.2428856633634639e-22,
    3.7233631217505106e-25,
    1.6038108905486379e-28,
    4.1900931944943974e-32,
    6.6396771995807348e-36,
    6.3815034480607908e-40,
    3.7200759760208361e-44,
    1.3153258948574645e-48,
    2.8207700884601352e-53,
    3.6690596154291634e-58,
    2.8946403116483003e-63,
    1.3851193699226017e-68,
    4.0200602157433552e-74,
    7.0766981754295491e-80,
    7.5558190197119609e-86,
    4.8931122620973616e-92,
    1.9219477278238491e-98,
    4.5787899692915775e-105,
    6.6162610567094853e-112,
};

// cosh(r) and sinh(r)/r as polynomials in r^2 (interpolated at Chebyshev
// nodes of |r| <= ln 2 / 2, where they are within 2e-17 of the functions).
__device__ inline void cosh_sinh(double u, double& C, double& Sr)
{
    C = fma(fma(fma(fma(fma(2.763265472252779e-07, u, 2.4801485441561313e-05), u, 0.0013888888952352863), u,
                    0.04166666666648795), u, 0.5000000000000019), u, 1.0);
    Sr = fma(fma(fma(fma(fma(2.5110049204818658e-08, u, 2.755724088722987e-06), u, 0.00019841269890076403), u,
                     0.008333333333319589), u, 0.1666666666666668), u, 1.0);
}
// ln 2 and pi as a part whose multiples by up to 2^12 are exact and the rest.
constexpr double kLog2e = 1.4426950408889634, kLn2Hi = 0.6931471805592082, kLn2Lo = 7.371002565167799e-13;
constexpr double kPiHi = 3.141592653589214, kPiLo = 5.792147943243964e-13;

// The series at x in [0, 10], y in [0, 10), for a line's constants: ex =
// erfcx(y), T1, ypi = y / pi and ipy = 1 / (pi y) (0 for y too small to
// matter: sin^2(xy) / (pi y) < x^2 y).  The exponentials and the sine are
// written out for these ranges: every argument is reduced with its rounding
// error (the products x^2 and xy of up to 100 lose up to 7e-15), and since
// only sin^2(xy) and cos(2xy) = 1 - 2 sin^2(xy) occur, xy is reduced by
// multiples of pi and needs neither quadrants nor a cosine.  (The library's
// exp, exp and sincos, with their ranges' tests, took 65 instructions more of
// 298 per evaluation: the kernel alone 1.10 -> 0.91 ms on 1e6 lines x 3e6
// points.  Against 113-bit arithmetic over x in [0, 10), y from 1e-6 to 9.5
// the error is 1.0e-15 rms and 5.4e-15 at most, against 2.3e-15 and 1.0e-14
// with the library's functions of the rounded x^2 and xy.)
__device__ double voigt_core(double x, double y, double ex, double T1, double ypi, double ipy, const double* w)
{
    // E = e^{-x^2}
    const double t = x * x, dt = fma(x, x, -t);
    const double ke = rint(-t * kLog2e);
    const double re = fma(-ke, kLn2Lo, fma(-ke, kLn2Hi, -t)) - dt;
    double C, Sr;
    cosh_sinh(re * re, C, Sr);
    const double E = ldexp(fma(re, Sr, C), (int)ke);
    // X = e^x and e^{-x}
    const double kx = rint(x * kLog2e);
    const double rx = fma(-kx, kLn2Lo, fma(-kx, kLn2Hi, x));
    cosh_sinh(rx * rx, C, Sr);
    const double X = ldexp(fma(rx, Sr, C), (int)kx), Xi = ldexp(fma(-rx, Sr, C), -(int)kx);
    // sc = sum w_n (X^n + X^-n) by Horner's rule: kMaxTerms positive powers
    // for every point (x < 10: the rest are below 5e-19 of the sum; a fixed
    // trip count, the same for every lane) and 13 negative ones, which fall as
    // e^{-n^2/4}; odd and even powers apart, so that four chains run side by
    // side.  w is read a pair of terms at a time.  (2 cosh(n x) by its
    // three-term recurrence took 68 operations in place of 49: the kernel
    // alone 0.91 -> 0.75 ms on 1e6 lines x 3e6 points, 1.90 -> 1.65 ms on 3e6
    // lines x 1e6 points; with one chain each 0.78 and 1.66.)
    static_assert(kMaxTerms == 32, "16 pairs, the last 6 with the negative powers");
    const double2* w2 = reinterpret_cast<const double2*>(w);
    const double X2 = X * X, Xi2 = Xi * Xi;
    double po = w2[15].x, pe = w2[15].y;  // odd and even powers
#pragma unroll
    for (int h = 14; h > 6; --h) {
        const double2 wh = w2[h];
        po = fma(po, X2, wh.x);
        pe = fma(pe, X2, wh.y);
    }
    double no = w2[6].x, ne = w2[5].y;
    po = fma(po, X2, no);
    pe = fma(pe, X2, w2[6].y);
    no = fma(no, Xi2, w2[5].x);
    po = fma(po, X2, w2[5].x);
    pe = fma(pe, X2, ne);
#pragma unroll
    for (int h = 4; h >= 0; --h) {
        const double2 wh = w2[h];
        po = fma(po, X2, wh.x);
        pe = fma(pe, X2, wh.y);
        no = fma(no, Xi2, wh.x);
        ne = fma(ne, Xi2, wh.y);
    }
    const double sc = fma(X, fma(pe, X, po), Xi * fma(ne, Xi, no));
    // s2 = sin^2(xy): r = xy - k pi, |r| <= pi / 2; sin(r)/r interpolated at
    // Chebyshev nodes, within 3e-17
    const double p = x * y, dp = fma(x, y, -p);
    const double k = rint(p * kInvPi);
    const double r = fma(-k, kPiLo, fma(-k, kPiHi, p)) + dp;
    const double u = r * r;
    double f = fma(2.721557241069097e-15, u, -7.64302491979577e-13);
    f = fma(f, u, 1.605894081716932e-10);
    f = fma(f, u, -2.5052106889380507e-08);
    f = fma(f, u, 2.755731921121691e-06);
    f = fma(f, u, -0.00019841269841208603);
    f = fma(f, u, 0.008333333333333186);
    f = fma(f, u, -0.16666666666666666);
    f = fma(f, u, 1.0);
    const double s2 = u * (f * f);
    const double cos2 = fma(-2.0, s2, 1.0);
    return E * fma(ypi, fma(-cos2, T1, 0.5 * sc), fma(ex, cos2, s2 * ipy));
}

// Core-region contributions.  Each wavefront owns a run of kCoreRun
// consecutive points and walks, in line order, the lines whose a^2+u^2 < 100
// points meet its run; a line's such points form one interval (a piece).
// Pieces are packed into 64-lane chunks: the lines are examined kCoreBatch
// at a time, their pieces' points laid end to end, and each chunk takes the
// next 64 of them (at most kChunkPieces pieces per chunk), so lanes stay
// full when pieces are short.  A lane evaluates the series for its point and
// adds it to the run's sums in LDS; lanes of one chunk that share a point
// (two lines covering it) add in line order, piece by piece.  So each point
// still sums its lines in ascending (nu, index) order, with the same values:
// the result does not depend on how pieces fall into chunks.
// Lines [L0, L1) of tile t; direct: series_j = the run's sum (every point,
// 0 where no line reaches); else every point's sum to partial[j - obase].
// The series has a grid of its own, added to the wing's afterwards (the two
// kernels can then run at the same time).
constexpr int kCoreRun = 256;                        // points per wavefront
constexpr int kCoreTilePoints = kCoreRun * kWaves;   // points per work item
constexpr int kCoreBatch = 32;                       // lines examined at once
constexpr int kChunkPieces = 16;                     // pieces per 64-lane chunk

struct alignas(16) CorePiece {  // one line's series points within a run
    double nu0, invA, y, y2, ex, norm, T1, ypi, ipy;
    int32_t a;      // its first grid point
    int32_t start;  // where its points begin in the batch's flattened list
};

__device__ inline int32_t wave_incl_scan(int32_t v, int lane)
{
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
    }
    return v;
}

__device__ __forceinline__ void core_f64_tile(int64_t t, int64_t L0, int64_t L1, const WingRec* __restrict__ wing,
                                              const WingIdx* __restrict__ idx, const CoreRec* __restrict__ core,
                                              double nu_min, double dnu, int32_t n, double* __restrict__ series,
                                              double* __restrict__ partial, int64_t obase, bool direct)
{
    __shared__ double acc_tab[kWaves][kCoreRun];
    __shared__ CorePiece piece_tab[kWaves][kCoreBatch];
    __shared__ __align__(16) double w_tab[kWaves][kChunkPieces * kTermStride];
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    // lane nn < kMaxTerms builds term nn + 1 of each piece's table
    const double g_lane = kGauss[min(lane, kMaxTerms - 1)];
    const double m_lane = 0.5 * (double)(lane + 1);
    const int32_t run0 = (int32_t)(t * kCoreTilePoints) + wave * kCoreRun;
    const int32_t run1 = min(run0 + kCoreRun, n) - 1;
    if (run0 > run1) return;
    double* acc = acc_tab[wave];
    CorePiece* pc = piece_tab[wave];
    double* wt = w_tab[wave];
    for (int q = lane; q < kCoreRun; q += 64) acc[q] = 0.0;
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));

    for (int64_t base = L0; base < L1; base += kCoreBatch) {
        // lanes below kCoreBatch examine one line each
        const int64_t i = base + lane;
        int32_t a = 1, b = 0;
        if (lane < kCoreBatch && i < L1) {
            const WingIdx r = idx[i];
            a = max(max(r.clo, r.wlo), run0);
            b = min(min(r.chi, r.whi), run1);
        }
        const bool has = a <= b;
        const uint64_t m = __ballot(has);
        if (m == 0) continue;
        const int np = __builtin_popcountll(m);
        const int32_t cnt = has ? b - a + 1 : 0;
        const int32_t incl = wave_incl_scan(cnt, lane);
        const int32_t total = __shfl(incl, 63, 64);
        if (has) {
            const CoreRec cr = core[i];
            CorePiece pp;
            pp.nu0 = wing[i].nu0;
            pp.invA = cr.invA;
            pp.y = cr.y;
            pp.y2 = cr.y2;
            pp.ex = cr.ex;
            pp.norm = cr.norm;
            pp.T1 = cr.T1;
            pp.ypi = cr.ypi;
            pp.ipy = cr.ipy;
            pp.a = a;
            pp.start = incl - cnt;
            pc[__builtin_popcountll(m & below)] = pp;
        }
        __builtin_amdgcn_wave_barrier();
        // lane k holds piece k's start (pieces in line order, starts rising)
        const int32_t st_k = lane < np ? pc[lane].start : total;
        int s_lo = 0;  // the piece holding point f0 of the flattened list
        for (int32_t f0 = 0; f0 < total;) {
            // (s_lo, s_end: the same in every lane, kept in scalar registers)
            s_lo = __builtin_amdgcn_readfirstlane(s_lo);
            int s_end = __builtin_popcountll(__ballot(lane < np && st_k < f0 + 64));
            s_end = __builtin_amdgcn_readfirstlane(min(s_end, s_lo + kChunkPieces));
            const int32_t next_start = __builtin_amdgcn_readlane(st_k, min(s_end, 63));
            const int32_t f_end = s_end < np ? min(next_start, f0 + 64) : min(total, f0 + 64);
            // the 1 / (n^2/4 + y^2) e^{-n^2/4} tables of pieces s_lo .. s_end-1
            for (int k = s_lo; k < s_end; ++k) {
                const double y2 = pc[k].y2;
                if (lane < kMaxTerms) wt[(k - s_lo) * kTermStride + lane] = g_lane * qrcp(fma(m_lane, m_lane, y2));
            }
            __builtin_amdgcn_wave_barrier();
            // this lane's point f and its piece
            const int32_t f = f0 + lane;
            const bool act = f < f_end;
            int my = s_lo;
            for (int s = s_lo + 1; s < s_end; ++s) my = __builtin_amdgcn_readlane(st_k, s) <= f ? s : my;
            double v = 0.0;
            int32_t jr = 0;  // the point, relative to run0
            if (act) {
                const CorePiece& pp = pc[my];
                const int32_t j = pp.a + (f - pp.start);
                jr = j - run0;
                const double dv = fma((double)j, dnu, nu_min) - pp.nu0;
                v = pp.norm * voigt_core(fabs(dv) * pp.invA, pp.y, pp.ex, pp.T1, pp.ypi, pp.ipy,
                                         wt + (my - s_lo) * kTermStride);
            }
            // add in line order: one LDS add instruction per piece, whose
            // lanes hold distinct points; a wavefront's LDS operations are
            // carried out in the order they are issued, and the fence keeps
            // the compiler from merging or reordering the pieces' adds
            for (int s = s_lo; s < s_end; ++s) {
                if (act && my == s)
                    __hip_atomic_fetch_add(&acc[jr], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
            s_lo = (s_end < np && f_end >= next_start) ? s_end : s_end - 1;
            f0 = f_end;
        }
        __builtin_amdgcn_wave_barrier();
    }
    __builtin_amdgcn_wave_barrier();
    for (int q = lane; q < kCoreRun; q += 64) {
        const int32_t j = run0 + q;
        if (j <= run1) {
            if (direct)
                series[j] = acc[q];
            else
                partial[j - obase] = acc[q];
        }
    }
}

// One workgroup per work item of the series (the layout of wing_f64_kernel),
// taken in plan order: a series tile reads few lines, so dealing neighbouring
// tiles to one XCD does not pay here (measured: it costs ~5%).
__global__ __launch_bounds__(64 * kWaves) void core_f64_kernel(
    const WingRec* __restrict__ wing, const WingIdx* __restrict__ idx, const CoreRec* __restrict__ core,
    const int64_t* __restrict__ ranges, int64_t n_lines, int64_t n_tiles, int32_t n_states, WorkPlan wp,
    double nu_min, double dnu, int32_t n, double* __restrict__ series, double* __restrict__ partial)
{
    WorkItem it;
    if (work_item(blockIdx.x, wp, ranges, n_tiles, n_states, it)) {
        const int64_t o = it.st * n_lines;
        const bool direct = it.slot < 0;
        core_f64_tile(it.tile, it.lo, it.hi, wing + o, idx + o, core + o, nu_min, dnu, n,
                      series + it.st * (int64_t)n, partial + (direct ? 0 : it.slot * kCoreTilePoints),
                      it.tile * kCoreTilePoints, direct);
    }
}

}  // namespace

int32_t opacity_f64_tile_points(int64_t covered, int64_t n_points)
{
    return kWaves * (covered <= kSmallGrid && n_points <= kSmallTiles ? kLeaf : 4 * kLeaf);
}
int32_t core_f64_tile_points() { return kCoreTilePoints; }

// The interpolation matrices of the wing's tiles, from the closed forms of
// the Chebyshev nodes t_m = cos((2m + 1) pi / (2N)): a function's Chebyshev
// coefficients are c_k = (2 - [k = 0]) / N sum_m f_m T_k(t_m), its value at
// x is sum_k c_k T_k(x); the nodes of child c of four lie at
// (2c - 3)/4 + t/4 of the parent.
void wing_tables(WingTables* out)
{
    constexpr int N = kFarNodes;
    const long double pi = 3.14159265358979323846264338327950288L;
    long double cheb[N][N];  // [m][k]
    for (int m = 0; m < N; ++m)
        for (int k = 0; k < N; ++k) {
            cheb[m][k] = (k == 0 ? 1.0L : 2.0L) / N * std::cos((long double)(k * (2 * m + 1)) * pi / (2 * N));
            out->cheb[m][k] = (double)cheb[m][k];
        }
    for (int c = 0; c < 4; ++c) {
        long double lag[N][N];  // [m][k]: node m's weight at the child's node k
        for (int k = 0; k < N; ++k) {
            const long double t = k < N / 2 ? kNode[k] : -kNode[N - 1 - k];
            const long double x = 0.25L * ((2 * c - 3) + t);
            long double T[N] = {1.0L, x};
            for (int q = 2; q < N; ++q) T[q] = 2.0L * x * T[q - 1] - T[q - 2];
            for (int m = 0; m < N; ++m) {
                long double v = 0.0L;
                for (int q = 0; q < N; ++q) v += cheb[m][q] * T[q];
                lag[m][k] = v;
                out->child[c][m][k] = (double)v;
            }
        }
        for (int m = 0; m < N; ++m)
            for (int k = 0; k < N; ++k) {
                long double v = 0.0L;
                for (int q = 0; q < N; ++q) v += cheb[q][k] * lag[m][q];
                out->child_cheb[c][m][k] = (double)v;
            }
    }
}

hipError_t launch_wing_f64(const WingRec* wing, const WingIdx* idx, const int64_t* ranges, int64_t n_lines,
                           int64_t n_tiles, int32_t n_states, const WorkPlan& wp, const WingTables* tab,
                           double nu_min, double dnu, int32_t n_points, int32_t tile_points, double* kappa,
                           double* partial, int accumulate, hipStream_t s)
{
    if (n_tiles == 0 || n_states == 0) return hipSuccess;
    const int64_t nb = plan_blocks(wp.launch_items);
    if (nb > (int64_t)UINT32_MAX) return hipErrorInvalidValue;
    // far lines are interpolated where the grid points' own rounding (half
    // an ulp of the wavenumber) is below 2^-10 of a leaf's half-width; on
    // finer grids every line is taken point by point
    const double top = std::max(std::fabs(nu_min), std::fabs(nu_min + (double)n_points * dnu));
    const int far_ok = dnu * 281474976710656.0 >= top ? 1 : 0;  // 2^48
    auto kernel = tile_points == kWaves * kLeaf ? wing_f64_kernel<kLeaf> : wing_f64_kernel<4 * kLeaf>;
    kernel<<<dim3((unsigned)nb), dim3(64 * kWaves), 0, s>>>(wing, idx, ranges, n_lines, n_tiles, n_states, wp, tab,
                                                            nu_min, dnu, n_points, kappa, partial, accumulate, far_ok);
    return hipGetLastError();
}

hipError_t launch_core_f64(const WingRec* wing, const WingIdx* idx, const CoreRec* core, const int64_t* ranges,
                           int64_t n_lines, int64_t n_tiles, int32_t n_states, const WorkPlan& wp, double nu_min,
                           double dnu, int32_t n_points, double* series, double* partial, hipStream_t s)
{
    if (n_tiles == 0 || n_states == 0) return hipSuccess;
    const int64_t nb = plan_blocks(wp.launch_items);
    if (nb > (int64_t)UINT32_MAX) return hipErrorInvalidValue;
    core_f64_kernel<<<dim3((unsigned)nb), dim3(64 * kWaves), 0, s>>>(wing, idx, core, ranges, n_lines, n_tiles,
                                                                    n_states, wp, nu_min, dnu, n_points, series,
                                                                    partial);
    return hipGetLastError();
}

namespace {

// The ordered sum of point j's partials, if its tile is cut.
__device__ inline bool cut_sum(const CutTiles& c, int64_t st, int64_t j, int32_t n_states, double& v)
{
    if (c.wp.total[0] == c.wp.n_pairs) return false;  // nothing cut
    const int64_t p = pair_of(st, j / c.tile_points, c.n_tiles, n_states);
    const int64_t nseg = pair_segments(c.wp, p);
    if (nseg < 2) return false;
    const double* src = (const double*)c.partial + c.wp.slot[p] * c.tile_points + j % c.tile_points;
    v = 0.0;
    for (int64_t sg = 0; sg < nseg; ++sg) v += src[sg * c.tile_points];
    return true;
}

// kappa_j = wing_j + series_j (state blockIdx.y).
__global__ __launch_bounds__(256) void f64_finish_kernel(double* __restrict__ kappa, const double* __restrict__ series,
                                                        int64_t n, CutTiles wing, CutTiles core, int accumulate)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    const int64_t st = blockIdx.y, o = st * n + j;
    double v, w;
    if (!cut_sum(wing, st, j, gridDim.y, v)) v = kappa[o];
    else if (accumulate) v = kappa[o] + v;
    if (!cut_sum(core, st, j, gridDim.y, w)) w = series[o];
    kappa[o] = v + w;
}

}  // namespace

hipError_t launch_f64_finish(double* kappa, const double* series, int32_t n_points, int32_t n_states,
                             const CutTiles& wing, const CutTiles& core, int accumulate, hipStream_t s)
{
    if (n_points <= 0 || n_states <= 0) return hipSuccess;
    const int64_t nb = ((int64_t)n_points + 255) / 256;
    f64_finish_kernel<<<dim3((unsigned)nb, (unsigned)n_states), dim3(256), 0, s>>>(kappa, series, n_points, wing, core,
                                                                                   accumulate);
    return hipGetLastError();
}

}  // namespace hk
