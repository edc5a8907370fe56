// work_plan.hip -- the work items of the wing kernels (the scheme is stated
// beside WorkPlan in hk_internal.h): the segment length of each state, then
// each (state, tile) pair's segment count and the exclusive prefix sums that
// number the items and the partial slots, in three passes (block sums, one
// scan of the block sums, offsets).
#include <algorithm>

#include "hk_internal.h"

namespace hk {
namespace {

constexpr int kThreads = 256;
constexpr int kPerThread = 4;
constexpr int64_t kPerBlock = (int64_t)kThreads * kPerThread;
// A state's tiles are uneven when the fullest reference tile holds more than
// kUneven times the mean (CutRule).
constexpr int64_t kUneven = 3;

// Segment length of a state from its reference tiles' statistics: the smallest power of two >=
// min_seg and >= W / (4 n_points), W = 512 sum_t c_t + 4096 n_lines (c_t:
// lines of reference tile t).  W bounds the sum over any tiles of <= 2048
// points of (lines in the tile's range) x (tile points): a line's reach
// covers |A| grid points, which lie in >= |A| / 512 reference tiles and meet
// <= |A| / tp + 2 tiles of tp points.  So the items stay <= sum_t (c_t / L
// + 2) <= 6 n_tiles and the partial points <= 6 n_points + 2 tile points.
__device__ inline int64_t seg_length(int64_t busy, int64_t mx, int64_t sum, int64_t n_points, int64_t n_lines,
                                     const PlanJob& j, int32_t st)
{
    const CutRule& c = (j.reach_of ? j.reach_of[st] : j.reach) >= j.wide_reach ? j.wide : j.cut;
    if (!(sum > 0 && mx >= c.lines && (busy < c.busy || mx * busy > kUneven * sum))) return kNoSplit;
    const double W = 512.0 * (double)sum + 4096.0 * (double)n_lines;
    const double need = W / (4.0 * (double)n_points);
    int64_t L = j.min_seg;
    while ((double)L < need && L < kNoSplit) L <<= 1;  // kNoSplit: not cut after all
    return L;
}

// One workgroup per state.
__global__ __launch_bounds__(kThreads) void seg_length_kernel(PlanJob j, int64_t n_points, int64_t n_lines)
{
    __shared__ int64_t red[3][kThreads];
    const int64_t* rg = j.ref + (int64_t)blockIdx.x * 2 * j.n_ref;
    int64_t busy = 0, mx = 0, sum = 0;
    for (int64_t t = threadIdx.x; t < j.n_ref; t += kThreads) {
        const int64_t c = rg[2 * t + 1] - rg[2 * t];
        busy += c > 0;
        mx = max(mx, c);
        sum += c;
    }
    red[0][threadIdx.x] = busy;
    red[1][threadIdx.x] = mx;
    red[2][threadIdx.x] = sum;
    __syncthreads();
    for (int h = kThreads / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            red[0][threadIdx.x] += red[0][threadIdx.x + h];
            red[1][threadIdx.x] = max(red[1][threadIdx.x], red[1][threadIdx.x + h]);
            red[2][threadIdx.x] += red[2][threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0)
        j.seg[blockIdx.x] = seg_length(red[0][0], red[1][0], red[2][0], n_points, n_lines, j, blockIdx.x);
}

__device__ inline void pair_counts(int64_t p, int64_t n_pairs, const int64_t* __restrict__ ranges,
                                   int64_t n_tiles, int32_t n_states, const int64_t* __restrict__ seg,
                                   int64_t& items, int64_t& slots)
{
    items = 0;
    slots = 0;
    if (p >= n_pairs) return;
    int64_t st, k;
    pair_decode(p, n_tiles, n_states, st, k);
    const int64_t t = n_tiles - 1 - k;
    const int64_t* rg = ranges + st * 2 * n_tiles;
    const int64_t lo = rg[2 * t], hi = rg[2 * t + 1];
    const int64_t L = seg[st];
    items = hi > lo ? (hi - 1) / L - lo / L + 1 : 1;
    slots = items > 1 ? items : 0;
}

// Exclusive scan of (a, b) over the workgroup; returns the totals.
__device__ inline void block_scan(int64_t& a, int64_t& b, int64_t& ta, int64_t& tb)
{
    __shared__ int64_t sa[kThreads], sb[kThreads];
    sa[threadIdx.x] = a;
    sb[threadIdx.x] = b;
    __syncthreads();
    for (int o = 1; o < kThreads; o <<= 1) {
        const int64_t va = (int)threadIdx.x >= o ? sa[threadIdx.x - o] : 0;
        const int64_t vb = (int)threadIdx.x >= o ? sb[threadIdx.x - o] : 0;
        __syncthreads();
        sa[threadIdx.x] += va;
        sb[threadIdx.x] += vb;
        __syncthreads();
    }
    ta = sa[kThreads - 1];
    tb = sb[kThreads - 1];
    a = sa[threadIdx.x] - a;
    b = sb[threadIdx.x] - b;
    __syncthreads();
}

// Pass 1: per-pair counts, block-local exclusive prefixes, block totals.
__global__ __launch_bounds__(kThreads) void plan_count_kernel(const int64_t* __restrict__ ranges, int64_t n_tiles,
                                                              int32_t n_states, const int64_t* __restrict__ seg,
                                                              int64_t n_pairs, int64_t* __restrict__ first,
                                                              int64_t* __restrict__ slot,
                                                              int64_t* __restrict__ bsum)
{
    const int64_t p0 = (int64_t)blockIdx.x * kPerBlock + (int64_t)threadIdx.x * kPerThread;
    int64_t it[kPerThread], sl[kPerThread];
    int64_t a = 0, b = 0;
    for (int i = 0; i < kPerThread; ++i) {
        pair_counts(p0 + i, n_pairs, ranges, n_tiles, n_states, seg, it[i], sl[i]);
        a += it[i];
        b += sl[i];
    }
    int64_t ta, tb;
    block_scan(a, b, ta, tb);
    for (int i = 0; i < kPerThread; ++i) {
        if (p0 + i < n_pairs) {
            first[p0 + i] = a;
            slot[p0 + i] = b;
        }
        a += it[i];
        b += sl[i];
    }
    if (threadIdx.x == 0) {
        bsum[2 * blockIdx.x] = ta;
        bsum[2 * blockIdx.x + 1] = tb;
    }
}

// Pass 2 (one workgroup): exclusive scan of the block totals in place, and
// the grand totals.
__global__ __launch_bounds__(kThreads) void plan_scan_kernel(int64_t* __restrict__ bsum, int64_t n_blocks,
                                                             int64_t* __restrict__ total)
{
    int64_t ra = 0, rb = 0;  // running totals of earlier rounds
    for (int64_t base = 0; base < n_blocks; base += kThreads) {
        const int64_t i = base + threadIdx.x;
        int64_t a = i < n_blocks ? bsum[2 * i] : 0;
        int64_t b = i < n_blocks ? bsum[2 * i + 1] : 0;
        int64_t ta, tb;
        block_scan(a, b, ta, tb);
        if (i < n_blocks) {
            bsum[2 * i] = ra + a;
            bsum[2 * i + 1] = rb + b;
        }
        ra += ta;
        rb += tb;
    }
    if (threadIdx.x == 0) {
        total[0] = ra;
        total[1] = rb;
    }
}

// Pass 3: add each block's offset.
__global__ __launch_bounds__(kThreads) void plan_offset_kernel(int64_t n_pairs, const int64_t* __restrict__ bsum,
                                                               int64_t* __restrict__ first,
                                                               int64_t* __restrict__ slot)
{
    const int64_t oa = bsum[2 * blockIdx.x], ob = bsum[2 * blockIdx.x + 1];
    const int64_t p0 = (int64_t)blockIdx.x * kPerBlock;
    for (int64_t i = threadIdx.x; i < kPerBlock; i += kThreads) {
        const int64_t p = p0 + i;
        if (p < n_pairs) {
            first[p] += oa;
            slot[p] += ob;
        }
    }
}

// Both plans of a pass in one launch, a workgroup each (plans of up to
// kSmallPairs pairs): the states' segment lengths (a wavefront per state, in
// turn), then the pairs kSmallThreads at a time with running totals.
constexpr int kSmallThreads = 1024;
constexpr int64_t kSmallPairs = 16384;
struct PlanJobs {
    PlanJob job[2];
};
__global__ __launch_bounds__(kSmallThreads) void plan_small_kernel(PlanJobs jobs, int64_t n_points, int64_t n_lines)
{
    const PlanJob& j = jobs.job[blockIdx.x];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int kW = kSmallThreads / 64;
    __shared__ int64_t wa[kW], wb[kW], part[3][kW];
    // every wavefront a share of a state's reference tiles
    for (int32_t st = 0; st < j.n_states; ++st) {
        const int64_t* rg = j.ref + (int64_t)st * 2 * j.n_ref;
        int64_t busy = 0, mx = 0, sum = 0;
        for (int64_t t = threadIdx.x; t < j.n_ref; t += kSmallThreads) {
            const int64_t c = rg[2 * t + 1] - rg[2 * t];
            busy += c > 0;
            mx = max(mx, c);
            sum += c;
        }
        for (int o = 32; o > 0; o >>= 1) {
            busy += __shfl_xor(busy, o, 64);
            mx = max(mx, (int64_t)__shfl_xor(mx, o, 64));
            sum += __shfl_xor(sum, o, 64);
        }
        if (lane == 0) {
            part[0][wave] = busy;
            part[1][wave] = mx;
            part[2][wave] = sum;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            busy = mx = sum = 0;
            for (int w = 0; w < kW; ++w) {
                busy += part[0][w];
                mx = max(mx, part[1][w]);
                sum += part[2][w];
            }
            j.seg[st] = seg_length(busy, mx, sum, n_points, n_lines, j, st);
        }
        __syncthreads();
    }
    const int64_t n_pairs = j.n_tiles * j.n_states;
    int64_t ra = 0, rb = 0;  // totals of the pairs before
    for (int64_t base = 0; base < n_pairs; base += kSmallThreads) {
        const int64_t p = base + threadIdx.x;
        int64_t it, sl;
        pair_counts(p, n_pairs, j.ranges, j.n_tiles, j.n_states, j.seg, it, sl);
        int64_t ia = it, ib = sl;
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t va = __shfl_up(ia, o, 64), vb = __shfl_up(ib, o, 64);
            if (lane >= o) {
                ia += va;
                ib += vb;
            }
        }
        if (lane == 63) {
            wa[wave] = ia;
            wb[wave] = ib;
        }
        __syncthreads();
        int64_t oa = ra, ob = rb;
        for (int w = 0; w < kW; ++w) {
            if (w < wave) {
                oa += wa[w];
                ob += wb[w];
            }
            ra += wa[w];
            rb += wb[w];
        }
        if (p < n_pairs) {
            j.first[p] = oa + ia - it;
            j.slot[p] = ob + ib - sl;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        j.total[0] = ra;
        j.total[1] = rb;
    }
}

}  // namespace

int64_t plan_scratch_count(int64_t n_pairs) { return 2 * std::max<int64_t>(1, (n_pairs + kPerBlock - 1) / kPerBlock); }

hipError_t launch_work_plans(const PlanJob* jobs, int n_jobs, int64_t n_points, int64_t n_lines, hipStream_t s)
{
    if (n_jobs < 1 || n_jobs > 2) return hipErrorInvalidValue;
    // One workgroup per plan walks its states in turn, then its pairs 1024 at a
    // time: 7 us for one state of 40 pairs, 18 for 2930, 30 for 5860, 41 for 16
    // states of 40, against 28 us in eight launches (14 a plan of 17 states) and
    // the gaps between them.
    bool small = true;
    for (int k = 0; k < n_jobs; ++k) {
        const PlanJob& j = jobs[k];
        if (j.min_seg < 1 || (j.min_seg & (j.min_seg - 1)) != 0) return hipErrorInvalidValue;
        if (j.n_states <= 0) return hipSuccess;
        small = small && j.n_tiles * j.n_states <= kSmallPairs && j.n_ref * j.n_states <= 2 * kSmallPairs &&
                j.n_states <= 16;
    }
    if (small) {
        PlanJobs pj;
        for (int k = 0; k < n_jobs; ++k) pj.job[k] = jobs[k];
        plan_small_kernel<<<dim3((unsigned)n_jobs), dim3(kSmallThreads), 0, s>>>(pj, n_points, n_lines);
        return hipGetLastError();
    }
    for (int k = 0; k < n_jobs; ++k) {
        const PlanJob& j = jobs[k];
        const int64_t n_pairs = j.n_tiles * (int64_t)j.n_states;
        const int64_t nb = std::max<int64_t>(1, (n_pairs + kPerBlock - 1) / kPerBlock);
        seg_length_kernel<<<dim3((unsigned)j.n_states), dim3(kThreads), 0, s>>>(j, n_points, n_lines);
        plan_count_kernel<<<dim3((unsigned)nb), dim3(kThreads), 0, s>>>(j.ranges, j.n_tiles, j.n_states, j.seg, n_pairs,
                                                                        j.first, j.slot, j.bsum);
        plan_scan_kernel<<<dim3(1), dim3(kThreads), 0, s>>>(j.bsum, nb, j.total);
        plan_offset_kernel<<<dim3((unsigned)nb), dim3(kThreads), 0, s>>>(n_pairs, j.bsum, j.first, j.slot);
    }
    return hipGetLastError();
}

}  // namespace hk
