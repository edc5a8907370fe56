// kdist.hip -- the "Sort" stage (§2.2, §2.6): per-bin sort of the opacity
// grid, cumulative coordinate g_i = (i+1)/M, and k(g) at the requested g by
// the step or the midpoint-linear rule.
//
// The paper sorts the whole grid at once with bin tags (Thrust, §2.6).  Here
// bins are independent, and keys are the opacities' bit patterns
// (non-negative IEEE values order like their unsigned integer images).  A
// bin of up to kRadixMaxKeys keys is sorted by one workgroup in registers
// and LDS, by a radix sort whose ranking uses wavefront ballots (below); a
// larger bin is cut into chunks, each sorted in that way, then merged eight
// runs at a time in global memory (each key finds its rank in the other seven
// by binary searches; ties keep the earlier run first).
#include <algorithm>

#include "hk_internal.h"

namespace hk {
size_t radix_lds_bytes(int elem_bytes, int64_t keys);
namespace {

template <typename K>
struct KeyMax;
template <>
struct KeyMax<uint64_t> {
    static constexpr uint64_t v = ~0ull;
};
template <>
struct KeyMax<uint32_t> {
    static constexpr uint32_t v = ~0u;
};

template <typename K>
__device__ inline double key_value(K k);
template <>
__device__ inline double key_value<uint64_t>(uint64_t k)
{
    return __longlong_as_double((long long)k);
}
template <>
__device__ inline double key_value<uint32_t>(uint32_t k)
{
    return (double)__uint_as_float(k);
}

// k(g) read off a bin's m sorted keys s[0 .. m).  Step rule: the smallest
// rank r whose g_r = (r+1)/m reaches g.  Midpoint-linear rule: key i sits at
// (i + 1/2)/m, straight lines between neighbours, the end keys held outside;
// no contraction, so the binary64 result is that of the expression as written.
template <typename K>
__device__ inline double k_of_g(const K* s, int64_t m, double g, int rule)
{
#pragma clang fp contract(off)
    if (rule == kRuleStep) {
        int64_t r = (int64_t)ceil(g * (double)m) - 1;
        r = r < 0 ? 0 : (r > m - 1 ? m - 1 : r);
        return key_value<K>(s[r]);
    }
    const double u = g * (double)m - 0.5;
    const double fl = floor(u);
    if (u <= 0.0) return key_value<K>(s[0]);
    if (fl >= (double)(m - 1)) return key_value<K>(s[m - 1]);
    const int64_t i = (int64_t)fl;  // 0 <= i <= m - 2
    const double a = key_value<K>(s[i]), b = key_value<K>(s[i + 1]);
    return a + (u - fl) * (b - a);
}

// LDS radix sort of one bin per workgroup (bins of up to kRadixMaxKeys keys):
// kRadixThreads threads hold the bin's keys in registers -- wavefront w
// holds positions [w R 64, (w+1) R 64), lane l of it key r at position
// w R 64 + r 64 + l (R keys per thread) -- and sort them least significant
// digit first, 8 bits per pass (binary32 keys: 4 passes; binary64 keys: the
// 4 passes of the high words and a finish, below).
// Each pass is stable: a wavefront ranks its keys round by round (so in
// position order) among equal digits with eight ballots (the lanes sharing a
// lane's digit are the AND over the digit's bits of each bit's ballot or its
// complement) and keeps a running count per digit in its own LDS counters,
// with no barrier between rounds; then the counters become offsets (waves in
// order, digits by a scan), every key is written to its place in LDS and read
// back in position order.  Four barriers per pass.
constexpr int kRadixThreads = 1024;
constexpr int kRadixWaves = kRadixThreads / 64;
constexpr int kRadixMaxRounds = 16;
constexpr int64_t kRadixMaxKeys = (int64_t)kRadixThreads * kRadixMaxRounds;
static_assert(kRadixMaxKeys <= (1 << 16), "LDS positions and counters fit 32 bits with room");

// The bin sorted into buf[0, m).  Binary32 keys: four passes.  Binary64
// keys: the four passes of their high words first; keys whose high words
// are equal (values within about 2^-20 of each other: few, in short runs)
// are then put in order by one thread per run, by insertion on the whole
// key.  Should a run be longer than kRunMax, the eight passes of the whole
// key follow instead.  Either way buf ends in ascending order of the keys.
constexpr int kRunMax = 32;

__device__ inline uint32_t key_hi(uint64_t k) { return (uint32_t)(k >> 32); }

template <typename K>
__device__ inline void radix_sort_block(K (&key)[kRadixMaxRounds], int rounds, int m, K* buf, uint32_t* cnt,
                                        uint32_t* wsum)
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    lds_volatile<uint32_t>* wc = (lds_volatile<uint32_t>*)(cnt + wave * 256);  // this wavefront's counters
    uint32_t rank[kRadixMaxRounds];
    constexpr bool wide = sizeof(K) == 8;
    int n_pass = 4;
    for (int it = 0; it < n_pass; ++it) {
        // binary64: the high word's bytes, then (only after a long run) all
        // eight from the lowest
        const int shift = !wide ? 8 * it : (it < 4 ? 32 + 8 * it : 8 * (it - 4));
        for (int q = lane; q < 256; q += 64) wc[q] = 0u;
#pragma unroll
        for (int r = 0; r < kRadixMaxRounds; ++r) {
            if (r < rounds) {
                const bool valid = wave * 64 * rounds + r * 64 + lane < m;
                const uint32_t d = (uint32_t)(key[r] >> shift) & 0xffu;
                // peers: the lanes whose digit equals this lane's, as two
                // 32-bit halves; bit b of the digit takes each lane's mask
                // mb = 0 where the bit is set and all ones where it is not,
                // and keeps the lanes of the ballot (bit set) XOR mb
                const uint64_t vb = __ballot(valid);
                uint32_t plo = (uint32_t)vb, phi = (uint32_t)(vb >> 32);
                const uint32_t nd = ~d;
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const uint32_t mb = (uint32_t)((int32_t)(nd << (31 - b)) >> 31);
                    const uint64_t bal = __ballot(mb == 0u);
                    plo &= (uint32_t)bal ^ mb;
                    phi &= (uint32_t)(bal >> 32) ^ mb;
                }
                const uint32_t rk = __builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, 0u));
                const uint32_t old = wc[d];
                rank[r] = old + rk;
                if (valid && rk == 0) wc[d] = old + (uint32_t)(__builtin_popcount(plo) + __builtin_popcount(phi));
            }
        }
        __syncthreads();
        // digit t (threads 0 .. 255): the waves' starts in wave order, then
        // the digits' starts by an exclusive scan of their totals
        uint32_t tot = 0;
        uint32_t pre[kRadixWaves];  // digit t's count in the waves before each
        if (t < 256) {
#pragma unroll
            for (int w = 0; w < kRadixWaves; ++w) pre[w] = cnt[w * 256 + t];
#pragma unroll
            for (int w = 0; w < kRadixWaves; ++w) {
                const uint32_t c = pre[w];
                pre[w] = tot;
                tot += c;
            }
        }
        uint32_t incl = tot;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t u = __shfl_up(incl, o, 64);
            if (lane >= o) incl += u;
        }
        if (t < 256 && lane == 63) wsum[wave] = incl;
        __syncthreads();
        if (t < 256) {
            uint32_t base = incl - tot;
            for (int w = 0; w < wave; ++w) base += wsum[w];
#pragma unroll
            for (int w = 0; w < kRadixWaves; ++w) cnt[w * 256 + t] = base + pre[w];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kRadixMaxRounds; ++r) {
            if (r < rounds && wave * 64 * rounds + r * 64 + lane < m) {
                const uint32_t d = (uint32_t)(key[r] >> shift) & 0xffu;
                const uint32_t pos = cnt[wave * 256 + d] + rank[r];
                if (pos < (uint32_t)m) buf[pos] = key[r];  // pos < m always
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kRadixMaxRounds; ++r) {
            const int p = wave * 64 * rounds + r * 64 + lane;
            if (r < rounds && p < m) key[r] = buf[p];
        }
        if (wide && it == 3) {
            bool long_run = false;
            for (int p = t; p + kRunMax < m; p += kRadixThreads)
                long_run |= key_hi((uint64_t)buf[p]) == key_hi((uint64_t)buf[p + kRunMax]);
            // (also the barrier after every thread's read-back)
            if (__syncthreads_or(long_run)) n_pass = 12;
        }
    }
    if (!wide || n_pass > 4) return;
    // (a thread reads the high words next to its run while other threads
    // reorder theirs: within a run every key has the same high word, so what
    // it reads does not depend on their progress)
    for (int p = t; p < m; p += kRadixThreads) {
        const uint32_t h = key_hi((uint64_t)buf[p]);
        if ((p > 0 && key_hi((uint64_t)buf[p - 1]) == h) || p + 1 >= m || key_hi((uint64_t)buf[p + 1]) != h)
            continue;
        int q = p + 1;  // the run [p, q] of high word h: at most kRunMax keys
        while (q + 1 < m && key_hi((uint64_t)buf[q + 1]) == h) ++q;
        for (int i = p + 1; i <= q; ++i) {
            const K v = buf[i];
            int j = i - 1;
            while (j >= p && buf[j] > v) {
                buf[j + 1] = buf[j];
                --j;
            }
            buf[j + 1] = v;
        }
    }
    __syncthreads();
}

// One workgroup per bin: bins of ppb consecutive points of n_states grids
// of n_points each (grid s at s * n_points; a grid's last bin may be short).
// Sorted keys to dst (optional, same layout) and k(g) to k_out[bin][g.n].
template <typename K>
__global__ __launch_bounds__(kRadixThreads) void radix_bin_kernel(const K* __restrict__ src, int64_t n_points,
                                                                  int64_t ppb, int64_t bins_per_grid,
                                                                  K* __restrict__ dst, GValues g,
                                                                  double* __restrict__ k_out)
{
    extern __shared__ __align__(16) unsigned char radix_lds[];
    const int64_t bin = blockIdx.x;
    const int64_t st = bin / bins_per_grid, lb = bin - st * bins_per_grid;
    const int64_t b0 = st * n_points + lb * ppb;
    const int m = (int)min(ppb, n_points - lb * ppb);
    const int rounds = (m + kRadixThreads - 1) / kRadixThreads;
    K* buf = reinterpret_cast<K*>(radix_lds);
    uint32_t* cnt = reinterpret_cast<uint32_t*>(radix_lds + (size_t)rounds * kRadixThreads * sizeof(K));
    uint32_t* wsum = cnt + kRadixWaves * 256;
    K key[kRadixMaxRounds];
    const int base_p = (int)(threadIdx.x >> 6) * 64 * rounds + (int)(threadIdx.x & 63);
#pragma unroll
    for (int r = 0; r < kRadixMaxRounds; ++r) {
        const int p = base_p + r * 64;
        key[r] = (r < rounds && p < m) ? src[b0 + p] : KeyMax<K>::v;
    }
    radix_sort_block<K>(key, rounds, m, buf, cnt, wsum);
    if (dst) {  // the sorted bin, from LDS (coalesced)
        for (int p = (int)threadIdx.x; p < m; p += kRadixThreads) dst[b0 + p] = buf[p];
    }
    // buf holds the bin in order after the last pass
    if ((int)threadIdx.x < g.n) k_out[bin * g.n + threadIdx.x] = k_of_g<K>(buf, m, g.g[threadIdx.x], g.rule);
}

// One workgroup per chunk of a larger bin (one grid): the chunk's keys in
// order to dst, same layout.  `chunk` is a whole number of rounds.
template <typename K>
__global__ __launch_bounds__(kRadixThreads) void radix_chunk_kernel(const K* __restrict__ src, int64_t n_points,
                                                                    int64_t ppb, int chunk, uint32_t chunks_per_bin,
                                                                    K* __restrict__ dst)
{
    extern __shared__ __align__(16) unsigned char radix_lds[];
    const uint32_t bin = blockIdx.x / chunks_per_bin;
    const int64_t first = (int64_t)(blockIdx.x - bin * chunks_per_bin) * chunk;  // in the bin
    const int64_t b0 = bin * ppb + first;
    const int64_t left = min(ppb - first, n_points - b0);
    if (left <= 0) return;
    const int m = (int)min((int64_t)chunk, left);
    const int rounds = chunk / kRadixThreads;
    K* buf = reinterpret_cast<K*>(radix_lds);
    uint32_t* cnt = reinterpret_cast<uint32_t*>(radix_lds + (size_t)chunk * sizeof(K));
    uint32_t* wsum = cnt + kRadixWaves * 256;
    K key[kRadixMaxRounds];
    const int base_p = (int)(threadIdx.x >> 6) * 64 * rounds + (int)(threadIdx.x & 63);
#pragma unroll
    for (int r = 0; r < kRadixMaxRounds; ++r) {
        const int p = base_p + r * 64;
        key[r] = (r < rounds && p < m) ? src[b0 + p] : KeyMax<K>::v;
    }
    radix_sort_block<K>(key, rounds, m, buf, cnt, wsum);
    for (int p = (int)threadIdx.x; p < m; p += kRadixThreads) dst[b0 + p] = buf[p];
}

// One pass of merging groups of kWays sorted runs of `run` keys (a
// multiple of kMergeThreads, so a workgroup's keys are of one run) inside
// each bin; src and dst differ.  One thread per key, which goes to its place
// in its own run plus its ranks in the others (keys of earlier runs count when
// equal).  Bound: latency on few keys, the probes on many.  The workgroup's
// first and last keys bound the windows of the other runs that its keys fall
// into: two searches per run of 16 lanes each, 16 probes a step (a run of 16384 keys
// in 4 dependent loads, not 14).  The windows, about kMergeThreads keys each,
// then are searched in LDS; where the runs' ranges differ so much that they
// do not fit there, in global memory.  The runs of a group are 8, or 4 or 2
// where no more are left to merge (each further run costs every key a search).
// Measured, binary64, the whole sort against chunks of 4096 keys by a bitonic
// network and merges of two runs with a search per key: 3 bins of 1e5 keys 95
// -> 52 us (16 chunks, 16 a merge), one of 3e6 493 -> 289, 150 of 2e4 189 ->
// 129, one of 2e7 4.5 -> 2.5 ms.
constexpr int kMergeWays = 8, kMergeThreads = 256, kMergeWindow = 3072;
static_assert(kMergeThreads == 2 * kMergeWays * 16, "a search of 16 lanes per bound");
template <typename K, int kWays>
__global__ __launch_bounds__(kMergeThreads) void merge_runs_kernel(const K* __restrict__ src, K* __restrict__ dst,
                                                                   int64_t n_points, int64_t ppb,
                                                                   uint32_t blocks_per_bin, int64_t run)
{
    __shared__ K win[kMergeWindow + 1];
    __shared__ uint32_t bound[2 * kMergeWays];
    const uint32_t bin = blockIdx.x / blocks_per_bin;
    const int64_t b0 = bin * ppb;
    const int64_t m = min(ppb, n_points - b0);
    const int64_t i0 = (int64_t)(blockIdx.x - bin * blocks_per_bin) * kMergeThreads;
    if (i0 >= m) return;
    const int t = threadIdx.x;
    const int64_t r = i0 / run;
    const int own = (int)(r % kWays);
    const int64_t g0 = (r - own) * run;  // the group's first key in the bin
    const K* grp = src + b0 + g0;
    // no key after the run's end: runs end at multiples of kMergeThreads or at m
    const int n_own = (int)min((int64_t)kMergeThreads, m - i0);
    const K key = src[b0 + i0 + min(t, n_own - 1)];
    {
        const int j = t >> 5;
        const K bk = src[b0 + i0 + ((t >> 4) & 1 ? n_own - 1 : 0)];
        const int64_t left = m - g0 - j * run;
        const K* rj = grp + j * run;
        uint32_t lo = 0u, hi = j >= kWays || j == own || left <= 0 ? 0u : (uint32_t)min(left, run);
        for (uint32_t size = (uint32_t)run; size; size = (size + 15u) / 16u - 1u) {
            // 16 lanes probe the ends of the 16 parts of [lo, hi)
            const uint32_t part = (hi - lo + 15u) / 16u;
            const uint32_t p = lo + ((t & 15) + 1u) * part;
            const bool in = part && p <= hi;
            const K v = in ? rj[p - 1] : K(0);
            const uint64_t before = __ballot(in && (v < bk || (v == bk && j < own)));
            const uint32_t c = __builtin_popcount((uint32_t)(before >> (t & 48)) & 0xffffu);
            if (part) {
                lo += c * part;
                hi = min(hi, lo + part - 1u);
            }
        }
        if ((t & 15) == 0) bound[t >> 4] = lo;
    }
    __syncthreads();
    uint32_t from[kWays], len[kWays], off[kWays], total = 0u, most = 0u;
#pragma unroll
    for (int j = 0; j < kWays; ++j) {
        from[j] = __builtin_amdgcn_readfirstlane(bound[2 * j]);
        len[j] = __builtin_amdgcn_readfirstlane(bound[2 * j + 1]) - from[j];
        off[j] = total;
        total += len[j];
        most = max(most, len[j]);
    }
    uint32_t lo[kWays] = {};
    const bool staged = total <= (uint32_t)kMergeWindow;
    if (staged) {
        for (uint32_t q0 = 0; q0 < total; q0 += 8 * kMergeThreads) {
            K v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint32_t q = min(q0 + u * kMergeThreads + t, total - 1u);
                int64_t at = from[0] + (int64_t)q;
#pragma unroll
                for (int j = 1; j < kWays; ++j)
                    at = q >= off[j] ? j * run + from[j] + (int64_t)(q - off[j]) : at;
                v[u] = grp[at];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint32_t q = q0 + u * kMergeThreads + t;
                if (q < total) win[q] = v[u];
            }
        }
        __syncthreads();
    }
    uint32_t step = most ? 1u << (31 - __builtin_clz(most)) : 0u;
    // the searches side by side, their loads in flight together (an empty
    // window reads some key and takes none)
    auto search = [&](auto at) {
        for (; step; step >>= 1) {
#pragma unroll
            for (int j = 0; j < kWays; ++j) {
                const uint32_t p = lo[j] + step;
                const K v = at(j, max(min(p, len[j]), 1u) - 1u);
                const bool take = (p <= len[j]) & ((v < key) | ((v == key) & (j < own)));
                lo[j] = take ? p : lo[j];
            }
        }
    };
    if (staged)
        search([&](int j, uint32_t q) { return win[off[j] + q]; });
    else
        search([&](int j, uint32_t q) { return grp[len[j] ? j * run + from[j] + (int64_t)q : 0]; });
    if (t >= n_own) return;
    int64_t at = i0 - r * run + t;
#pragma unroll
    for (int j = 0; j < kWays; ++j) at += from[j] + lo[j];
    dst[b0 + g0 + at] = key;
}

template <typename K>
__global__ __launch_bounds__(64) void kdist_pick_kernel(const K* __restrict__ sorted,
                                                        int64_t n_points, int64_t ppb, GValues g,
                                                        double* __restrict__ k_out)
{
    const int64_t bin = blockIdx.x;
    const int64_t b0 = bin * ppb;
    const int64_t m = min(ppb, n_points - b0);
    if ((int)threadIdx.x < g.n)
        k_out[bin * g.n + threadIdx.x] = k_of_g<K>(sorted + b0, m, g.g[threadIdx.x], g.rule);
}

// Chunks of a large bin: as short as gives each CU one, in steps of two
// rounds (a merge's workgroups that write to the same lines then are a
// multiple of 8 apart, so on one XCD).
constexpr int64_t kChunkShare = 256 * kRadixThreads;

template <typename K>
hipError_t run_kdist(const K* kappa, int64_t n_points, int64_t ppb, const GValues& g,
                     double* k_out, K* sorted_out, K* scratch, int64_t radix_keys,
                     int32_t n_states, hipStream_t s)
{
    const int64_t n_bins = (n_points + ppb - 1) / ppb;
    if (ppb <= radix_keys) {  // one LDS radix sort per bin, every grid in one launch
        const int rounds = (int)((ppb + kRadixThreads - 1) / kRadixThreads);
        const size_t shm = radix_lds_bytes(sizeof(K), rounds * kRadixThreads);
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&radix_bin_kernel<K>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
        if (e != hipSuccess) return e;
        const int64_t nb = n_bins * n_states;
        if (nb > (int64_t)UINT32_MAX) return hipErrorInvalidValue;
        radix_bin_kernel<K><<<dim3((unsigned)nb), dim3(kRadixThreads), shm, s>>>(kappa, n_points, ppb, n_bins,
                                                                                  sorted_out, g, k_out);
        return hipGetLastError();
    }
    if (n_states != 1) return hipErrorInvalidValue;  // bins above one LDS sort: one grid per call
    // chunks, then merges until one run covers the bin.  Ping-pong between the
    // scratch halves; the last step lands in sorted_out when given.
    const int64_t span = std::min(ppb, n_points);
    const int64_t rounds =
        std::min((n_points + 2 * kChunkShare - 1) / (2 * kChunkShare) * 2, radix_keys / kRadixThreads);
    const int64_t chunk = rounds * kRadixThreads;
    const int64_t cpb = (span + chunk - 1) / chunk, bpb = (span + kMergeThreads - 1) / kMergeThreads;
    const size_t shm = radix_lds_bytes(sizeof(K), chunk);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&radix_chunk_kernel<K>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    if (e != hipSuccess) return e;
    if (n_bins * bpb > (int64_t)UINT32_MAX) return hipErrorInvalidValue;
    K* cur = chunk >= span && sorted_out ? sorted_out : scratch;
    K* nxt = scratch + n_points;
    radix_chunk_kernel<K><<<dim3((unsigned)(n_bins * cpb)), dim3(kRadixThreads), shm, s>>>(
        kappa, n_points, ppb, (int)chunk, (uint32_t)cpb, cur);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (int64_t run = chunk; run < span; run *= kMergeWays) {
        K* out = run * kMergeWays >= span && sorted_out ? sorted_out : nxt;
        const int64_t runs = (span + run - 1) / run;  // (the last pass may have fewer than kMergeWays left)
        auto* merge = runs > 4 ? &merge_runs_kernel<K, 8> : runs > 2 ? &merge_runs_kernel<K, 4> : &merge_runs_kernel<K, 2>;
        merge<<<dim3((unsigned)(n_bins * bpb)), dim3(kMergeThreads), 0, s>>>(cur, out, n_points, ppb, (uint32_t)bpb,
                                                                              run);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        nxt = cur;
        cur = out;
    }
    kdist_pick_kernel<K><<<dim3((unsigned)n_bins), dim3(64), 0, s>>>(cur, n_points, ppb, g, k_out);
    return hipGetLastError();
}

}  // namespace

size_t radix_lds_bytes(int elem_bytes, int64_t keys)
{
    return (size_t)keys * elem_bytes + (size_t)kRadixWaves * 256 * 4 + 64;
}

int64_t kdist_radix_max_keys(int elem_bytes, int64_t lds_max)
{
    // whole rounds of kRadixThreads keys whose sort fits the workgroup's LDS
    int64_t r = kRadixMaxRounds;
    while (r > 0 && radix_lds_bytes(elem_bytes, r * kRadixThreads) > (size_t)lds_max) --r;
    return r * kRadixThreads;
}

size_t kdist_scratch_bytes(int elem_bytes, int64_t n_points, int64_t ppb, int64_t lds_max)
{
    if (ppb <= kdist_radix_max_keys(elem_bytes, lds_max)) return 0;
    return (size_t)2 * (size_t)n_points * (size_t)elem_bytes;
}

hipError_t launch_kdist(const void* kappa, int elem_bytes, int64_t n_points, int64_t ppb,
                        const GValues& g, double* k_out, void* sorted_out, void* scratch,
                        int64_t lds_max, int32_t n_states, hipStream_t s)
{
    if (n_points == 0 || n_states == 0) return hipSuccess;
    const int64_t rk = kdist_radix_max_keys(elem_bytes, lds_max);
    if (elem_bytes == 8)
        return run_kdist<uint64_t>(static_cast<const uint64_t*>(kappa), n_points, ppb, g, k_out,
                                   static_cast<uint64_t*>(sorted_out),
                                   static_cast<uint64_t*>(scratch), rk, n_states, s);
    return run_kdist<uint32_t>(static_cast<const uint32_t*>(kappa), n_points, ppb, g, k_out,
                               static_cast<uint32_t*>(sorted_out), static_cast<uint32_t*>(scratch),
                               rk, n_states, s);
}

// The fixed sort scratch of hk_kdist_noalloc: one array per device, made
// when the code object is loaded and held until the process ends.  Host code
// reaches it only through the address hipGetSymbolAddress returns for the
// current device (the array's name is a host-side stand-in).
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

hipError_t noalloc_scratch_address(void** ptr)
{
    *ptr = nullptr;
    return hipGetSymbolAddress(ptr, HIP_SYMBOL(scratch));
}

}  // namespace hk
