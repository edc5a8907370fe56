// sort_dev.h -- the device sorts of kdist.hip and line_sort.hip: a radix sort
// of one workgroup's keys in registers and LDS, and for more keys than that
// sorted chunks merged eight runs at a time in global memory (each key finds
// its rank in the other seven by searches; ties keep the earlier run first).
// Keys are unsigned integers (the bit patterns of non-negative IEEE values
// order like the values); either may carry a 32-bit index, and both are stable.
#pragma once

#include <algorithm>

#include "hk_internal.h"

namespace hk {
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

// LDS radix sort of up to kRadixMaxKeys keys by one workgroup: kRadixThreads
// threads hold the keys in registers -- wavefront w
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

// The keys sorted into buf[0, m), with kIdx their index values into ibuf in
// the same order (stable: equal keys keep theirs).  Binary32 keys: four passes.  Binary64
// keys: the four passes of their high words first; keys whose high words
// are equal (values within about 2^-20 of each other: few, in short runs)
// are then put in order by one thread per run, by insertion on the whole
// key.  Should a run of different keys be longer than kRunMax (or have half
// of that on one side of two different neighbours), the eight passes of the
// whole key follow instead; a run of equal keys (the zeros where no line
// reaches) is in order as it is.  Either way buf ends in ascending order of
// the keys.  (300 bins of 1e4 keys, three or nine in ten of them 0: 180 us with
// the eight passes for every run longer than kRunMax, 78 now; without zeros 75
// and 76.)
constexpr int kRunMax = 32;

__device__ inline uint32_t key_hi(uint64_t k) { return (uint32_t)(k >> 32); }

template <typename K, bool kIdx>
__device__ inline void radix_sort_block(K (&key)[kRadixMaxRounds], uint32_t (&idx)[kIdx ? kRadixMaxRounds : 1],
                                        int rounds, int m, K* buf, uint32_t* ibuf, uint32_t* cnt, uint32_t* wsum)
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
                if (pos < (uint32_t)m) {  // always
                    buf[pos] = key[r];
                    if constexpr (kIdx) ibuf[pos] = idx[r];
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kRadixMaxRounds; ++r) {
            const int p = wave * 64 * rounds + r * 64 + lane;
            if (r < rounds && p < m) {
                key[r] = buf[p];
                if constexpr (kIdx) idx[r] = ibuf[p];
            }
        }
        if (wide && it == 3) {
            bool long_run = false;
            constexpr int kHalf = kRunMax / 2;  // one side of a pair in a run longer than kRunMax
            for (int p = t; p + 1 < m; p += kRadixThreads) {
                const K a = buf[p], b = buf[p + 1];
                const uint32_t h = key_hi((uint64_t)a);
                if (a == b || key_hi((uint64_t)b) != h) continue;
                long_run |= (p >= kHalf - 1 && key_hi((uint64_t)buf[p - (kHalf - 1)]) == h) ||
                            (p + kHalf < m && key_hi((uint64_t)buf[p + kHalf]) == h);
            }
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
        int q = p + 1;  // the run [p, q] of high word h; beyond kRunMax keys it is of equal keys
        while (q + 1 < m && q - p < kRunMax && key_hi((uint64_t)buf[q + 1]) == h) ++q;
        if (q - p >= kRunMax) continue;
        for (int i = p + 1; i <= q; ++i) {
            const K v = buf[i];
            uint32_t vi = 0u;
            if constexpr (kIdx) vi = ibuf[i];
            int j = i - 1;
            while (j >= p && buf[j] > v) {
                buf[j + 1] = buf[j];
                if constexpr (kIdx) ibuf[j + 1] = ibuf[j];
                --j;
            }
            buf[j + 1] = v;
            if constexpr (kIdx) ibuf[j + 1] = vi;
        }
    }
    __syncthreads();
}

// dynamic LDS of a radix sort of `keys` keys of elem_bytes (and, with an index
// each, of index_bytes = 4 more)
inline size_t radix_lds_bytes(int elem_bytes, int64_t keys, int index_bytes = 0)
{
    return (size_t)keys * (elem_bytes + index_bytes) + (size_t)kRadixWaves * 256 * 4 + kRadixWaves * 4;
}

// One workgroup per chunk of a bin (one grid): the chunk's keys in order to
// dst, same layout, and with kIdx their positions in src to idst (dst then may
// be NULL).  `chunk` is a whole number of rounds.
template <typename K, bool kIdx>
__global__ __launch_bounds__(kRadixThreads) void radix_chunk_kernel(const K* __restrict__ src, int64_t n_points,
                                                                    int64_t ppb, int chunk, uint32_t chunks_per_bin,
                                                                    K* __restrict__ dst, uint32_t* __restrict__ idst)
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
    uint32_t* ibuf = wsum + kRadixWaves;
    K key[kRadixMaxRounds];
    uint32_t idx[kIdx ? kRadixMaxRounds : 1];
    const int base_p = (int)(threadIdx.x >> 6) * 64 * rounds + (int)(threadIdx.x & 63);
#pragma unroll
    for (int r = 0; r < kRadixMaxRounds; ++r) {
        const int p = base_p + r * 64;
        key[r] = (r < rounds && p < m) ? src[b0 + p] : KeyMax<K>::v;
        if constexpr (kIdx) idx[r] = (uint32_t)(b0 + p);
    }
    radix_sort_block<K, kIdx>(key, idx, rounds, m, buf, ibuf, cnt, wsum);
    for (int p = (int)threadIdx.x; p < m; p += kRadixThreads) {
        if (!kIdx || dst) dst[b0 + p] = buf[p];
        if constexpr (kIdx) idst[b0 + p] = ibuf[p];
    }
}

// One pass of merging groups of kWays sorted runs of `run` keys (a
// multiple of kMergeThreads, so a workgroup's keys are of one run) inside
// each bin; src and dst differ; with kIdx the keys' indexes go along (and dst
// may be NULL: a last pass of which only they are wanted).  One thread per key, which goes to its place
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
template <typename K, int kWays, bool kIdx>
__global__ __launch_bounds__(kMergeThreads) void merge_runs_kernel(const K* __restrict__ src, K* __restrict__ dst,
                                                                   int64_t n_points, int64_t ppb,
                                                                   uint32_t blocks_per_bin, int64_t run,
                                                                   const uint32_t* __restrict__ isrc,
                                                                   uint32_t* __restrict__ idst)
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
    uint32_t idx = 0u;
    if constexpr (kIdx) idx = isrc[b0 + i0 + min(t, n_own - 1)];
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
    if (!kIdx || dst) dst[b0 + g0 + at] = key;
    if constexpr (kIdx) idst[b0 + g0 + at] = idx;
}

// Chunks: as short as gives each CU one, in steps of two
// rounds (a merge's workgroups that write to the same lines then are a
// multiple of 8 apart, so on one XCD).
constexpr int64_t kChunkShare = 256 * kRadixThreads;


// The bins of ppb keys of src[0 .. n) (larger than one workgroup sorts, or not)
// in order, in chunks of at most max_rounds rounds and merges until one run
// covers a bin.  Ping-pong between k0 and k1 (n keys each; k0 also where there
// is one chunk per bin), with kIdx i0 and i1; the last step's keys go to `last`
// when given, with kIdx nowhere else.
template <typename K, bool kIdx>
hipError_t sort_in_runs(const K* src, int64_t n, int64_t ppb, K* k0, K* k1, uint32_t* i0, uint32_t* i1, K* last,
                        int64_t max_rounds, const K** keys_out, const uint32_t** idx_out, hipStream_t s)
{
    const int64_t span = std::min(ppb, n), n_bins = (n + ppb - 1) / ppb;
    const int64_t rounds = std::min((n + 2 * kChunkShare - 1) / (2 * kChunkShare) * 2, max_rounds);
    const int64_t chunk = rounds * kRadixThreads;
    const int64_t cpb = (span + chunk - 1) / chunk, bpb = (span + kMergeThreads - 1) / kMergeThreads;
    const size_t shm = radix_lds_bytes(sizeof(K), chunk, kIdx ? 4 : 0);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&radix_chunk_kernel<K, kIdx>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    if (e != hipSuccess) return e;
    if (n_bins * bpb > (int64_t)UINT32_MAX) return hipErrorInvalidValue;
    K* cur = chunk >= span && (kIdx || last) ? last : k0;
    K* nxt = k1;
    radix_chunk_kernel<K, kIdx><<<dim3((unsigned)(n_bins * cpb)), dim3(kRadixThreads), shm, s>>>(
        src, n, ppb, (int)chunk, (uint32_t)cpb, cur, i0);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (int64_t run = chunk; run < span; run *= kMergeWays) {
        K* out = run * kMergeWays >= span && (kIdx || last) ? last : nxt;
        const int64_t runs = (span + run - 1) / run;  // (the last pass may have fewer than kMergeWays left)
        auto* merge = runs > 4   ? &merge_runs_kernel<K, 8, kIdx>
                      : runs > 2 ? &merge_runs_kernel<K, 4, kIdx>
                                 : &merge_runs_kernel<K, 2, kIdx>;
        merge<<<dim3((unsigned)(n_bins * bpb)), dim3(kMergeThreads), 0, s>>>(cur, out, n, ppb, (uint32_t)bpb, run, i0,
                                                                              i1);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        nxt = cur;
        cur = out;
        std::swap(i0, i1);
    }
    if (keys_out) *keys_out = cur;
    if (idx_out) *idx_out = i0;
    return hipSuccess;
}

}  // namespace
}  // namespace hk
