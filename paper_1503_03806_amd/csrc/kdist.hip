// kdist.hip -- the "Sort" stage (§2.2, §2.6): per-bin sort of the opacity
// grid, cumulative coordinate g_i = (i+1)/M, and k(g) at the requested g by
// the step or the midpoint-linear rule.
//
// The paper sorts the whole grid at once with bin tags (Thrust, §2.6).  Here
// bins are independent, and keys are the opacities' bit patterns
// (non-negative IEEE values order like their unsigned integer images).  A
// bin of up to kRadixMaxKeys keys is sorted by one workgroup, a larger one in
// chunks that are merged (sort_dev.h).
#include "hk_internal.h"
#include "sort_dev.h"

namespace hk {
namespace {

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

// One workgroup per bin, from bin0 on: bins of ppb consecutive points of n_states
// grids of n_points each (grid s at s * n_points; a grid's last bin may be short).
// Sorted keys to dst (optional, same layout) and k(g) to k_out[bin][g.n].
template <typename K>
__global__ __launch_bounds__(kRadixThreads) void radix_bin_kernel(const K* __restrict__ src, int64_t n_points,
                                                                  int64_t ppb, int64_t bins_per_grid, int64_t bin0,
                                                                  K* __restrict__ dst, GValues g,
                                                                  double* __restrict__ k_out)
{
    extern __shared__ __align__(16) unsigned char radix_lds[];
    const int64_t bin = bin0 + blockIdx.x;
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
    uint32_t none[1];
    radix_sort_block<K, false>(key, none, rounds, m, buf, nullptr, cnt, wsum);
    if (dst) {  // the sorted bin, from LDS (coalesced)
        for (int p = (int)threadIdx.x; p < m; p += kRadixThreads) dst[b0 + p] = buf[p];
    }
    // buf holds the bin in order after the last pass
    if ((int)threadIdx.x < g.n) k_out[bin * g.n + threadIdx.x] = k_of_g<K>(buf, m, g.g[threadIdx.x], g.rule);
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
        // (a launch holds less than 2^32 threads)
        constexpr int64_t most = (int64_t)1 << 21;
        for (int64_t b = 0, nb = n_bins * n_states; b < nb; b += most)
            radix_bin_kernel<K><<<dim3((unsigned)std::min(most, nb - b)), dim3(kRadixThreads), shm, s>>>(
                kappa, n_points, ppb, n_bins, b, sorted_out, g, k_out);
        return hipGetLastError();
    }
    if (n_states != 1) return hipErrorInvalidValue;  // bins above one LDS sort: one grid per call
    const K* sorted = nullptr;
    hipError_t e = sort_in_runs<K, false>(kappa, n_points, ppb, scratch, scratch + n_points, nullptr, nullptr,
                                          sorted_out, radix_keys / kRadixThreads, &sorted, nullptr, s);
    if (e != hipSuccess) return e;
    kdist_pick_kernel<K><<<dim3((unsigned)n_bins), dim3(64), 0, s>>>(sorted, n_points, ppb, g, k_out);
    return hipGetLastError();
}

}  // namespace

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
