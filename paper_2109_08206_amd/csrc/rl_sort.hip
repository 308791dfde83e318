// Stable key-value radix sort (rocPRIM through hipCUB), used to put rods in
// cell order deterministically: equal cells keep ascending rod index.
#include <algorithm>

#include <hipcub/hipcub.hpp>

#include "rl_internal.hpp"

namespace rl {

__global__ void k_iota(int64_t n, int *__restrict__ v)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) v[i] = (int)i;
}

// perm[t] = rod with the t-th smallest (key, index); keys_out receives the keys.
int stable_sort_by_key(rl_ctx *h, int64_t n, const int *keys, int bits, int *keys_out, int *perm)
{
    hipStream_t st = h->stream;
    int werr = 0;
    int *idx = (int *)ws_get(h, kWsSortIdx, sizeof(int) * (n > 0 ? n : 1), &werr);
    if (werr) return werr;
    hipLaunchKernelGGL(k_iota, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, n, idx);
    RL_HIP(hipGetLastError());
    size_t tmp_bytes = 0;
    RL_HIP(hipcub::DeviceRadixSort::SortPairs(nullptr, tmp_bytes, keys, keys_out, idx, perm, (int)n, 0, bits, st));
    void *tmp = ws_get(h, kWsSortTmp, tmp_bytes, &werr);
    if (werr) return werr;
    RL_HIP(hipcub::DeviceRadixSort::SortPairs(tmp, tmp_bytes, keys, keys_out, idx, perm, (int)n, 0, bits, st));
    return RL_OK;
}

__global__ void k_scan_ends(int64_t m, int *__restrict__ out, int64_t *__restrict__ total)
{
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    out[0] = 0;
    if (total) *total = out[m];
}

int scan_tmp_bytes(int64_t m, size_t *bytes)
{
    *bytes = 0;
    if (m <= kScanOne) return RL_OK;
    RL_HIP(hipcub::DeviceScan::InclusiveSum(nullptr, *bytes, (const int *)nullptr, (int *)nullptr, (int)m,
                                            (hipStream_t)0));
    return RL_OK;
}

// Exclusive sums of one or two arrays of m <= kScanOne counts, a workgroup
// each: all of a thread's counts are loaded at once, and three barriers join
// the waves.  (The library's scan takes two launches and the ends a third:
// 5.0 us at 1,000 counts, this one 2.9.)  total (may be null) receives the
// first sum; rep: see rl_internal.hpp.
constexpr int kScanBlock = 1024, kScanTiles = 4;
static_assert(kScanOne == 4 * kScanBlock * kScanTiles, "four counts per thread and tile");

__global__ void __launch_bounds__(kScanBlock)
    k_scan_one(int m, const int *__restrict__ in0, int *__restrict__ out0, const int *__restrict__ in1,
               int *__restrict__ out1, int64_t *__restrict__ total, ScanReport rep)
{
    __shared__ int part[kScanTiles * kScanBlock / 64];
    const int *in = blockIdx.x ? in1 : in0;
    int *out = blockIdx.x ? out1 : out0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int v[kScanTiles][4], incl[kScanTiles];
#pragma unroll
    for (int k = 0; k < kScanTiles; ++k)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = 4 * (k * kScanBlock + (int)threadIdx.x) + u;
            v[k][u] = i < m ? in[i] : 0;
        }
#pragma unroll
    for (int k = 0; k < kScanTiles; ++k) {
        incl[k] = v[k][0] + v[k][1] + v[k][2] + v[k][3];
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(incl[k], d, 64);
            if (lane >= d) incl[k] += t;
        }
        if (lane == 63) part[k * (kScanBlock / 64) + wave] = incl[k];
    }
    __syncthreads();
    static_assert(kScanTiles * kScanBlock / 64 == 64, "one wave adds the waves' sums");
    if (wave == 0) {
        int s = part[lane];
        const int own = s;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(s, d, 64);
            if (lane >= d) s += t;
        }
        part[lane] = s - own;
        if (blockIdx.x == 0 && lane == 63) {
            if (total) *total = s;
            if (rep.host) {
                rep.host[0] = rep.count ? (int64_t)*rep.count : (int64_t)s;
                rep.host[1] = *rep.flag;
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) out[0] = 0;
#pragma unroll
    for (int k = 0; k < kScanTiles; ++k) {
        int run = part[k * (kScanBlock / 64) + wave] + incl[k] - (v[k][0] + v[k][1] + v[k][2] + v[k][3]);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = 4 * (k * kScanBlock + (int)threadIdx.x) + u;
            run += v[k][u];
            if (i < m) out[i + 1] = run;
        }
    }
}

hipError_t launch_scan_one(hipStream_t st, int64_t m, const int *in0, int *out0, const int *in1, int *out1,
                           int64_t *total, const ScanReport &rep)
{
    hipLaunchKernelGGL(k_scan_one, dim3(in1 ? 2 : 1), dim3(kScanBlock), 0, st, (int)m, in0, out0, in1, out1, total,
                       rep);
    return hipGetLastError();
}

int device_scan(rl_ctx *h, const int *in, int64_t m, int *out, int64_t *total, void *tmp)
{
    hipStream_t st = h->stream;
    if (m <= kScanOne) {
        RL_HIP(launch_scan_one(st, m, in, out, nullptr, nullptr, total, ScanReport{nullptr, nullptr, nullptr}));
        return RL_OK;
    }
    {
        int werr = 0;
        size_t tmp_bytes = 0;
        RL_HIP(hipcub::DeviceScan::InclusiveSum(nullptr, tmp_bytes, in, out + 1, (int)m, st));
        if (!tmp) tmp = ws_get(h, kWsScanTmp, tmp_bytes, &werr);
        if (werr) return werr;
        RL_HIP(hipcub::DeviceScan::InclusiveSum(tmp, tmp_bytes, in, out + 1, (int)m, st));
    }
    hipLaunchKernelGGL(k_scan_ends, dim3(1), dim3(64), 0, st, m, out, total);
    RL_HIP(hipGetLastError());
    return RL_OK;
}

int sort_tmp_bytes(int64_t n, int64_t m, size_t *bytes)
{
    size_t rods = 0, forces = 0;
    const int *k = nullptr;
    const unsigned long long *w = nullptr;
    const double *v = nullptr;
    RL_HIP(hipcub::DeviceRadixSort::SortPairs(nullptr, rods, k, (int *)nullptr, k, (int *)nullptr, (int)n, 0, 31,
                                              (hipStream_t)0));
    RL_HIP(hipcub::DeviceRadixSort::SortPairs(nullptr, forces, w, (unsigned long long *)nullptr, v, (double *)nullptr,
                                              (int)m, 0, 64, (hipStream_t)0));
    *bytes = std::max(rods, forces);
    return RL_OK;
}

// sorts m (key, value) pairs by key into keys_out / vals_out
int sort_key_values(rl_ctx *h, int64_t m, const unsigned long long *keys, const double *vals,
                    unsigned long long *keys_out, double *vals_out)
{
    hipStream_t st = h->stream;
    if (m <= 0) return RL_OK;
    int werr = 0;
    size_t tmp_bytes = 0;
    RL_HIP(hipcub::DeviceRadixSort::SortPairs(nullptr, tmp_bytes, keys, keys_out, vals, vals_out, (int)m, 0, 64, st));
    void *tmp = ws_get(h, kWsSortTmp, tmp_bytes, &werr);
    if (werr) return werr;
    RL_HIP(hipcub::DeviceRadixSort::SortPairs(tmp, tmp_bytes, keys, keys_out, vals, vals_out, (int)m, 0, 64, st));
    return RL_OK;
}

}  // namespace rl
