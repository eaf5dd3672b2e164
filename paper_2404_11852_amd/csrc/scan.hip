// Exclusive prefix sum of uint32 counts (ray -> first live sample, brick ->
// first bucket slot); out has n+1 entries, out[n] is the grand total.  Up to
// kScanOne counts: one block in one launch.  More: per-block scans with block
// totals, then an add-back whose blocks sum the totals before them by
// themselves.  A launch and its gap take about 8 us here, more than the scan
// of an 800x800 frame's counts: 64x64 frame, three launches of 8.6 us in all and
// their gaps -> one of 3.5 us (frame 67.6 -> 63.0 us).
#include "kernels.h"

namespace cic {

constexpr int kScanThreads = 256;
constexpr int kScanPer = 8;
constexpr int kScanBlock = kScanThreads * kScanPer;   // 2048 elements per block

size_t scan_tmp_elems(int64_t n)
{
    int64_t blocks = (n + kScanBlock - 1) / kScanBlock;
    return (size_t)blocks + 1;
}

// Block-wide exclusive scan of one value per thread; returns the block total.
template <int THREADS>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t &total)
{
    __shared__ uint32_t wsum[THREADS / kWave];
    const int l = lane_id(), w = threadIdx.x / kWave;
    uint32_t x = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        uint32_t u = __shfl_up(x, off, kWave);
        if (l >= off) x += u;
    }
    if (l == kWave - 1) wsum[w] = x;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < THREADS / kWave; ++i) {
        if (i < w) before += wsum[i];
        all += wsum[i];
    }
    __syncthreads();
    total = all;
    return before + x - v;
}

constexpr int kOneThreads = 1024, kOnePer = 16;
constexpr int64_t kScanOne = (int64_t)kOneThreads * kOnePer;   // most counts of the one-block scan

// Each thread takes `per` consecutive counts, 16-byte loads of four; in and
// out may be the same array, 16-byte aligned and with room for the last four.
__global__ __launch_bounds__(kOneThreads) void k_scan_one(const uint32_t *in, uint32_t *out, int n)
{
    typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
    const int per = ((n + kOneThreads - 1) / kOneThreads + 3) & ~3, base = (int)threadIdx.x * per;
    u4_t v[kOnePer / 4];
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < kOnePer / 4; ++i) {
        const int at = base + 4 * i;
        v[i] = 4 * i < per && at < n ? *(const u4_t *)(in + at) : u4_t{0u, 0u, 0u, 0u};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (at + e >= n) v[i][e] = 0u;
            s += v[i][e];
        }
    }
    uint32_t total;
    uint32_t pre = block_exclusive_scan<kOneThreads>(s, total);   // its barriers separate the reads from the writes
#pragma unroll
    for (int i = 0; i < kOnePer / 4; ++i) {
        const int at = base + 4 * i;
        u4_t w;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            w[e] = pre;
            pre += v[i][e];
        }
        if (4 * i >= per) break;
        if (at + 4 <= n) {
            *(u4_t *)(out + at) = w;
        } else {
            for (int e = 0; e < 4 && at + e < n; ++e) out[at + e] = w[e];
        }
    }
    if (threadIdx.x == 0) out[n] = total;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_blocks(const uint32_t *in, uint32_t *out, uint32_t *tmp,
                                                              int64_t n)
{
    const int64_t base = (int64_t)blockIdx.x * kScanBlock + (int64_t)threadIdx.x * kScanPer;
    uint32_t v[kScanPer];
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < kScanPer; ++i) {
        v[i] = (base + i < n) ? in[base + i] : 0u;
        s += v[i];
    }
    uint32_t total;
    uint32_t pre = block_exclusive_scan<kScanThreads>(s, total);
#pragma unroll
    for (int i = 0; i < kScanPer; ++i) {
        if (base + i < n) out[base + i] = pre;
        pre += v[i];
    }
    if (threadIdx.x == 0) tmp[blockIdx.x] = total;
}

// Adds the totals of the blocks before this one (at most kScanBlock of them,
// summed by the block itself).
__global__ __launch_bounds__(kScanThreads) void k_scan_add(uint32_t *out, const uint32_t *tmp, int64_t n, int64_t nb)
{
    __shared__ uint32_t wsum[2][kScanThreads / kWave];
    uint32_t before = 0, all = 0;
    for (int64_t i = threadIdx.x; i < nb; i += kScanThreads) {
        const uint32_t t = tmp[i];
        all += t;
        before += i < (int64_t)blockIdx.x ? t : 0u;
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        before += __shfl_xor(before, off, kWave);
        all += __shfl_xor(all, off, kWave);
    }
    if (lane_id() == 0) {
        wsum[0][threadIdx.x / kWave] = before;
        wsum[1][threadIdx.x / kWave] = all;
    }
    __syncthreads();
    uint32_t add = 0, total = 0;
#pragma unroll
    for (int i = 0; i < kScanThreads / kWave; ++i) {
        add += wsum[0][i];
        total += wsum[1][i];
    }
    const int64_t base = (int64_t)blockIdx.x * kScanBlock + (int64_t)threadIdx.x * kScanPer;
#pragma unroll
    for (int i = 0; i < kScanPer; ++i)
        if (base + i < n) out[base + i] += add;
    if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = total;
}

void launch_exclusive_scan(const uint32_t *in, uint32_t *out, uint32_t *tmp, int64_t n, hipStream_t s)
{
    // n <= kScanBlock * kScanBlock (4M) is guaranteed by the callers.
    if (n <= kScanOne) {
        hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(kOneThreads), 0, s, in, out, (int)n);
        return;
    }
    const int64_t nb = (n + kScanBlock - 1) / kScanBlock;
    hipLaunchKernelGGL(k_scan_blocks, dim3((unsigned)nb), dim3(kScanThreads), 0, s, in, out, tmp, n);
    hipLaunchKernelGGL(k_scan_add, dim3((unsigned)nb), dim3(kScanThreads), 0, s, out, tmp, n, nb);
}

}  // namespace cic
