// Per-expert selection counts (the bincount behind the load-balancing statistic f,
// Appendix "Training"): counts[e] = #{(t, j) : idx[t][j] == e}.
//
// A workgroup counts, for one slice of the ids, the ids that fall into its range of experts, in LDS;
// with one slice it stores its range, with more it adds the non-empty bins with global atomics.
// Every range reads all the ids (from L2), which is cheap next to the atomics that this saves: they
// run at about 20 per ns on the whole chip, and 262144 ids of 16384 experts in 64 slices of all
// experts took 225000 of them (13.5 us); four slices take at most 65536.  Counts are
// cleared by a fill kernel (not a memset) so the sequence stays valid inside a captured HIP graph;
// the routing calls clear them in a kernel of their own instead, and one slice needs no clearing.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lowrank.h"

namespace more {

constexpr int32_t kHistBins = 16384;       // experts per range, at most (LDS)
constexpr int64_t kHistSlice = 65536;      // ids per workgroup, about: 3 us of scanning
constexpr int kHistThreads = 1024;
constexpr int kHistGroups = 256;           // workgroups aimed at (one per CU)

__global__ __launch_bounds__(256) void fill_zero_kernel(int32_t* __restrict__ p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// blockIdx.x: slice of n / gridDim.x ids; blockIdx.y: experts [M y / gridDim.y, M (y + 1) / gridDim.y).
__global__ __launch_bounds__(kHistThreads) void histogram_kernel(const int32_t* __restrict__ idx,
                                                                 int64_t n, int32_t M,
                                                                 int32_t* __restrict__ counts) {
    __shared__ int32_t bins[kHistBins];
    const int32_t b0 = (int32_t)((int64_t)M * blockIdx.y / gridDim.y);
    const int32_t nb = (int32_t)((int64_t)M * (blockIdx.y + 1) / gridDim.y) - b0;
    for (int32_t e = threadIdx.x; e < nb; e += kHistThreads) bins[e] = 0;
    __syncthreads();
    const int64_t per = ((n + gridDim.x - 1) / gridDim.x + 3) / 4 * 4;
    const int64_t i0 = (int64_t)blockIdx.x * per;
    const int64_t i1 = i0 + per < n ? i0 + per : n;
    auto count = [&](int32_t id) {
        const uint32_t e = (uint32_t)id - (uint32_t)b0;  // ids below b0 wrap past nb
        if (e < (uint32_t)nb) atomicAdd(&bins[e], 1);
    };
    int64_t i = i0 + 4 * threadIdx.x;
    if ((reinterpret_cast<uintptr_t>(idx) & 15) == 0) {  // i0 is a multiple of 4
        for (; i + 4 * kHistThreads + 3 < i1; i += 8 * kHistThreads) {  // two loads in flight
            const int4 a = *reinterpret_cast<const int4*>(idx + i);
            const int4 b = *reinterpret_cast<const int4*>(idx + i + 4 * kHistThreads);
            count(a.x), count(a.y), count(a.z), count(a.w);
            count(b.x), count(b.y), count(b.z), count(b.w);
        }
    }
    for (; i < i1; i += 4 * kHistThreads)
        for (int64_t j = i; j < i + 4 && j < i1; ++j) count(idx[j]);
    __syncthreads();
    for (int32_t e = threadIdx.x; e < nb; e += kHistThreads) {
        const int32_t c = bins[e];
        if (gridDim.x == 1)
            counts[b0 + e] = c;
        else if (c)
            atomicAdd(&counts[b0 + e], c);
    }
}

hipError_t histogram_launch(const int32_t* idx, int64_t n, int32_t M, int32_t* counts,
                            hipStream_t st, bool counts_zeroed) {
    int64_t slices = (n + kHistSlice - 1) / kHistSlice;
    if (slices > 65536) slices = 65536;
    if (!counts_zeroed && slices != 1) {
        int64_t blocks = ((int64_t)M + 255) / 256;
        if (blocks > 1024) blocks = 1024;
        hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, st, counts,
                           (int64_t)M);
    }
    if (n > 0) {
        // ranges of at least 256 experts while there are fewer workgroups than CUs
        int64_t ranges = kHistGroups / slices;
        if (ranges > M / 256) ranges = M / 256;
        const int64_t least = ((int64_t)M + kHistBins - 1) / kHistBins;
        if (ranges < least) ranges = least;
        hipLaunchKernelGGL(histogram_kernel, dim3((unsigned)slices, (unsigned)ranges),
                           dim3(kHistThreads), 0, st, idx, n, M, counts);
    }
    return hipGetLastError();
}

}  // namespace more
