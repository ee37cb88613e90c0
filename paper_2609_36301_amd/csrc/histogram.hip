// Per-expert selection counts (the bincount behind the load-balancing statistic f,
// Appendix "Training"): counts[e] = #{(t, j) : idx[t][j] == e}.
//
// histogram_kernel: a workgroup counts, for one slice of the ids, the ids that fall into its range of
// experts, in LDS; with one slice it stores its range, with more it adds the non-empty bins with
// global atomics.  Every range reads all the ids (from L2).  histogram_hash_kernel, where that would
// be too many reads: a workgroup aggregates its slice in an LDS hash table.
// Counts are cleared by a fill kernel (not a memset) so the sequence stays valid inside a captured
// HIP graph; the routing calls clear them in a kernel of their own instead, and one slice needs no
// clearing.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lowrank.h"

namespace more {

constexpr int32_t kHistBins = 16384;       // experts per range, at most (LDS)
constexpr int kHistThreads = 1024;
constexpr int kHistGroups = 256;           // workgroups aimed at (one per CU)

__global__ __launch_bounds__(256) void fill_zero_kernel(int32_t* __restrict__ p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// blockIdx.x: slice of n / gridDim.x ids; blockIdx.y: experts [M y / gridDim.y, M (y + 1) / gridDim.y).
// A hot expert serialises: LDS atomics of a wave on one address take a cycle each (65536 ids of 256
// experts, a third of them one expert, in one workgroup: 24 us, 7 evenly spread).  So either the slices are
// short, or (one slice) every bin has `copies` copies (a power of two), lane l counting in copy l mod copies
// (6.1 us both ways).
template <bool COPIES>
__global__ __launch_bounds__(kHistThreads) void histogram_kernel(const int32_t* __restrict__ idx,
                                                                 int64_t n, int32_t M, int32_t copies,
                                                                 int32_t* __restrict__ counts) {
    __shared__ int32_t bins[kHistBins];
    const int32_t b0 = (int32_t)((int64_t)M * blockIdx.y / gridDim.y);
    const int32_t nb = (int32_t)((int64_t)M * (blockIdx.y + 1) / gridDim.y) - b0;
    const int32_t cs = COPIES ? copies : 1, own = (int32_t)threadIdx.x & (cs - 1);
    for (int32_t e = threadIdx.x; e < nb * cs; e += kHistThreads) bins[e] = 0;
    __syncthreads();
    const int64_t per = ((n + gridDim.x - 1) / gridDim.x + 3) / 4 * 4;
    const int64_t i0 = (int64_t)blockIdx.x * per;
    const int64_t i1 = i0 + per < n ? i0 + per : n;
    auto count = [&](int32_t id) {
        const uint32_t e = (uint32_t)id - (uint32_t)b0;  // ids below b0 wrap past nb
        if (e < (uint32_t)nb) atomicAdd(&bins[(int32_t)e * cs + own], 1);
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
        int32_t c = 0;
        for (int32_t q = 0; q < cs; ++q) c += bins[e * cs + ((q + own) & (cs - 1))];
        if (gridDim.x == 1)
            counts[b0 + e] = c;
        else if (c)
            atomicAdd(&counts[b0 + e], c);
    }
}

// Each workgroup aggregates one slice of kHashSlice ids in an LDS hash table (linear probing, twice as
// many slots as ids) and adds every distinct expert of the slice to counts with one global atomic.
constexpr int kHashSlice = 1024;
constexpr int kHashSlots = 2 * kHashSlice;  // power of two

__global__ __launch_bounds__(256) void histogram_hash_kernel(const int32_t* __restrict__ idx,
                                                             int64_t n, int32_t M,
                                                             int32_t* __restrict__ counts) {
    __shared__ int32_t key[kHashSlots], cnt[kHashSlots];
    for (int i = threadIdx.x; i < kHashSlots; i += blockDim.x) {
        key[i] = -1;
        cnt[i] = 0;
    }
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * kHashSlice;
    const int64_t i1 = i0 + kHashSlice < n ? i0 + kHashSlice : n;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
        const int32_t e = idx[i];
        if (e < 0 || e >= M) continue;
        uint32_t hh = ((uint32_t)e * 2654435761u) & (kHashSlots - 1);
        // at most kHashSlice distinct keys in kHashSlots slots: a free or matching slot exists
        for (int probe = 0; probe < kHashSlots; ++probe) {
            const int32_t old = atomicCAS(&key[hh], -1, e);
            if (old == -1 || old == e) {
                atomicAdd(&cnt[hh], 1);
                break;
            }
            hh = (hh + 1) & (kHashSlots - 1);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kHashSlots; i += blockDim.x)
        if (key[i] >= 0) atomicAdd(&counts[key[i]], cnt[i]);
}

// How a call is split.  Measured (us of the kernel, ids spread evenly / skewed so that the hottest of M
// experts has M^(-1/6) of them):
//   n 262144, M 256:      slices of 65536 ids 7.6 / 24, of 16384 3.7 / 7.9, of 4096 4.2 / 4.7
//   n 262144, M 16384:    5.6 / 13.5, 3.7 / 5.3, 6.3 / 5.4
//   n 2097152, M 16384:   6.8 / 14.2, 11.9 / 9.3, 19.2 / 17.8 (the atomics of the non-empty bins)
// so slices of 16384 ids where at most 2^19 bins have to be added up, else longer ones up to 65536.
// The ranges fill the chip, 256 experts or more each.  Reads grow with the number of ranges: at
// n 262144, M 2^20 (64 ranges) 12.2 / 10.8 against 14.6 / 60 with the hash table, at M 2^22 (256) a
// whole call takes 26.8 against 19.6, at n 65536, M 2^22 9.3 against 12.8.
struct HistSplit {
    int64_t slices, ranges;
    int32_t copies;
};

static bool histogram_split(int64_t n, int32_t M, bool counts_zeroed, HistSplit* p) {
    const int64_t least = (n + 65535) / 65536;
    int64_t slices = (n + 16383) / 16384;
    const int64_t room = ((int64_t)1 << 19) / M;
    if (slices > room) slices = room;
    // (up to 65536 ids one slice saves the launch that clears the counts)
    if (slices < least || (least == 1 && !counts_zeroed)) slices = least;
    if (slices > 65536) slices = 65536;
    int64_t ranges = kHistGroups / slices;
    if (ranges > M / 256) ranges = M / 256;
    const int64_t fit = ((int64_t)M + kHistBins - 1) / kHistBins;
    if (ranges < fit) ranges = fit;
    const int64_t nb = (M + ranges - 1) / ranges;
    p->slices = slices;
    p->ranges = ranges;
    p->copies = 1;
    if (slices == 1)
        while (p->copies < 32 && 2 * p->copies * nb <= 8192) p->copies *= 2;
    return ranges <= 64 || (n * ranges <= ((int64_t)1 << 25) && ranges <= 4096);
}

hipError_t histogram_launch(const int32_t* idx, int64_t n, int32_t M, int32_t* counts,
                            hipStream_t st, bool counts_zeroed) {
    HistSplit p{0, 0, 1};
    const bool dense = n > 0 && histogram_split(n, M, counts_zeroed, &p);
    if (!counts_zeroed && !(dense && p.slices == 1)) {
        int64_t blocks = ((int64_t)M + 255) / 256;
        if (blocks > 1024) blocks = 1024;
        hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, st, counts,
                           (int64_t)M);
    }
    const dim3 grid((unsigned)p.slices, (unsigned)p.ranges);
    if (dense && p.copies > 1)
        hipLaunchKernelGGL(histogram_kernel<true>, grid, dim3(kHistThreads), 0, st, idx, n, M, p.copies,
                           counts);
    else if (dense)
        hipLaunchKernelGGL(histogram_kernel<false>, grid, dim3(kHistThreads), 0, st, idx, n, M, 1, counts);
    else if (n > 0)
        hipLaunchKernelGGL(histogram_hash_kernel, dim3((unsigned)((n + kHashSlice - 1) / kHashSlice)),
                           dim3(256), 0, st, idx, n, M, counts);
    return hipGetLastError();
}

}  // namespace more
