// Bucket route (bucket.hip): one screening sweep that keeps bucket maxima, then an exact selection
// from the few buckets that can hold the top k.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace more {

constexpr int32_t kBucketMaxRank = 256;
// Below, each token's selection reads a large part of all rows.  T 16384, r 128, against the three-piece
// sweep of the wide route: k 8 83 us and 115 at M 2048, 81 and 103 at 1536, 78 and 90 at 1024, 75 and 73 at
// 512; k 32 147 and 243 at 1024, 263 and 179 at 512: the crossing lies between 512 and 1024, and this line
// is on the safe side of it.
constexpr int32_t kBucketMinExperts = 2048;
constexpr int32_t kBucketMaxExperts = 1 << 24;

struct BucketPlan {
    int64_t slab;  // tokens per sweep and select launch
    int32_t nCp;   // floats per token of the coarse maxima
    size_t off_cd;  // d of the screening bounds, all tokens (the z pass writes it)
    size_t off_fine, off_coarse, off_fnorm, off_cnorm, bytes;
};

struct BucketArgs {
    const float* z;        // fp32 [T][r]
    const uint16_t* zhi;   // bf16(z) [T][r]
    const float* cz;       // screening scales c and d [T] (screen_scale, mean_scale)
    const float* cd;
    const uint16_t* R2t;
    int64_t T;
    int32_t r, M, k;
    bool pieces;           // exact logits as sums of eight products added up (closer to exact at long
                           // ranks), else as one chain, bit for bit as the resident route's
    int32_t* hist;         // nullable; cleared
    int32_t* idx;
    float *gate, *topval;  // topval nullable
};

// false when the shape is outside the route's limits.  beside: bytes that the caller keeps beside the
// route's scratch; up to 208 MB of them, the slab is chosen so that both stay within 240 MB.
bool bucket_make_plan(int64_t T, int32_t r, int32_t M, int32_t k, size_t beside, BucketPlan* plan);
hipError_t bucket_launch(const BucketPlan& plan, const BucketArgs& a, void* scratch,
                         hipStream_t stream);

}  // namespace more
