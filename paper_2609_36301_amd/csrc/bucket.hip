// Bucket route of the low-rank router (gfx950): softmax(TopK(x R1 R2)) with one matrix-core sweep
// over the expert axis and without the T x M logits in memory (Appendix "Pseudocode", inference
// algorithm; MoRE layer in "Preliminaries").  It follows the z pass and runs two launches per slab
// of tokens:
//
//   bucket_sweep_kernel   s_e = z_hi . u_e on the matrix cores; of each bucket of 16 experts only
//                         the maximum is kept (bf16, "fine"), and of every eight buckets the
//                         maximum in fp32 ("coarse");
//   bucket_select_kernel  one wave per token: the k-th largest coarse lower bound gives a
//                         threshold that k distinct experts provably reach; the fine maxima of the
//                         few coarse buckets that can hold an expert above it tighten it; the
//                         experts of the few fine buckets that still can are evaluated exactly in
//                         fp32 and ranked.
//
// Screening bounds.  With the token's scales c and d (route_device.h) and, over a bucket's experts,
// N >= ||u'|| and m >= |mu| of the rows u = mu 1 + u' (mu the row's mean), the logit lies within
// w = c N + d m of s_e.  (A per-expert offset, as a skewed load has, puts most of a long row's norm
// into mu, where only the sum of z's rounding errors meets it: with offsets of variance 0.5 at r 256,
// M 65536, k 8 a token has 10 fine buckets to read instead of 70, and 21 instead of 770 at most; 4096
// tokens 195 us a call instead of 980.  The selection at T 16384, r 64, M 65536: 71 us before, 40.)
// A bucket's maximum belongs to one of its
// experts, so the k largest of (maximum - w) over distinct buckets are reached by k distinct
// experts, and theta, the k-th of them, is a lower bound of the k-th logit.  An expert of the top k
// has l_e >= theta, so its bucket's maximum is at least theta - w: no other bucket is read.  The
// candidates' logits are evaluated as on the other routes (fp32 z times the bf16 row, rank entries in
// increasing order), and l >= theta keeps k or more of them, so the result is the exact top k
// under the total order (larger logit first, then smaller expert id) of the fp32 logits.
//
// Experts.  Super-group sg holds experts 256 sg .. 256 sg + 255 as eight MFMA tiles of 32; coarse
// bucket 2 sg + half holds the rows of lane half `half` of its tiles, fine bucket 8 (2 sg + half) + j
// those of tile j: experts 256 sg + 32 j + 8 (b >> 2) + 4 half + (b & 3), b = 0 .. 15.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bucket.h"
#include "device_common.h"
#include "route_device.h"

namespace more {

namespace {

// Value of a bucket without experts (rows past M): below every real lower bound, and finite, so
// that no bound computed from it is a NaN.
constexpr float kNoBucket = -0x1.8p127f;

constexpr int kSgTiles = 8;                  // MFMA tiles of a super-group
constexpr int kSgExperts = 32 * kSgTiles;    // 256
constexpr int kSweepWaves = 8;
constexpr int kSweepThreads = 64 * kSweepWaves;
static_assert(kSweepThreads == 2 * kSgExperts, "the norm bounds take two super-groups at a time");
constexpr int kSweepLds = 140 * 1024;        // expert rows of a workgroup

// Layout of the expert rows in LDS.  Powers of two keep the unpadded XOR swizzle of RouteCfg; other
// ranks are rounded up to RC chunks of 16 (the padding columns are zero in both operands) and
// the rows padded by 16 bytes, an odd number of 16-byte units, which also spreads the operand
// reads over all banks.
template <int RC>
struct SweepCfg {
    static constexpr bool POW2 = RC == 1 || RC == 2 || RC == 4;
    static constexpr int R = 16 * RC;
    static constexpr int STRIDE = POW2 ? R : R + 8;      // bf16 per row in LDS
    static constexpr int SPR = R / 8;                    // 16-byte segments per row
    // super-groups per workgroup: 128 KiB at the powers of two
    static constexpr int SG_FIT = kSweepLds / (2 * STRIDE * kSgExperts);
    static constexpr int SGS = POW2 ? 128 * 1024 / (2 * R * kSgExperts) : SG_FIT;
    static constexpr int DPS = SPR / 2;                  // loads per wave and super-group (POW2)
    static constexpr int TPW = RC <= 4 ? 4 : 2;          // token groups of 32 per wave
    // the token groups in two halves, one half's maxima taken while the other's MFMAs run; with
    // more rank chunks the operands of both leave no registers for it (the SIMD's other wave
    // fills the gap)
    static constexpr bool HALVES = RC <= 8;
    // coarse maxima are stored for four super-groups at a time (32 bytes per token)
    static constexpr bool QUADS = SGS >= 4;
    static_assert(SGS >= 1, "one super-group fits");
    __device__ static constexpr int pos(int e, int s) {  // position of segment s of row e
        return POW2 ? (s ^ ((e / (16 / (SPR < 16 ? SPR : 16))) % SPR)) : s;
    }
};

// N and m of one row from its fp32 sums of squares and of entries, both by chains of up to 128 bf16
// dot products rounding by 2^-22 each: 2^-13 of the square covers them (and any mu near the mean will do).
__device__ __forceinline__ float2 row_bounds(float ss, float su, float rinv) {
    const float mu = su * rinv;
    return make_float2(sqrtf(fmaf(ss, 0x1p-13f, fmaxf(fmaf(-su, mu, ss), 0.0f))) * (1.0f + 0x1p-20f),
                       fabsf(mu) * (1.0f + 0x1p-20f));
}
constexpr uint32_t kOnes = 0x3F803F80u;  // two bf16 ones

__device__ __forceinline__ float max16(const f32x16& a) {
    float m = fmaxf(fmaxf(a[0], a[1]), a[2]);
#pragma unroll
    for (int i = 3; i < 15; i += 2) m = fmaxf(fmaxf(m, a[i]), a[i + 1]);
    return fmaxf(m, a[15]);
}

// Grid: chunks x splits workgroups; a workgroup holds the rows of super-groups [s0, s1) of its
// chunk in LDS and sweeps them for its range of token blocks.  The 8 waves form 8 / ew token
// positions (TPW groups of 32 tokens each) times ew expert positions (position i takes
// super-groups s0 + i, s0 + i + ew, ...): ew > 1 keeps the waves busy when there are few tokens.
// Each A operand read from LDS feeds TPW MFMAs.  Per tile and token group the epilogue is eight
// v_max3 and half a pack, against RC MFMAs: the sweep is bound by the matrix cores.
// Measured (T 32768, r 64, M 16384): 61 us, 1.1 PFLOP/s, of which the stores of the maxima take 9 and
// the first loads of the rows 5; the two sweeps of the resident route (screen and collect) that
// it replaces took 66 + 88 us.  At r 16 the stores bound it: 1024 tokens, M 2^20 58 us, 168 MB of maxima
// (88 with the coarse ones going out 4 bytes at a time).
template <int RC>
__global__ __launch_bounds__(kSweepThreads, 2) void bucket_sweep_kernel(
    const uint16_t* __restrict__ zh, const uint16_t* __restrict__ R2t, int32_t T, int32_t r,
    int32_t M, int32_t chunks, int32_t splits, int32_t ew, int32_t unit, int32_t Tp, int32_t nCp,
    uint32_t* __restrict__ fine, float* __restrict__ coarse, float2* __restrict__ fnorm,
    float2* __restrict__ cnorm, int32_t* __restrict__ hist) {
    using C = SweepCfg<RC>;
    constexpr int TPW = C::TPW, H = C::HALVES ? TPW / 2 : TPW;
    __shared__ __attribute__((aligned(16))) uint16_t rows[C::SGS * kSgExperts * C::STRIDE];
    __shared__ float2 nred[2][16];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, half = lane >> 5;
    const int32_t chunk = (int32_t)(blockIdx.x % (unsigned)chunks);
    const int32_t split = (int32_t)(blockIdx.x / (unsigned)chunks);
    const int32_t nsg = (M + kSgExperts - 1) / kSgExperts;
    const int32_t nu = (nsg + unit - 1) / unit;
    const int32_t s0 = (int32_t)((int64_t)nu * chunk / chunks) * unit;
    const int32_t s1 = min((int32_t)((int64_t)nu * (chunk + 1) / chunks) * unit, nsg);
    const int nl = s1 - s0;
    if (hist)  // cleared for the histogram kernel (no memset: graph-safe)
        for (int64_t e = (int64_t)blockIdx.x * kSweepThreads + tid; e < M;
             e += (int64_t)gridDim.x * kSweepThreads)
            hist[e] = 0;

    const int tw = kSweepWaves / ew;                // token positions
    const int wt = w / ew, we = w % ew;
    const int btok = tw * 32 * TPW;                 // tokens per block
    const int32_t ntb = (T + btok - 1) / btok;
    const int32_t blk0 = (int32_t)((int64_t)ntb * split / splits);
    const int32_t blk1 = (int32_t)((int64_t)ntb * (split + 1) / splits);
    int off[RC];
#pragma unroll
    for (int c = 0; c < RC; ++c) off[c] = n * C::STRIDE + C::pos(n, 2 * c + half) * 8;
    // z_hi operands of a block.  Tokens past T re-read the last one (their maxima are not stored),
    // rank chunks past r a valid one (their expert columns are zero): no select, so that no
    // wait stands between these loads and the ones that follow.
    bf16x8 z[TPW][RC];
    auto load_z = [&](int32_t first) __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < TPW; ++g) {
            int32_t t = first + 32 * g + n;
            t = t < T ? t : T - 1;
#pragma unroll
            for (int c = 0; c < RC; ++c)
                z[g][c] = load_bf16x8(zh + (int64_t)t * r + (C::POW2 || 16 * c < r ? 16 * c + 8 * half : 0));
        }
    };
    // Waits for them and the loads before them.
    auto z_arrived = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
#pragma unroll
        for (int g = 0; g < TPW; ++g)
#pragma unroll
            for (int c = 0; c < RC; ++c) asm volatile("" : "+v"(z[g][c]));
    };

    // ---- rows of the chunk (rows past M re-read row M - 1; their maxima are masked below).
    if constexpr (C::POW2) {
        // direct-to-LDS loads: DPS per wave and super-group, 64 consecutive 16-byte slots each
        constexpr int DPS = C::DPS;
        for (int i = 0; i < nl; ++i) {
#pragma unroll
            for (int d = 0; d < DPS; ++d) {
                const int q = (w * DPS + d) * 64 + lane;  // slot in the super-group
                const int e = i * kSgExperts + q / C::SPR, p = q % C::SPR;
                int32_t ge = s0 * kSgExperts + e;
                ge = ge < M ? ge : M - 1;
                lds_dma16(R2t + (int64_t)ge * C::R + 8 * C::pos(e, p),
                          rows + (i * kSgExperts * C::SPR + (w * DPS + d) * 64) * 8);
            }
        }
        load_z(blk0 * btok + wt * 32 * TPW);
        z_arrived();
        lds_barrier();
    } else {
        load_z(blk0 * btok + wt * 32 * TPW);
        const int nseg = nl * kSgExperts * C::SPR;
        const int64_t e0 = (int64_t)s0 * kSgExperts;
        constexpr int UNR = 8;  // loads in flight per thread
        for (int base = 0; base < nseg; base += UNR * kSweepThreads) {
            u32x4 v[UNR];
#pragma unroll
            for (int i = 0; i < UNR; ++i) {
                int seg = base + i * kSweepThreads + tid;
                seg = seg < nseg ? seg : nseg - 1;
                const int e = seg / C::SPR, s = seg % C::SPR;
                int64_t ge = e0 + e;
                ge = ge < M ? ge : M - 1;
                const bool in = 8 * s < r;
                v[i] = *reinterpret_cast<const u32x4*>(R2t + ge * r + (in ? s * 8 : 0));
                if (!in) v[i] = u32x4{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int i = 0; i < UNR; ++i) {
                const int seg = base + i * kSweepThreads + tid;
                if (seg < nseg) {
                    const int e = seg / C::SPR, s = seg % C::SPR;
                    *reinterpret_cast<u32x4*>(rows + e * C::STRIDE + s * 8) = v[i];
                }
            }
        }
        __syncthreads();
    }

    // ---- token blocks
    for (int32_t blk = blk0; blk < blk1; ++blk) {
        const int32_t first = blk * btok + wt * 32 * TPW;
        if (first >= T) break;                      // wave-uniform
        if (blk > blk0) {
            load_z(first);
            z_arrived();
        }
        [[maybe_unused]] float last[TPW][3];        // coarse maxima of the three super-groups before
        for (int32_t s = s0 + we; s < s1; s += ew) {
            const uint16_t* sgrows = rows + (s - s0) * kSgExperts * C::STRIDE;
            bf16x8 a[RC];
            f32x16 acc[TPW];
            float hold[TPW], cm[TPW];
            uint32_t pk[TPW][kSgTiles / 2];
#pragma unroll
            for (int g = 0; g < TPW; ++g) cm[g] = kNoBucket;
            auto fetch = [&](auto jj) __attribute__((always_inline)) {
                constexpr int J = decltype(jj)::value;
#pragma unroll
                for (int c = 0; c < RC; ++c)
                    a[c] = load_bf16x8(sgrows + J * 32 * C::STRIDE + off[c]);
            };
            auto fetch4 = [&](auto jj, int c0) __attribute__((always_inline)) {
#pragma unroll
                for (int c = c0; c < c0 + 4; ++c)
                    a[c] = load_bf16x8(sgrows + decltype(jj)::value * 32 * C::STRIDE + off[c]);
            };
            // EDGE (the super-group that holds expert M - 1): rows past M start at kNoBucket, which
            // absorbs their products
            auto mfmas = [&](auto jj, auto hh, auto edge) __attribute__((always_inline)) {
                constexpr int J = decltype(jj)::value, G0 = decltype(hh)::value * H;
                f32x16 cin = zero_f32x16();
                if constexpr (decltype(edge)::value) {
                    const int32_t left = M - (s * kSgTiles + J) * 32 - 4 * half;  // rows below M
#pragma unroll
                    for (int b = 0; b < 16; ++b) cin[b] = 8 * (b >> 2) + (b & 3) < left ? 0.0f : kNoBucket;
                }
                if constexpr (!C::HALVES) fetch4(jj, 0);
#pragma unroll
                for (int g = G0; g < G0 + H; ++g) acc[g] = mfma_32x32x16(a[0], z[g][0], cin);
#pragma unroll
                for (int c = 1; c < RC; ++c) {
                    if constexpr (!C::HALVES)
                        if (c % 4 == 0) {
                            __builtin_amdgcn_sched_barrier(0);
                            fetch4(jj, c);
                        }
#pragma unroll
                    for (int g = G0; g < G0 + H; ++g)
                        acc[g] = mfma_32x32x16(a[c], z[g][c], acc[g]);
                }
            };
            // maxima of tile j of the super-group
            auto finish = [&](auto jj, auto hh) __attribute__((always_inline)) {
                constexpr int J = decltype(jj)::value, G0 = decltype(hh)::value * H;
#pragma unroll
                for (int g = G0; g < G0 + H; ++g) {
                    const float m = max16(acc[g]);
                    if constexpr ((J & 1) == 0) {
                        hold[g] = m;
                    } else {
                        const bf16x2 p = {(__bf16)hold[g], (__bf16)m};
                        pk[g][J / 2] = __builtin_bit_cast(uint32_t, p);
                        cm[g] = fmaxf(fmaxf(cm[g], hold[g]), m);
                    }
                }
            };
            using I0 = std::integral_constant<int, 0>;
            using I1 = std::integral_constant<int, 1>;
            auto tiles = [&](auto edge) __attribute__((always_inline)) {
                if constexpr (C::HALVES) fetch(I0{});
                unroll<kSgTiles>([&](auto jj) __attribute__((always_inline)) {
                    constexpr int J = decltype(jj)::value;
                    // the scheduler keeps each half tile together: moving loads and MFMAs of
                    // later tiles up would need more registers than there are
                    if constexpr (C::HALVES) {
                        mfmas(jj, I0{}, edge);
                        if constexpr (J > 0) finish(std::integral_constant<int, J - 1>{}, I1{});
                        __builtin_amdgcn_sched_barrier(0);
                        mfmas(jj, I1{}, edge);
                        if constexpr (J + 1 < kSgTiles) fetch(std::integral_constant<int, J + 1>{});
                        finish(jj, I0{});
                    } else {
                        mfmas(jj, I0{}, edge);
                        finish(jj, I0{});
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (C::HALVES)
                    finish(std::integral_constant<int, kSgTiles - 1>{}, I1{});
            };
            if ((s + 1) * kSgExperts > M)  // wave-uniform; rows past M lie in the last super-group
                tiles(std::true_type{});
            else
                tiles(std::false_type{});
#pragma unroll
            for (int g = 0; g < TPW; ++g) {
                const int32_t t = first + 32 * g + n;
                if (t < T) {
                    const uint32_t fo = ((uint32_t)s * (uint32_t)Tp + (uint32_t)t) * 8u + 4u * half;
                    *reinterpret_cast<u32x4*>(fine + fo) =
                        u32x4{pk[g][0], pk[g][1], pk[g][2], pk[g][3]};
                }
            }
            // Coarse maxima: where a wave takes four super-groups of a multiple of four in turn, the two
            // lane halves exchange theirs and each lane stores two of them.
            const bool quad = C::QUADS && ew == 1 && s1 - (s & ~3) >= 4 && (s & ~3) >= s0;
            if (!quad) {  // wave-uniform
#pragma unroll
                for (int g = 0; g < TPW; ++g) {
                    const int32_t t = first + 32 * g + n;
                    if (t < T) coarse[(uint32_t)t * (uint32_t)nCp + (uint32_t)(2 * s + half)] = cm[g];
                }
            } else if constexpr (C::QUADS) {
                if ((s & 3) == 3) {
#pragma unroll
                    for (int g = 0; g < TPW; ++g) {
                        const int32_t t = first + 32 * g + n;
                        float q[4] = {last[g][0], last[g][1], last[g][2], cm[g]};
                        lane_swap32(q[0], q[2]);
                        lane_swap32(q[1], q[3]);
                        if (t < T)
                            *reinterpret_cast<f32x4*>(coarse + (uint32_t)t * (uint32_t)nCp +
                                                      (uint32_t)(2 * (s - 3) + 4 * half)) =
                                f32x4{q[0], q[2], q[1], q[3]};
                    }
                }
#pragma unroll
                for (int g = 0; g < TPW; ++g) {
                    last[g][0] = last[g][1];
                    last[g][1] = last[g][2];
                    last[g][2] = cm[g];
                }
            }
        }
    }

    // ---- norm bounds of the buckets, two super-groups at a time; the splits share the chunk's.
    const float rinv = 1.0f / (float)r;
    const int part = tid / kSgExperts, row = tid % kSgExperts;  // (part is wave-uniform)
    for (int i0 = 2 * split; i0 < nl; i0 += 2 * splits) {       // workgroup-uniform
        if (i0 + part < nl) {
            const int e = (i0 + part) * kSgExperts + row;
            float ss = 0.0f, su = 0.0f;
#pragma unroll
            for (int sg = 0; sg < C::SPR; ++sg) {
                const bf16x8 v = load_bf16x8(rows + e * C::STRIDE + C::pos(e, sg) * 8);
#pragma unroll
                for (int q = 0; q < 8; q += 2) {
                    const bf16x2 pq = {v[q], v[q + 1]};
                    ss = __builtin_amdgcn_fdot2_f32_bf16(pq, pq, ss, false);
                    su = __builtin_amdgcn_fdot2_f32_bf16(pq, __builtin_bit_cast(bf16x2, kOnes), su, false);
                }
            }
            float2 nb = row_bounds(ss, su, rinv);
            // the 16 rows of a tile in the same lane half
            auto over = [&](auto d) __attribute__((always_inline)) {
                nb.x = fmaxf(nb.x, lane_xor<decltype(d)::value>(nb.x));
                nb.y = fmaxf(nb.y, lane_xor<decltype(d)::value>(nb.y));
            };
            over(std::integral_constant<int, 1>{});
            over(std::integral_constant<int, 2>{});
            over(std::integral_constant<int, 8>{});
            over(std::integral_constant<int, 16>{});
            if ((lane & 27) == 0) {
                const int f = ((row >> 2) & 1) * kSgTiles + (row >> 5);
                fnorm[(s0 + i0 + part) * 16 + f] = nb;
                nred[part][f] = nb;
            }
        }
        __syncthreads();
        if (tid < 4 && i0 + (tid >> 1) < nl) {
            const float2* half_nb = &nred[tid >> 1][(tid & 1) * kSgTiles];
            float2 m = half_nb[0];
#pragma unroll
            for (int q = 1; q < kSgTiles; ++q) {
                m.x = fmaxf(m.x, half_nb[q].x);
                m.y = fmaxf(m.y, half_nb[q].y);
            }
            cnorm[2 * (s0 + i0) + tid] = m;
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------ select
constexpr int kSelWaves = 4;
constexpr int kSelThreads = 64 * kSelWaves;
constexpr int kSelQ = 4;       // 16-byte pieces of the coarse row per lane and round
constexpr int kSelList = 256;  // listed coarse or fine buckets per token
constexpr int kSelFine = 4;    // fine values per lane and round
// Few tokens: a workgroup takes one, for a shorter chain of loads, against more work in all.  Whole calls,
// one token per workgroup / two per wave: M 16384, r 64, k 8: 30.4 / 31.9 us at 512 tokens, 33.0 / 32.8 at
// 1024, 36.6 / 34.5 at 1536; M 65536: 35.9 / 40.0 at 1024, 41.7 / 43.6, 48.7 / 45.4 at 2048; M 262144: 57 / 70,
// 72 / 81, 90 / 98; r 16 and 128, k 16 and 32 cross at the same sizes or a little later.
bool one_token_per_workgroup(int32_t T, int32_t M) { return T <= 1024 || (T <= 2048 && M >= 1 << 18); }

// Lanes per token: 32, two tokens per wave (the bookkeeping is bound by issue, and two tokens share
// it); the longest lists need the 64 lanes' maxima.  COOP: the four waves of a workgroup share one
// token (few tokens: the chain of loads of one token sets the time).
template <int K, bool COOP>
struct SelectCfg {
    static constexpr int LPT = COOP || K > 16 ? 64 : 32;      // of one wave
    static constexpr int TPW = 64 / LPT;                      // tokens per wave
    static constexpr int TOKENS = COOP ? 1 : kSelWaves * TPW; // tokens per workgroup
    static constexpr int NCAND = 128;                         // candidates evaluated exactly per token
};

// Of a token whose lists are long (the end of bucket_select_kernel); in the place of the lists of the
// tokens side by side, whose 32000 bytes at r 64 let five workgroups share a CU (another 1 KB, four of
// them: 60.2 us instead of 56.6 at T 32768, M 16384).
constexpr int kLongBuckets = 32;  // fine buckets per batch
template <int K>
struct LongLists {
    uint64_t fresh[kSelThreads];               // keys of a batch above the k-th best
    uint64_t best[K];                          // the largest so far, in order
    int32_t bucket[kSelThreads];               // fine buckets of a round and their upper bounds
    float bound[kSelThreads];
    int32_t cand[16 * kLongBuckets];           // experts of a batch and their upper bounds
    float cbound[16 * kLongBuckets];
    float wmax[kSelWaves][64];                 // lower bounds by wave and lane
};

// (logit, expert) as an integer that orders like the selection: larger logit first, then smaller
// expert id (-0 as +0).  Never 0 for an expert id.
__device__ __forceinline__ uint64_t selection_key(float l, int32_t e) {
    const uint32_t u = __builtin_bit_cast(uint32_t, l + 0.0f);
    const uint32_t o = u & 0x80000000u ? ~u : u | 0x80000000u;
    return ((uint64_t)o << 32) | (uint32_t)~e;
}
__device__ __forceinline__ float selection_logit(uint64_t key) {
    const uint32_t o = (uint32_t)(key >> 32);
    return __builtin_bit_cast(float, o & 0x80000000u ? o & 0x7FFFFFFFu : ~o);
}

// Lanes of a wave (as a 64-bit mask) that keep the larger value of their pair in a bitonic stage.
constexpr uint64_t sort_keeps_larger(int size, int d, int lpt) {
    uint64_t m = 0;
    for (int l = 0; l < 64; ++l)
        if (((l & d) == 0) == ((l & size) == 0 || size == lpt)) m |= 1ull << l;
    return m;
}

// x sorted descending across the LPT lanes of a token (lane 0 of it the largest): bitonic network;
// which value a lane keeps is a constant mask in scalar registers.
template <int LPT>
__device__ __forceinline__ float token_sort_desc(float x) {
    auto stage = [&](auto ss, auto dd) __attribute__((always_inline)) {
        constexpr int SIZE = decltype(ss)::value, D = decltype(dd)::value;
        constexpr uint64_t KEEP = sort_keeps_larger(SIZE, D, LPT);
        float a = x, b;
        if constexpr (D == 32) {
            lane_pair32(x, a, b);
        } else if constexpr (D == 16) {
            lane_pair16(x, a, b);
        } else {
            b = lane_xor<D>(x);
        }
        const float hi = fmaxf(a, b), lo = fminf(a, b);
        x = __builtin_amdgcn_inverse_ballot_w64(KEEP) ? hi : lo;
    };
    unroll<6>([&](auto i) __attribute__((always_inline)) {
        constexpr int SIZE = 2 << decltype(i)::value;
        if constexpr (SIZE <= LPT)
            unroll<decltype(i)::value + 1>([&](auto jj) __attribute__((always_inline)) {
                stage(std::integral_constant<int, SIZE>{},
                      std::integral_constant<int, ((SIZE / 2) >> decltype(jj)::value)>{});
            });
    });
    return x;
}

// Not infinite and not NaN, as an integer test: this file is compiled without NaNs in comparisons.
__device__ __forceinline__ bool finite(float x) {
    return (__builtin_bit_cast(uint32_t, x) & 0x7F800000u) != 0x7F800000u;
}

// The fine maxima are rounded to bf16: 2^-8 relative at most (and subnormals).
__device__ __forceinline__ float slack(float x) { return fmaf(fabsf(x), 0x1.01p-8f, 0x1p-125f); }

// The logit of the expert with row ur for the token with row zr (LDS): rank entries in increasing
// order (pieces: sums of eight, added up); ES segments of eight per step.
template <int ES>
__device__ __forceinline__ float exact_logit(const uint16_t* __restrict__ ur, const float* zr, int32_t r,
                                             bool pieces) {
    float l = 0.0f;
    for (int c0 = 0; c0 < r; c0 += 8 * ES) {
        const int ns = r - c0 < 8 * ES ? (r - c0) / 8 : ES;
        bf16x8 u[ES];
#pragma unroll
        for (int g = 0; g < ES; ++g) u[g] = load_bf16x8(ur + c0 + 8 * (g < ns ? g : 0));
#pragma unroll
        for (int g = 0; g < ES; ++g) {
            if (g < ns) {
                const f32x4 za = *reinterpret_cast<const f32x4*>(zr + c0 + 8 * g);
                const f32x4 zb = *reinterpret_cast<const f32x4*>(zr + c0 + 8 * g + 4);
                float p = pieces ? 0.0f : l;
#pragma unroll
                for (int t = 0; t < 4; ++t) p = fmaf(za[t], (float)u[g][t], p);
#pragma unroll
                for (int t = 0; t < 4; ++t) p = fmaf(zb[t], (float)u[g][4 + t], p);
                l = pieces ? l + p : p;
            }
        }
    }
    return l;
}

struct SelectArgs {
    const float* z;
    const uint16_t* zh;
    const float *cz, *cd;
    const uint16_t* R2t;
    const uint16_t* fine;
    const float* coarse;
    const float2 *fnorm, *cnorm;
    int32_t T, Tp, nCp, r, M, k;
    bool pieces;
    int32_t* idx;
    float *gate, *topval;
};

// Long lists: tokens with more buckets or experts near the threshold than the lists hold (bounds
// that are loose against the spacing of the logits, ties) go through the same tests again, the whole
// workgroup on one token: rounds of 32 coarse buckets, of whose fine ones up to 256 pass, and batches of
// 32 of those.  After each batch the threshold follows the k-th largest of the experts' own lower
// bounds (a row's norm comes with its product) and of the exact logits so far.
// Bound by the chain of a batch (about 8 us at r 256).  With a fifth of 4096 tokens coming here (r 256,
// M 65536, k 16, offsets of variance 0.5 against bounds by the whole norm) 1.25 ms a call, 14.3 with a
// sweep of all experts by a thread per row in its place; one such token among 16384 at r 64 made a
// call of 302 us take 750.
template <int SEG, int NS, bool EXACT, int K>
__device__ __forceinline__ void select_long(const SelectArgs& a, LongLists<K>& m, int32_t* found,
                                            const float* zr, float* ex, int32_t t, float theta,
                                            float cr, float dr) {
    constexpr int ES = 8 * SEG * NS < 64 ? SEG * NS : 8;  // segments per step of the exact sum
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t r = a.r, M = a.M, k = a.k, nC = 2 * ((M + kSgExperts - 1) / kSgExperts);
    constexpr int RPL = 64 / SEG;             // rows of a wave's load
    constexpr int BPW = NS == 1 ? 4 : 2;      // buckets per wave and step
    constexpr int LOADS = 16 * BPW / RPL;
    static_assert(LOADS >= 1 && kLongBuckets % (BPW * kSelWaves) == 0 && kLongBuckets * 16 <= 2 * kSelThreads &&
                  kSelThreads / kSgTiles == 32, "batches");
    const int seg = lane % SEG;
    const float rinv = 1.0f / (float)r;
    // place of a lane's entry in a list counted by found[q]
    auto put = [&](int q, bool in) __attribute__((always_inline)) {
        const uint64_t mask = __ballot(in);
        int b = 0;
        if (mask && lane == 0) b = atomicAdd(&found[q], (int)__popcll(mask));
        return __builtin_amdgcn_readfirstlane(b) +
               (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                              __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
    };
    const float c = a.cz[t], d = a.cd[t];
    // infinite or NaN bounds say nothing: every expert is evaluated
    bool every = !finite(c) || !finite(d) || !finite(cr) || !finite(dr);
    if (!finite(theta)) theta = 2.0f * kNoBucket;
    u32x4 zv[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) {
        const bool in = 8 * (SEG * q + seg) < r;
        zv[q] = *reinterpret_cast<const u32x4*>(a.zh + (int64_t)t * r + (in ? 8 * (SEG * q + seg) : 0));
        if (!in) zv[q] = u32x4{0u, 0u, 0u, 0u};
    }
    int nb = 0;                           // entries of best
    for (int attempt = 0; attempt < 2 && nb < k; ++attempt) {
        uint64_t least = 0;               // the k-th of them
        float lm = 2.0f * kNoBucket;      // this lane's largest lower bound
        for (int c0 = 0; c0 < nC; c0 += kSelThreads / kSgTiles) {
            __syncthreads();              // (bucket and found[0] are read no more)
            if (tid == 0) found[0] = 0;
            __syncthreads();
            {
                const int ci = c0 + tid / kSgTiles, f = c0 * kSgTiles + tid;
                bool pass = ci < nC;
                float ub = __builtin_inff();
                if (pass && !every) {
                    const float2 cb = a.cnorm[ci];
                    const float cu = a.coarse[(uint32_t)t * (uint32_t)a.nCp + (uint32_t)ci] +
                                     fmaf(d, cb.y, c * cb.x);
                    pass = cu >= theta;
                    // at best a tie with the k-th, and only larger ids than its
                    if (least && fmaf(fabsf(cu), 0x1p-20f, cu) <= selection_logit(least) &&
                        (ci >> 1) * kSgExperts > ~(int32_t)least)
                        pass = false;
                    if (pass) {
                        const float fv = bf16_bits_to_f32(
                            a.fine[(uint32_t)(ci >> 1) * (16u * (uint32_t)a.Tp) + 16u * (uint32_t)t +
                                   (uint32_t)(f & 15)]);
                        const float2 fb = a.fnorm[f];
                        ub = fv + slack(fv) + fmaf(d, fb.y, c * fb.x);
                        pass = ub >= theta;
                    }
                }
                const int o = put(0, pass);
                if (pass) {
                    m.bucket[o] = f;
                    m.bound[o] = ub;
                }
            }
            __syncthreads();
            const int n2 = found[0];
            for (int b0 = 0; b0 < n2; b0 += kLongBuckets) {
                if (tid == 0) found[1] = 0;
                __syncthreads();
                // rows of the batch, BPW buckets per wave at a time
                const int be = b0 + kLongBuckets < n2 ? b0 + kLongBuckets : n2;
                int turn = 0;
                for (int bw = b0 + BPW * w; bw < be; bw += BPW * kSelWaves) {  // wave-uniform
                    u32x4 u[LOADS][NS];
                    int32_t er[LOADS];
                    bool live[LOADS];
#pragma unroll
                    for (int i = 0; i < LOADS; ++i) {
                        const int q = i * RPL + lane / SEG, b = q % 16;
                        const int bi = bw + q / 16 < be ? bw + q / 16 : bw;
                        const int f = m.bucket[bi];
                        er[i] = (f >> 4) * kSgExperts + (f & 7) * 32 + 4 * ((f >> 3) & 1) +
                                8 * (b >> 2) + (b & 3);
                        live[i] = bw + q / 16 < be && er[i] < M && (every || m.bound[bi] >= theta);
                        const uint16_t* ur = a.R2t + (uint32_t)(live[i] ? er[i] : 0) * (uint32_t)r;
#pragma unroll
                        for (int q2 = 0; q2 < NS; ++q2) {
                            const int col = 8 * (SEG * q2 + seg);
                            u[i][q2] = *reinterpret_cast<const u32x4*>(ur + (EXACT || col < r ? col : 0));
                        }
                    }
#pragma unroll
                    for (int i = 0; i < LOADS; ++i) {
                        float s = 0.0f, ss = 0.0f, su = 0.0f;  // z_hi . u, u . u and u . 1
#pragma unroll
                        for (int q2 = 0; q2 < NS; ++q2) {
                            const bool in = EXACT || 8 * (SEG * q2 + seg) < r;
#pragma unroll
                            for (int d = 0; d < 4; ++d) {
                                const uint32_t ud = in ? u[i][q2][d] : 0u, zd = zv[q2][d];
                                const bf16x2 up = __builtin_bit_cast(bf16x2, ud);
                                s = __builtin_amdgcn_fdot2_f32_bf16(up, __builtin_bit_cast(bf16x2, zd), s,
                                                                    false);
                                ss = __builtin_amdgcn_fdot2_f32_bf16(up, up, ss, false);
                                su = __builtin_amdgcn_fdot2_f32_bf16(
                                    up, __builtin_bit_cast(bf16x2, kOnes), su, false);
                            }
                        }
                        unroll<SEG == 8 ? 3 : (SEG == 4 ? 2 : 1)>([&](auto st) __attribute__((always_inline)) {
                            s += lane_xor<1 << decltype(st)::value>(s);
                            ss += lane_xor<1 << decltype(st)::value>(ss);
                            su += lane_xor<1 << decltype(st)::value>(su);
                        });
                        const float2 own = row_bounds(ss, su, rinv);
                        const float e = fmaf(dr, own.y, cr * own.x);
                        // the row's lanes keep the lower bounds in turn: 64 distinct experts
                        if (live[i] && (turn + i) % SEG == seg) lm = fmaxf(lm, s - e);
                        const bool pass = seg == 0 && live[i] && (every || s + e >= theta);
                        const int o = put(1, pass);
                        if (pass) {
                            m.cand[o] = er[i];
                            m.cbound[o] = s + e;
                        }
                    }
                    turn += LOADS;
                }
                m.wmax[w][lane] = lm;
                __syncthreads();
                const int n3 = found[1];
                float top = m.wmax[0][lane];
#pragma unroll
                for (int i = 1; i < kSelWaves; ++i) top = fmaxf(top, m.wmax[i][lane]);
                top = __shfl(token_sort_desc<64>(top), k - 1, kWave);
                if (finite(top)) theta = fmaxf(theta, top - fabsf(top) * 0x1p-20f);
                // exact logits, a thread each
                for (int i0 = 0; i0 < n3; i0 += kSelThreads) {  // workgroup-uniform
                    if (tid == 0) found[2] = 0;
                    __syncthreads();
                    const int i = i0 + tid;
                    uint64_t mine = 0;
                    if (i < n3 && (every || m.cbound[i] >= theta)) {
                        const int32_t e = m.cand[i];
                        mine = selection_key(
                            exact_logit<ES>(a.R2t + (uint32_t)e * (uint32_t)r, zr, r, a.pieces), e);
                    }
                    const bool pass = mine > least;  // (never for a thread without an expert)
                    const int o = put(2, pass);
                    if (pass) m.fresh[o] = mine;
                    __syncthreads();
                    const int nf = found[2];
                    if (nf) {  // workgroup-uniform: merged into the best by counting
                        uint64_t last = 0;
                        int rank = 0, rank2 = 0;
                        mine = tid < nf ? m.fresh[tid] : 0;
                        last = tid < nb ? m.best[tid] : 0;
#pragma unroll 4
                        for (int q = 0; q < nf; ++q) {
                            const uint64_t v = m.fresh[q];
                            rank += v > mine ? 1 : 0;
                            rank2 += v > last ? 1 : 0;
                        }
                        for (int q = 0; q < nb; ++q) rank += m.best[q] > mine ? 1 : 0;
                        rank2 += tid;
                        __syncthreads();
                        if (tid < nf && rank < k) m.best[rank] = mine;
                        if (tid < nb && rank2 < k) m.best[rank2] = last;
                        nb = nf + nb < k ? nf + nb : k;
                        __syncthreads();
                        if (nb == k) {
                            least = m.best[k - 1];
                            const float l = selection_logit(least);
                            if (finite(l)) theta = fmaxf(theta, l - fabsf(l) * 0x1p-20f);
                        }
                    }
                }
            }
        }
        // fewer than k (bounds spoilt by an overflow): once more without them
        if (nb < k) {
            every = true;
            nb = 0;
        }
    }
    __syncthreads();
    if (tid < k) {
        const float l = selection_logit(m.best[tid]);
        a.idx[(int64_t)t * k + tid] = ~(int32_t)m.best[tid];
        if (a.topval) a.topval[(int64_t)t * k + tid] = l;
        ex[tid] = expf(l - selection_logit(m.best[0]));
    }
    __syncthreads();
    if (tid < k) {
        float sum = 0.0f;  // in rank order
        for (int i = 0; i < k; ++i) sum += ex[i];
        a.gate[(int64_t)t * k + tid] = ex[tid] / sum;
    }
}

// Steps of a wave, for its tokens side by side (tk = lane / LPT, sub = lane % LPT):
//  1. theta = the k-th largest of the token's lanes' largest coarse lower bounds;
//  2. the coarse buckets whose upper bound reaches theta are listed;
//  3. their fine maxima raise theta in the same way, and the fine buckets whose upper bound
//     reaches it are listed;
//  4. refine: SEG lanes read a row of 16 SEG bytes together (whole lines; NS times for longer
//     rows) and form z_hi . u_e with bf16 dot products; a round of SEG loads leaves one row's
//     value in each lane, and the experts whose upper bound reaches theta are listed;
//  5. those (k and a few) are evaluated exactly, a lane each, the ones with l >= theta ranked.
// A token whose lists overflow (bounds that are loose against the spacing of the logits, ties) is
// taken by the whole workgroup at the end.  8 SEG NS >= r (EXACT: equal to r); K >= k.
// Bound by issue and by the rows' reads (r 64, M 16384: 10 buckets, 20 KB per token from L2; 32768
// tokens in 53 us; 59 with 64-bit addresses, a reduction per row and ranks by (logit, id) pairs,
// 92 with the rows staged in LDS, 127 with exact sums for all of them and a token per wave).
template <int SEG, int NS, bool EXACT, int K, bool COOP>
__global__ __launch_bounds__(kSelThreads) void bucket_select_kernel(const SelectArgs args) {
    const float* __restrict__ const z = args.z;
    const uint16_t* __restrict__ const zh = args.zh;
    const uint16_t* __restrict__ const R2t = args.R2t;
    const uint16_t* __restrict__ const fine = args.fine;
    const float* __restrict__ const coarse = args.coarse;
    const float2* __restrict__ const fnorm = args.fnorm;
    const float2* __restrict__ const cnorm = args.cnorm;
    const int32_t T = args.T, Tp = args.Tp, nCp = args.nCp, r = args.r, M = args.M, k = args.k;
    const bool pieces = args.pieces;
    int32_t* __restrict__ const idx = args.idx;
    float* __restrict__ const gate = args.gate;
    float* __restrict__ const topval = args.topval;
    using C = SelectCfg<K, COOP>;
    constexpr int LPT = C::LPT, TPW = C::TPW, NCAND = C::NCAND, TOKENS = C::TOKENS;
    constexpr int LANES = COOP ? kSelThreads : LPT;  // lanes of a token in all
    constexpr int ZMAX = 8 * SEG * NS;        // >= r
    constexpr uint32_t RS = 8 * SEG * NS;     // r when EXACT
    constexpr int ES = ZMAX < 64 ? ZMAX / 8 : 8;  // segments per step of the exact sum
    __shared__ __attribute__((aligned(16))) float zrow[TOKENS][ZMAX];
    struct Lists {
        uint64_t key[TOKENS][NCAND];          // candidates at or above theta
        int32_t list1[TOKENS][kSelList];
        int32_t list2[TOKENS][kSelList];
        int32_t list3[TOKENS][NCAND];
        float wmax[COOP ? 2 : 1][COOP ? kSelWaves : 1][COOP ? 64 : 1];
    };
    __shared__ union {
        Lists lists;                          // of the tokens side by side
        LongLists<K> one;                     // of one token, at the end
    } mem;
    auto& key = mem.lists.key;
    auto& list1 = mem.lists.list1;
    auto& list2 = mem.lists.list2;
    auto& list3 = mem.lists.list3;
    auto& wmax = mem.lists.wmax;
    __shared__ float over_theta[TOKENS], over_cr[TOKENS], over_dr[TOKENS];
    __shared__ int32_t found[4];              // COOP: entries of the four lists
    __shared__ float ex[TOKENS][K];
    __shared__ int32_t over_tok[TOKENS];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tk = lane / LPT;
    const int sub = lane % LPT;               // lane within the token's part of this wave
    const int gl = COOP ? 64 * w + lane : sub;  // ... and of all its lanes
    const int j = COOP ? 0 : w * TPW + tk;    // the token's place in the workgroup
    const int32_t tok0 = (int32_t)blockIdx.x * TOKENS + (COOP ? 0 : w * TPW);
    const int32_t tok = tok0 + tk;
    const bool ok = tok < T;
    const int32_t nC = 2 * ((M + kSgExperts - 1) / kSgExperts);
    bool over = false;
    if (COOP && threadIdx.x < 4) found[threadIdx.x] = 0;  // (kth's barrier comes before their use)
    if (tok0 < T) {  // wave-uniform (COOP: always)
        const int32_t tc = ok ? tok : T - 1;  // a wave's second token may lie past T
        const float c = args.cz[tc], d = args.cd[tc];
        float zn = 0.0f;                      // ||z||, for the rounding of the bf16 dot products
        uint32_t bits = 0;
        for (int i = 4 * sub; i < r; i += 4 * LPT) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(z + (int64_t)tc * r + i);
            if (!COOP || w == 0) *reinterpret_cast<f32x4*>(&zrow[j][i]) = v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                zn = fmaf(v[e], v[e], zn);
                bits |= __builtin_bit_cast(uint32_t, v[e]) << 1;  // 0 for +-0 alone
            }
        }
        // lanes of the token set in mask: those below this lane, and all
        auto below = [&](uint64_t mask) __attribute__((always_inline)) {
            if constexpr (LPT == 64)
                return (int)__builtin_amdgcn_mbcnt_hi(
                    (uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
            const uint32_t part = tk ? (uint32_t)(mask >> 32) : (uint32_t)mask;
            return __builtin_popcount(part & ((1u << sub) - 1u));
        };
        auto all = [&](uint64_t mask) __attribute__((always_inline)) {
            if constexpr (LPT == 64) return (int)__popcll(mask);
            return __builtin_popcount(tk ? (uint32_t)(mask >> 32) : (uint32_t)mask);
        };
        // z = 0 (a padding token): every logit is 0 and the smallest ids win.  Nothing is listed for
        // it; through the lists it would be a tie of all experts, and the sweep at the end.
        // (30% such tokens at T 4096, h 128, r 128, M 8192: 865 us a call that way, 44 this way).
        const bool zero = all(__ballot(bits != 0)) == 0;
        // LDS written by the token's lanes is read by them
        auto sync = [&]() __attribute__((always_inline)) {
            if constexpr (COOP)
                __syncthreads();  // workgroup-uniform: one token, no early exit
            else
                wave_lds_sync();
        };
        // place of this lane's entry in list L (n entries so far); `more` entries are added
        auto place = [&](auto L, uint64_t mask, int& n) __attribute__((always_inline)) {
            int base = n;
            if constexpr (COOP) {
                int b = 0;
                if (lane == 0) b = atomicAdd(&found[decltype(L)::value], (int)__popcll(mask));
                base = __builtin_amdgcn_readfirstlane(b);
            } else {
                n += all(mask);
            }
            return base + below(mask);
        };
        // after the list is complete: its number of entries
        auto total = [&](auto L, int n) __attribute__((always_inline)) {
            sync();
            return COOP ? found[decltype(L)::value] : n;
        };
        using L0 = std::integral_constant<int, 0>;
        using L1 = std::integral_constant<int, 1>;
        using L2 = std::integral_constant<int, 2>;
        using L3 = std::integral_constant<int, 3>;
        // the largest of a count over the wave's tokens
        auto most = [&](int n) __attribute__((always_inline)) {
            const int a = __builtin_amdgcn_readlane(n, 0);
            if constexpr (TPW == 1) return a;
            const int b = __builtin_amdgcn_readlane(n, LPT);
            return a > b ? a : b;
        };
        // the k-th largest of the lanes' values (COOP: of the 64 maxima over the waves), guarded
        auto kth = [&](auto call, float x) __attribute__((always_inline)) {
            if constexpr (COOP) {
                constexpr int B = decltype(call)::value;
                wmax[B][w][lane] = x;
                __syncthreads();
#pragma unroll
                for (int i = 0; i < kSelWaves; ++i) x = fmaxf(x, wmax[B][i][lane]);
            }
            const float s = token_sort_desc<LPT>(x);
            const float t = __shfl(s, (lane & ~(LPT - 1)) + k - 1, kWave);
            return t - fabsf(t) * 0x1p-20f;
        };
        // ---- 1. and 2. coarse maxima
        constexpr int PIECE = 4 * LANES, ROUND = kSelQ * PIECE;
        const float* crow = coarse + (uint32_t)tc * (uint32_t)nCp;
        const int nround = (nC + ROUND - 1) / ROUND;
        f32x4 q[kSelQ], nq[kSelQ][2];
        auto load_round = [&](int rd) __attribute__((always_inline)) {
#pragma unroll
            for (int m = 0; m < kSelQ; ++m) {
                const int i = rd * ROUND + PIECE * m + 4 * gl;
                if (rd * ROUND + PIECE * m < nC) {  // wave-uniform
                    const int ii = i < nC ? i : 0;
                    q[m] = *reinterpret_cast<const f32x4*>(crow + ii);
                    nq[m][0] = *reinterpret_cast<const f32x4*>(cnorm + ii);
                    nq[m][1] = *reinterpret_cast<const f32x4*>(cnorm + ii + 2);
                }
            }
        };
        // f(value, w, bucket, valid) for the round's coarse buckets
        auto scan = [&](int rd, auto&& f) __attribute__((always_inline)) {
#pragma unroll
            for (int m = 0; m < kSelQ; ++m) {
                if (rd * ROUND + PIECE * m < nC) {
                    const int i = rd * ROUND + PIECE * m + 4 * gl;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        f(q[m][e], fmaf(d, nq[m][e / 2][2 * (e & 1) + 1], c * nq[m][e / 2][2 * (e & 1)]),
                          i + e, i + e < nC);
                }
            }
        };
        float lm = 2.0f * kNoBucket;  // (-inf)
        for (int rd = 0; rd < nround; ++rd) {
            load_round(rd);
            scan(rd, [&](float v, float cn, int, bool valid) __attribute__((always_inline)) {
                const float lb = v - cn;
                lm = fmaxf(lm, valid ? lb : lm);
            });
        }
        float theta = kth(L0{}, lm);
        theta = zero ? __builtin_inff() : theta;
        int n1 = 0;
        for (int rd = 0; rd < nround; ++rd) {
            if (nround > 1) load_round(rd);
            scan(rd, [&](float v, float cn, int i, bool valid) __attribute__((always_inline)) {
                const bool pass = valid && v + cn >= theta;
                const uint64_t mask = __ballot(pass);
                if (mask) {
                    const int p = place(L0{}, mask, n1);
                    if (pass && p < kSelList) list1[j][p] = i;
                }
            });
        }
        n1 = total(L0{}, n1);
        over = n1 > kSelList;
        n1 = over ? 0 : n1;
        // ---- 3. fine maxima: eight lanes per coarse bucket
        constexpr int FPR = LANES / 8;           // coarse buckets per token and value
        const int n1m = most(n1);
        const int fround = (n1m + FPR * kSelFine - 1) / (FPR * kSelFine);
        float v[kSelFine], cn[kSelFine];
        int id[kSelFine];
        const uint32_t fstride = 16u * (uint32_t)Tp;                        // of a super-group
        const uint32_t fbase = 16u * (uint32_t)tc + (uint32_t)(sub & 7);    // token and tile
        auto load_fine = [&](int rd) __attribute__((always_inline)) {
#pragma unroll
            for (int m = 0; m < kSelFine; ++m) {
                const int p = (rd * kSelFine + m) * FPR + (gl >> 3);
                const int ci = list1[j][p < n1 ? p : 0];
                id[m] = p < n1 ? ci * kSgTiles + (sub & 7) : -1;
                const int cc = p < n1 ? ci : 0;
                // (the maxima of a slab take less than 2^32 bytes)
                const uint32_t fo = (uint32_t)(cc >> 1) * fstride + 8u * (cc & 1) + fbase;
                v[m] = bf16_bits_to_f32(fine[fo]);
                const float2 nb = fnorm[(uint32_t)(cc * kSgTiles + (sub & 7))];
                cn[m] = fmaf(d, nb.y, c * nb.x);
            }
        };
        float fm = 2.0f * kNoBucket;
        for (int rd = 0; rd < fround; ++rd) {
            load_fine(rd);
#pragma unroll
            for (int m = 0; m < kSelFine; ++m) {
                const float lb = v[m] - slack(v[m]) - cn[m];
                fm = fmaxf(fm, id[m] >= 0 ? lb : fm);
            }
        }
        theta = fmaxf(theta, kth(L1{}, fm));
        int n2 = 0;
        for (int rd = 0; rd < fround; ++rd) {
            if (fround > 1) load_fine(rd);
#pragma unroll
            for (int m = 0; m < kSelFine; ++m) {
                const bool pass = id[m] >= 0 && v[m] + slack(v[m]) + cn[m] >= theta;
                const uint64_t mask = __ballot(pass);
                if (mask) {
                    const int o = place(L1{}, mask, n2);
                    if (pass && o < kSelList) list2[j][o] = id[m];
                }
            }
        }
        n2 = total(L1{}, n2);
        over = over || n2 > kSelList;
        n2 = over ? 0 : n2;
        // ||z|| over the token's lanes
        zn += lane_xor<1>(zn);
        zn += lane_xor<2>(zn);
        zn += lane_xor<4>(zn);
        zn += lane_xor<8>(zn);
        zn += lane_xor<16>(zn);
        if constexpr (LPT == 64) zn += lane_xor<32>(zn);
        // a chain of r / 2 dot products, each rounded to 2^-22 relative at worst, against
        // ||u|| <= N + sqrt(r) m
        const float cr = fmaf(sqrtf(zn), 0x1p-14f, c), dr = fmaf(sqrtf(zn * (float)r), 0x1p-14f, d);
        if (COOP ? threadIdx.x == 0 : sub == 0) {
            over_theta[j] = theta;
            over_cr[j] = cr;
            over_dr[j] = dr;
        }
        // ---- 4. refine
        constexpr int BPR = LPT / 16;            // buckets per token and round
        constexpr int RPT = LPT / SEG;           // rows of a token per load
        constexpr int ITB = 16 / RPT;            // loads per bucket
        static_assert(RPT <= 16 && BPR * ITB == SEG, "a round is SEG loads, one row per lane");
        const int nr2 = (most(n2) + BPR - 1) / BPR;
        // row of the bucket that load it brings to this lane, as an offset from the bucket's base
        auto row_of = [](int it, int grp) __attribute__((always_inline)) {
            const int b = it * RPT + grp;
            return 8 * (b >> 2) + (b & 3);
        };
        const int seg = sub % SEG, grp = sub / SEG;
        u32x4 zv[NS];                            // z_hi, this lane's segments
#pragma unroll
        for (int c = 0; c < NS; ++c) {
            const bool in = 8 * (SEG * c + seg) < r;
            zv[c] = *reinterpret_cast<const u32x4*>(
                zh + (int64_t)tc * r + (in ? 8 * (SEG * c + seg) : 0));
            if (!in) zv[c] = u32x4{0u, 0u, 0u, 0u};
        }
        int n3 = 0;
        for (int rd = COOP ? w : 0; rd < nr2; rd += COOP ? kSelWaves : 1) {
            int32_t eb[BPR];
            int f[BPR];
            bool edge = false;
#pragma unroll
            for (int q = 0; q < BPR; ++q) {
                const int bi = rd * BPR + q;
                f[q] = list2[j][bi < n2 ? bi : 0];
                f[q] = n2 > 0 ? f[q] : 0;
                eb[q] = (f[q] >> 4) * kSgExperts + (f[q] & 7) * 32 + 4 * ((f[q] >> 3) & 1);
                edge = edge || eb[q] + 28 > M;
            }
            // this lane's own row: load seg of the round
            int fo = f[0];
            int32_t eo = eb[0];
#pragma unroll
            for (int q = 1; q < BPR; ++q) {
                fo = seg >= q * ITB ? f[q] : fo;
                eo = seg >= q * ITB ? eb[q] : eo;
            }
            eo += row_of(seg % ITB, grp);
            const float2 nb = fnorm[fo];
            const bool live = rd * BPR + seg / ITB < n2 && eo < M;
            float s = 0.0f;
            // byte offsets fit 32 bits; of a bucket's rows only the first is computed where the row
            // stride is a constant (the others follow at constant distances)
            auto rows = [&](auto clamp) __attribute__((always_inline)) {
                u32x4 u[SEG][NS];
#pragma unroll
                for (int i = 0; i < SEG; ++i) {
                    uint32_t base;
                    int ahead = 0;
                    if constexpr (decltype(clamp)::value) {
                        const int32_t er = eb[i / ITB] + row_of(i % ITB, grp);
                        base = (uint32_t)(er < M ? er : M - 1) * (2u * (uint32_t)r);
                    } else if constexpr (EXACT && RPT % 4 == 0) {
                        // row_of(it, grp) = row_of(0, grp) + 2 RPT it: whole groups of four rows
                        base = (uint32_t)(eb[i / ITB] + row_of(0, grp)) * (2u * RS);
                        ahead = (i % ITB) * 2 * RPT * 2 * RS;
                    } else {
                        base = (uint32_t)(eb[i / ITB] + row_of(i % ITB, grp)) * (2u * (uint32_t)r);
                    }
                    const char* rowp = reinterpret_cast<const char*>(R2t) + base;
#pragma unroll
                    for (int c = 0; c < NS; ++c) {
                        if constexpr (EXACT) {
                            u[i][c] = *reinterpret_cast<const u32x4*>(
                                reinterpret_cast<const char*>(R2t) + (base + 16u * seg) + ahead +
                                16 * SEG * c);
                        } else {
                            // (segments past the rank re-read the row's first, against a zero z)
                            const int col = 8 * (SEG * c + seg);
                            u[i][c] = *reinterpret_cast<const u32x4*>(rowp + 2 * (col < r ? col : 0));
                        }
                    }
                }
                float t[SEG];
#pragma unroll
                for (int i = 0; i < SEG; ++i) {
                    t[i] = 0.0f;
#pragma unroll
                    for (int c = 0; c < NS; ++c)
#pragma unroll
                        for (int d = 0; d < 4; ++d) {
                            const uint32_t ud = u[i][c][d], zd = zv[c][d];
                            t[i] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, ud),
                                                                   __builtin_bit_cast(bf16x2, zd),
                                                                   t[i], false);
                        }
                }
                // sums over the SEG lanes of a row, load i's ending up in lane seg = i: at each step
                // a lane keeps one of a pair of values and adds the other lane's part of it
                unroll<SEG == 8 ? 3 : (SEG == 4 ? 2 : 1)>([&](auto st) __attribute__((always_inline)) {
                    constexpr int D = 1 << decltype(st)::value;
                    const bool up = (seg & D) != 0;
#pragma unroll
                    for (int i = 0; i < SEG; i += 2 * D) {
                        const float keep = up ? t[i + D] : t[i], give = up ? t[i] : t[i + D];
                        t[i] = keep + lane_xor<D>(give);
                    }
                });
                s = t[0];
            };
            if (__ballot(edge))
                rows(std::true_type{});
            else
                rows(std::false_type{});
            const bool pass = live && fmaf(cr, nb.x, fmaf(dr, nb.y, s)) >= theta;
            const uint64_t mask = __ballot(pass);
            if (mask) {
                const int o = place(L2{}, mask, n3);
                if (pass && o < NCAND) list3[j][o] = eo;
            }
        }
        n3 = total(L2{}, n3);
        over = over || n3 > NCAND;
        n3 = over ? 0 : n3;
        // ---- 5. exact logits, a lane each; those >= theta are kept
        const int n3m = most(n3);
        int nc = 0;
        for (int i0 = 0; i0 < n3m; i0 += LANES) {
            const int i = i0 + gl;
            const int32_t e = i < n3 ? list3[j][i] : 0;
            const float l = exact_logit<ES>(R2t + (uint32_t)e * (uint32_t)r, zrow[j], r, pieces);
            const bool pass = i < n3 && l >= theta;
            const uint64_t mask = __ballot(pass);
            const int o = place(L3{}, mask, nc);  // at most n3 in all
            if (pass) key[j][o] = selection_key(l, e);
        }
        nc = total(L3{}, nc);
        // fewer than k cannot happen (k experts reach theta); the test is a guard, not a path
        over = (over || nc < k) && !zero;
        // nor do bounds that are infinite or NaN count for anything (d is, wherever z is)
        over = over || !finite(d) || !finite(cr) || !(zero || finite(theta));
        nc = over ? 0 : nc;
        // rank of each candidate by counting; ranks below k write their output slot
        const int ncm = most(nc);
        for (int i = nc + gl; i < ncm; i += LANES) key[j][i] = 0;  // (of the wave's other token: no rank)
        if constexpr (!COOP) wave_lds_sync();
        for (int i0 = 0; i0 < ncm; i0 += LANES) {
            const uint64_t mine = key[j][i0 + gl < nc ? i0 + gl : 0];
            int rank = 0;
#pragma unroll 4
            for (int t = 0; t < ncm; ++t) rank += key[j][t] > mine ? 1 : 0;
            if (ok && i0 + gl < nc && rank < k) {
                const float l = selection_logit(mine);
                idx[(int64_t)tok * k + rank] = ~(int32_t)mine;
                if (topval) topval[(int64_t)tok * k + rank] = l;
                ex[j][rank] = l;
            }
        }
        if (ok && zero && gl < k) {
            idx[(int64_t)tok * k + gl] = gl;
            if (topval) topval[(int64_t)tok * k + gl] = 0.0f;
            ex[j][gl] = 0.0f;
        }
        sync();
        const float mine = expf(ex[j][gl < k ? gl : 0] - ex[j][0]);
        sync();
        if (gl < k) ex[j][gl] = mine;
        sync();
        float sum = 0.0f;  // in rank order, as store_selection
        for (int i = 0; i < k; ++i) sum += ex[j][i];
        if (ok && !over && gl < k) gate[(int64_t)tok * k + gl] = mine / sum;
    }
    over = ok && over;
    if (COOP ? threadIdx.x == 0 : sub == 0) over_tok[j] = over;
    if (!__syncthreads_or(over)) return;  // workgroup-uniform
    // The arguments are read again: held in registers over the steps above they would be spilled there
    // (T 32768, r 64, M 16384: 61.6 us, 60.2 so).
    auto kernarg = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(kernarg));
    const SelectArgs& again = *(const SelectArgs*)kernarg;
    for (int jt = 0; jt < TOKENS; ++jt)
        if (over_tok[jt])  // workgroup-uniform
            select_long<SEG, NS, EXACT, K>(again, mem.one, found, zrow[jt], ex[jt],
                                           (int32_t)blockIdx.x * TOKENS + jt, over_theta[jt], over_cr[jt],
                                           over_dr[jt]);
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Rank chunks the sweep is compiled for.
int sweep_rc(int32_t r) {
    const int rc = r / 16;
    return rc <= 4 ? rc : (rc <= 6 ? 6 : (rc <= 8 ? 8 : (rc <= 12 ? 12 : 16)));
}

template <int RC>
void sweep_shape(int32_t* sgs, int32_t* wave_tokens) {
    *sgs = SweepCfg<RC>::SGS;
    *wave_tokens = 32 * SweepCfg<RC>::TPW;
}

void sweep_limits(int rc, int32_t* sgs, int32_t* wave_tokens) {
    switch (rc) {
        case 1: return sweep_shape<1>(sgs, wave_tokens);
        case 2: return sweep_shape<2>(sgs, wave_tokens);
        case 3: return sweep_shape<3>(sgs, wave_tokens);
        case 4: return sweep_shape<4>(sgs, wave_tokens);
        case 6: return sweep_shape<6>(sgs, wave_tokens);
        case 8: return sweep_shape<8>(sgs, wave_tokens);
        case 12: return sweep_shape<12>(sgs, wave_tokens);
        default: return sweep_shape<16>(sgs, wave_tokens);
    }
}

// Bytes of the maxima of one token (16 fine values of two bytes and two coarse of four per
// super-group).
size_t token_bytes(int32_t nsg) { return (size_t)nsg * 40 + 16; }

constexpr size_t kMaximaBytes = (size_t)208 << 20;    // largest slab: within the 256 MB last-level cache
constexpr size_t kMaximaLeast = (size_t)32 << 20;
constexpr size_t kScratchAim = (size_t)240 << 20;     // with what is beside them, while that leaves kMaximaLeast

struct SweepGrid {
    int32_t chunks, splits, ew, unit;
};

// Work split of a sweep over T tokens: as few expert chunks as fit LDS while there are 256
// workgroups (one per CU), else smaller chunks; with few tokens the waves of a workgroup share the
// token block and split the super-groups.
SweepGrid sweep_grid(int32_t rc, int32_t T, int32_t nsg) {
    SweepGrid g;
    int32_t sgs, wt;
    sweep_limits(rc, &sgs, &wt);
    g.ew = 1;
    while (g.ew < kSweepWaves && (kSweepWaves / (2 * g.ew)) * wt >= T && 2 * g.ew <= sgs) g.ew *= 2;
    const int32_t btok = kSweepWaves / g.ew * wt;
    const int32_t ntb = (T + btok - 1) / btok;
    const int32_t want = (256 + ntb - 1) / ntb;
    // super-groups times token blocks of the largest workgroup, with chunks of whole units
    auto split = [&](int32_t unit) {
        const int32_t nu = (nsg + unit - 1) / unit;
        int32_t C = (nu + sgs / unit - 1) / (sgs / unit);
        if (C < want) C = want < nu ? want : nu;
        const int32_t S = 256 / C;
        g.unit = unit;
        g.chunks = C;
        g.splits = S < 1 ? 1 : (S > ntb ? ntb : S);
        return (int64_t)unit * ((nu + C - 1) / C) * ((ntb + g.splits - 1) / g.splits);
    };
    // fours let the coarse maxima go out in whole pieces (see the kernel), if the split stays even
    const int64_t ones = split(1);
    if (g.ew == 1 && sgs % 4 == 0 && 16 * split(4) > 17 * ones) (void)split(1);
    return g;
}

template <int RC>
void launch_sweep(const SweepGrid& g, const BucketArgs& a, int32_t T, const uint16_t* zh,
                  int32_t Tp, int32_t nCp, uint32_t* fine, float* coarse, float2* fnorm,
                  float2* cnorm, int32_t* hist, hipStream_t st) {
    hipLaunchKernelGGL((bucket_sweep_kernel<RC>), dim3((unsigned)g.chunks * (unsigned)g.splits),
                       dim3(kSweepThreads), 0, st, zh, a.R2t, T, a.r, a.M, g.chunks, g.splits, g.ew,
                       g.unit, Tp, nCp, fine, coarse, fnorm, cnorm, hist);
}

template <int SEG, int NS, bool EXACT, int K, bool COOP>
void launch_select(const BucketArgs& a, int64_t t0, int32_t T, int32_t Tp, int32_t nCp,
                   const uint32_t* fine, const float* coarse, const float2* fnorm, const float2* cnorm,
                   hipStream_t st) {
    constexpr int TOK = SelectCfg<K, COOP>::TOKENS;
    const SelectArgs args{a.z + t0 * a.r, a.zhi + t0 * a.r, a.cz + t0, a.cd + t0, a.R2t,
                          reinterpret_cast<const uint16_t*>(fine), coarse, fnorm, cnorm, T, Tp, nCp, a.r,
                          a.M, a.k, a.pieces, a.idx + t0 * a.k, a.gate + t0 * a.k,
                          a.topval ? a.topval + t0 * a.k : nullptr};
    hipLaunchKernelGGL((bucket_select_kernel<SEG, NS, EXACT, K, COOP>),
                       dim3((unsigned)((T + TOK - 1) / TOK)), dim3(kSelThreads), 0, st, args);
}

template <int SEG, int NS, bool EXACT>
void launch_select_k(const BucketArgs& a, int64_t t0, int32_t T, int32_t Tp, int32_t nCp,
                     const uint32_t* fine, const float* coarse, const float2* fnorm,
                     const float2* cnorm, hipStream_t st) {
    constexpr int S4 = SEG < 4 ? 4 : SEG;  // 64 lanes per token: at most 16 rows per load
    constexpr bool X4 = EXACT && SEG >= 4;
#define MORE_SELECT(S, X, K, COOP) \
    launch_select<S, NS, X, K, COOP>(a, t0, T, Tp, nCp, fine, coarse, fnorm, cnorm, st)
    if (one_token_per_workgroup(T, a.M)) {
        if (a.k <= 8)
            MORE_SELECT(S4, X4, 8, true);
        else if (a.k <= 16)
            MORE_SELECT(S4, X4, 16, true);
        else
            MORE_SELECT(S4, X4, 32, true);
    } else if (a.k <= 8) {
        MORE_SELECT(SEG, EXACT, 8, false);
    } else if (a.k <= 16) {
        MORE_SELECT(SEG, EXACT, 16, false);
    } else {
        MORE_SELECT(S4, X4, 32, false);
    }
#undef MORE_SELECT
}

}  // namespace

bool bucket_make_plan(int64_t T, int32_t r, int32_t M, int32_t k, size_t beside, BucketPlan* p) {
    if (M < kBucketMinExperts || M > kBucketMaxExperts || r < 16 || r % 16 != 0 ||
        r > kBucketMaxRank || k > 32 || T < 1 || (int64_t)M * r >= ((int64_t)1 << 31))
        return false;
    const int32_t nsg = (M + kSgExperts - 1) / kSgExperts;
    size_t room = kMaximaBytes;
    if (beside + kMaximaLeast <= kScratchAim && room > kScratchAim - beside) room = kScratchAim - beside;
    int64_t slab = (int64_t)(room / token_bytes(nsg));
    // Whole rounds of the sweep, one token block for each of 256 workgroups, and what is left in a last
    // slab, whose sweep is split finer (T 32768, r 16, M 262144: 4096 tokens each instead of even slabs of
    // 4864, where some workgroups had a second block: 749 -> 644 us a call).
    int32_t sgs, wt;
    sweep_limits(sweep_rc(r), &sgs, &wt);
    const int32_t chunks = (nsg + sgs - 1) / sgs;
    const int64_t round = (int64_t)kSweepWaves * wt * (chunks < 256 ? 256 / chunks : 1);
    const bool whole = slab >= round;
    slab = whole ? slab / round * round : (slab >= 1024 ? slab / 1024 * 1024 : slab / 32 * 32);
    if (slab < 32) slab = 32;  // (M <= 2^24: 84 MB)
    const int64_t tp = (T + 31) / 32 * 32;
    if (slab > tp) slab = tp;
    if (!whole) {  // even slabs
        const int64_t ns = (T + slab - 1) / slab;
        const int64_t even = ((T + ns - 1) / ns + 255) / 256 * 256;
        if (even < slab) slab = even;
    }
    p->slab = slab;
    size_t o = 0;
    p->off_cd = o;
    o += align256((size_t)T * sizeof(float));
    p->off_fine = o;
    o += align256((size_t)nsg * p->slab * 32);
    p->off_coarse = o;
    p->nCp = (2 * nsg + 7) / 8 * 8;  // rows of whole 32-byte pieces
    o += align256((size_t)p->slab * p->nCp * sizeof(float));
    p->off_fnorm = o;
    o += align256((size_t)nsg * 16 * sizeof(float2));
    p->off_cnorm = o;
    o += align256((size_t)p->nCp * sizeof(float2));
    p->bytes = o;
    return true;
}

hipError_t bucket_launch(const BucketPlan& p, const BucketArgs& a, void* scratch, hipStream_t st) {
    char* ws = static_cast<char*>(scratch);
    uint32_t* fine = reinterpret_cast<uint32_t*>(ws + p.off_fine);
    float* coarse = reinterpret_cast<float*>(ws + p.off_coarse);
    float2* fnorm = reinterpret_cast<float2*>(ws + p.off_fnorm);
    float2* cnorm = reinterpret_cast<float2*>(ws + p.off_cnorm);
    const int32_t nsg = (a.M + kSgExperts - 1) / kSgExperts;
    const int32_t rc = sweep_rc(a.r);
    const int32_t Tp = (int32_t)p.slab;
    for (int64_t t0 = 0; t0 < a.T; t0 += p.slab) {
        const int32_t T = (int32_t)(a.T - t0 < p.slab ? a.T - t0 : p.slab);
        const SweepGrid g = sweep_grid(rc, T, nsg);
        const uint16_t* zh = a.zhi + t0 * a.r;
        int32_t* hist = t0 == 0 ? a.hist : nullptr;
        switch (rc) {
            case 1: launch_sweep<1>(g, a, T, zh, Tp, p.nCp, fine, coarse, fnorm, cnorm, hist, st); break;
            case 2: launch_sweep<2>(g, a, T, zh, Tp, p.nCp, fine, coarse, fnorm, cnorm, hist, st); break;
            case 3: launch_sweep<3>(g, a, T, zh, Tp, p.nCp, fine, coarse, fnorm, cnorm, hist, st); break;
            case 4: launch_sweep<4>(g, a, T, zh, Tp, p.nCp, fine, coarse, fnorm, cnorm, hist, st); break;
            case 6: launch_sweep<6>(g, a, T, zh, Tp, p.nCp, fine, coarse, fnorm, cnorm, hist, st); break;
            case 8: launch_sweep<8>(g, a, T, zh, Tp, p.nCp, fine, coarse, fnorm, cnorm, hist, st); break;
            case 12: launch_sweep<12>(g, a, T, zh, Tp, p.nCp, fine, coarse, fnorm, cnorm, hist, st); break;
            case 16: launch_sweep<16>(g, a, T, zh, Tp, p.nCp, fine, coarse, fnorm, cnorm, hist, st); break;
            default: return hipErrorInvalidValue;
        }
#define MORE_SELECT_R(SEG, NS, EXACT) \
    launch_select_k<SEG, NS, EXACT>(a, t0, T, Tp, p.nCp, fine, coarse, fnorm, cnorm, st)
        switch (a.r) {
            case 16: MORE_SELECT_R(2, 1, true); break;
            case 32: MORE_SELECT_R(4, 1, true); break;
            case 64: MORE_SELECT_R(8, 1, true); break;
            case 128: MORE_SELECT_R(8, 2, true); break;
            default:
                if (a.r < 64)
                    MORE_SELECT_R(8, 1, false);
                else if (a.r < 128)
                    MORE_SELECT_R(8, 2, false);
                else
                    MORE_SELECT_R(8, 4, false);
        }
#undef MORE_SELECT_R
    }
    return hipGetLastError();
}

}  // namespace more
