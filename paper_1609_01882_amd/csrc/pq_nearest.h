// Nearest of the 256 centroids of one sub-quantizer for 32 rows of a wave: searched on bfloat16 matrix
// products, decided by the float32 distances that every other place of the library uses (direct
// differences, one fused multiply-add per coordinate in ascending order; lowest number on ties), so the
// answer is theirs to the bit.  Used by the encoder and by the k-means step.
//
// With x' = x - mu, c' = c - mu (mu: the sub-quantizer's mean centroid) and both split in two bfloat16 parts
// (x' = xh + xl + rest, |rest| <= 2^-18 |x'|),
//     v(c) = || c' ||^2 - 2 x'.c'  ~  || c' ||^2 - 2 (xh ch + xl ch + xh cl):
// one contraction over 3 DSUB + 3 places (the norm in three parts against ones), in whole products of 16
// places (v_mfma_f32_32x32x16_bf16; lane l of A: centroid l % 32, places 8 (l / 32) .. + 7; of B: row l % 32).
// A lane receives 16 centroids of one row per product, so the smallest two values and where the smallest
// was are three registers of the lane, not of a row that is spread over 32 lanes.
// Error: 3 * 2^-18 from what the parts leave out, an addition's 2^-23 for each of the 16 kSteps places (partial
// sums stay below twice the sum of the two squared lengths) and 2^-18 for the 4 mantissa bits that carry
// the place within a tile, all relative to || x' ||^2 + || c' ||^2: below kUnit, with 2^-16 to spare for the
// rounding of the float32 distances.  By the smallest value v1, the nearest centroid is no longer than
// || x' || + d1, d1^2 <= (1 + 3 u) (|| x' ||^2 + v1 + 3 u || x' ||^2) + kLost, so its value lies within
//     2 u (|| x' ||^2 + min(max || c' ||^2, (|| x' || + d1)^2)) + kLost
// of v1.  kLost = 2^-116 is what numbers below 2^-126 lose, which no relative bound covers (centroids within 1e-18
// of mu, another one far out): in a value at most 2^-126 for each of the 3 parts of its norm, 6 DSUB of its products
// (times the other factor: below 1, or the relative bound is larger by far), 3 DSUB + 3 products, 16 kSteps
// additions and DSUB terms of || x' ||^2, 438 in all for DSUB = 32, and that twice.
// A row with one centroid there has its answer; with one in each half of its two lanes the two are compared;
// otherwise (and where squares come near the end of float32's range) the row's 256 distances are taken,
// by the whole wave for it, or by every row's own lanes if the wave has many such rows.  A wave that met many
// takes all distances of its further rows without searching first (`all_distances`, a row to each of its 64
// lanes), so that no data takes much longer than that does: 400k rows, 8 sub-vectors of 16, against taking all
// distances from the start 505 / 154 us, with every centroid twice 489 / 637.
#pragma once

#include "common.h"

namespace psc {

typedef __bf16 pq_bf16x8 __attribute__((ext_vector_type(8)));
typedef float pq_f32x16 __attribute__((ext_vector_type(16)));

template <int DSUB>
struct PqNearest {
    static constexpr int kSteps = (3 * DSUB + 3 + 15) / 16;  // products per tile of 32 centroids
    static constexpr int kTiles = kCentroids / 32;
    static constexpr int kWavesPerEu = DSUB <= 16 ? 4 : 2;  // (registers for their operands)
    static constexpr int kManyRows = 10;  // rows of a wave from which every row's own lanes take all distances
    static_assert(DSUB <= 32, "kUnit and kLost are sums over at most 7 products of 16 places");
    static constexpr float kUnit = 0x1p-14f + 0x1p-18f;
    static constexpr float kLost = 0x1p-116f;
    struct Shared {
        pq_bf16x8 image[kTiles * kSteps * 64];  // operands in the order of the products
        float mu[DSUB];
        float norm[kCentroids];
        uint32_t cmax2;  // bits of the largest squared length, rounded up (not a number: on top)
    };

    // part `which` of a value: 0 the high, 1 the low bfloat16
    static __device__ __forceinline__ float part(float v, int which)
    {
        const float h = (float)(__bf16)v;
        return which == 0 ? h : v - h;
    }

    // Called by the whole workgroup (a multiple of 256 threads); ends with a barrier.  cb: the sub-quantizer's.
    static __device__ __forceinline__ void prepare(Shared &s, const float *__restrict__ cb)
    {
        const int tid = (int)threadIdx.x, nthreads = (int)blockDim.x;
        // the mean: 256 / DSUB (or fewer) partial sums per coordinate, kept where the image will be
        float *part_sum = (float *)s.image;
        constexpr int kParts = 256 / DSUB;
        if (tid < kParts * DSUB) {
            const int t = tid % DSUB, p = tid / DSUB;
            float acc = 0.f;
            for (int c = p; c < kCentroids; c += kParts) acc += cb[c * DSUB + t];
            part_sum[p * DSUB + t] = acc;
        }
        if (tid == 0) s.cmax2 = 0u;
        __syncthreads();
        if (tid < DSUB) {
            float acc = 0.f;
            for (int p = 0; p < kParts; ++p) acc += part_sum[p * DSUB + tid];
            s.mu[tid] = acc * (1.0f / kCentroids);
        }
        __syncthreads();
        if (tid < kCentroids) {
            double n = 0.0;
#pragma unroll
            for (int t = 0; t < DSUB; ++t) {
                const double e = (double)(cb[tid * DSUB + t] - s.mu[t]);
                n += e * e;
            }
            s.norm[tid] = (float)n;
            // (bits of floats that are not negative are ordered as the floats are)
            atomicMax(&s.cmax2, __float_as_uint((float)n * 1.0001f) & 0x7fffffffu);
        }
        for (int e = tid; e < kTiles * kSteps * 64; e += nthreads) {
            const int lane = e & 63, step = (e >> 6) % kSteps, tile = (e >> 6) / kSteps;
            const int c = tile * 32 + (lane & 31), at = 16 * step + 8 * (lane >> 5);
            pq_bf16x8 v;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int p = at + i;
                float w = 0.f;
                if (p < 3 * DSUB) {
                    const int t = p < DSUB ? p : (p < 2 * DSUB ? p - DSUB : p - 2 * DSUB);
                    w = part(cb[c * DSUB + t] - s.mu[t], p < 2 * DSUB ? 0 : 1);
                }
                v[i] = (__bf16)w;
            }
            s.image[e] = v;
        }
        __syncthreads();
        // the norms' three parts, at places 3 DSUB .. 3 DSUB + 2
        for (int e = tid; e < kCentroids * 3; e += nthreads) {
            const int c = e & (kCentroids - 1), i = e / kCentroids, p = 3 * DSUB + i;
            float w = s.norm[c];
            for (int k = 0; k < i; ++k) w = part(w, 1);
            __bf16 *entry = (__bf16 *)&s.image[((c >> 5) * kSteps + p / 16) * 64 + ((p % 16) / 8) * 32 + (c & 31)];
            entry[p % 8] = (__bf16)w;
        }
        __syncthreads();
    }

    static __device__ __forceinline__ float distance(const float (&v)[DSUB], const float *__restrict__ cen)
    {
        float acc = 0.f;
#pragma unroll
        for (int t = 0; t < DSUB; ++t) {
            const float df = v[t] - cen[t];
            acc = fmaf(df, df, acc);
        }
        return acc;
    }

    // The nearest centroid of the lane's own row, all distances taken (the centroids, the same for every lane, come
    // through the scalar cache).
    static __device__ __forceinline__ int all_distances(const float *__restrict__ cb, const float (&v)[DSUB])
    {
        float best = __builtin_inff();
        int bi = 0;
#pragma unroll 2
        for (int c = 0; c < kCentroids; ++c) {
            const float d = distance(v, cb + c * DSUB);
            if (d < best) {
                best = d;
                bi = c;
            }
        }
        return bi;
    }

    // v: the sub-vector of row lane % 32 (both halves of the wave hold it); the whole wave calls.  live: whether the
    // answer is asked for (rows past the end are copies of the last one, and a close call there would be many: 500 rows,
    // 8 sub-vectors of 8, 24 us where it is 11).  `many` is set if many of the rows needed all distances.
    static __device__ __forceinline__ int search(const Shared &s, const float *__restrict__ cb, const float (&v)[DSUB],
                                                 bool live, bool &many)
    {
        const int lane = (int)(threadIdx.x & 63), half = lane >> 5;
        pq_bf16x8 row[kSteps];
        float x2 = 0.f;
        if constexpr (DSUB % 16 == 0) {  // a lane's places are the same coordinates in every part
            constexpr int kBlocks = DSUB / 16;
#pragma unroll
            for (int b = 0; b < kBlocks; ++b)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int t = 16 * b + i;
                    float lo = v[t], hi = v[t + 8];
                    asm("" : "+v"(lo), "+v"(hi));  // (a choice of registers: left alone it becomes one of addresses)
                    const float e = (half ? hi : lo) - s.mu[t + 8 * half];
                    x2 = fmaf(e, e, x2);
                    row[b][i] = (__bf16)(-2.f * e);
                    row[kBlocks + b][i] = (__bf16)part(-2.f * e, 1);
                }
#pragma unroll
            for (int b = 0; b < kBlocks; ++b) row[2 * kBlocks + b] = row[b];
#pragma unroll
            for (int i = 0; i < 8; ++i) row[3 * kBlocks][i] = (__bf16)(half == 0 && i < 3 ? 1.f : 0.f);
            x2 += __shfl_xor(x2, 32, 64);
        } else {
            float h[DSUB], l[DSUB];
#pragma unroll
            for (int t = 0; t < DSUB; ++t) {
                const float e = v[t] - s.mu[t];
                x2 = fmaf(e, e, x2);
                h[t] = part(-2.f * e, 0);
                l[t] = part(-2.f * e, 1);
            }
            auto place = [&](int p) {
                return p < DSUB ? h[p] : p < 2 * DSUB ? l[p - DSUB] : p < 3 * DSUB ? h[p - 2 * DSUB] : p < 3 * DSUB + 3 ? 1.f : 0.f;
            };
#pragma unroll
            for (int st = 0; st < kSteps; ++st)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float lo = place(16 * st + i), hi = place(16 * st + 8 + i);
                    row[st][i] = (__bf16)(half ? hi : lo);
                }
        }
        uint32_t keep = ~15u;
        asm("" : "+v"(keep));
        float best = __builtin_inff(), next = __builtin_inff();
        int at = 0;
        auto product = [&](int tile, pq_f32x16 &acc) {
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
            for (int st = 0; st < kSteps; ++st)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(s.image[(tile * kSteps + st) * 64 + lane], row[st], acc, 0, 0, 0);
        };
        auto see = [&](int tile, const pq_f32x16 &acc) {
            const float before = best;
#pragma unroll
            for (int i = 0; i < 16; i += 2) {  // the two smallest of the two so far and two more
                const float a = __uint_as_float((__float_as_uint(acc[i]) & keep) | (uint32_t)i);
                const float b = __uint_as_float((__float_as_uint(acc[i + 1]) & keep) | (uint32_t)(i + 1));
                const float mid = __builtin_amdgcn_fmed3f(best, a, b);
                asm("v_min_f32 %0, %0, %1" : "+v"(next) : "v"(mid));
                asm("v_min3_f32 %0, %0, %1, %2" : "+v"(best) : "v"(a), "v"(b));
            }
            at = best < before ? tile : at;
        };
        // (a tile's products are under way while the one before is looked through)
        pq_f32x16 even, odd;
        product(0, even);
#pragma unroll 1
        for (int tile = 0; tile < kTiles; tile += 2) {
            product(tile + 1, odd);
            see(tile, even);
            if (tile + 2 < kTiles) product(tile + 2, even);
            see(tile + 1, odd);
        }
        const int i = (int)(__float_as_uint(best) & 15u);
        const int mine = at * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
        const float least = fminf(best, __shfl_xor(best, 32, 64));
        const float cmax2 = __uint_as_float(s.cmax2);
        const float d2 = (fmaxf(least + x2, 0.f) + 3.f * kUnit * x2) * (1.f + 3.f * kUnit) + kLost;
        const float len = __builtin_amdgcn_sqrtf(x2) + __builtin_amdgcn_sqrtf(d2);
        const float reach = least + (2.f * kUnit * (x2 + fminf(cmax2, 1.001f * len * len)) + kLost);
        const bool finite = x2 + cmax2 < 1e37f;  // (no if either is not a number)
        const int near = best <= reach ? 1 : 0, deep = !finite || next <= reach ? 2 : 0;
        const int other = __shfl_xor(near | deep, 32, 64), theirs = __shfl_xor(mine, 32, 64);
        int winner = near ? mine : theirs;
        const bool all = live && ((deep | other) & 2) != 0, both = near && (other & 1) && !all;
        if (__ballot(both) != 0) {
            const float d = both ? distance(v, cb + mine * DSUB) : 0.f;
            const float o = __shfl_xor(d, 32, 64);
            if (both) winner = d < o || (d == o && mine < theirs) ? mine : theirs;
        }
        uint32_t rows = (uint32_t)__ballot(all);  // (the same in both halves)
        if (rows != 0u) {
            if (__builtin_popcount(rows) > kManyRows) {
                many = true;
                float b = __builtin_inff();
                int bi = 0;
#pragma unroll 1
                for (int c = 0; c < kCentroids / 2; ++c) {
                    const float d = distance(v, cb + (half * (kCentroids / 2) + c) * DSUB);
                    if (d < b) {
                        b = d;
                        bi = half * (kCentroids / 2) + c;
                    }
                }
                const float ob = __shfl_xor(b, 32, 64);
                const int obi = __shfl_xor(bi, 32, 64);
                if (all) winner = b < ob || (b == ob && bi < obi) ? bi : obi;
            } else {
                for (; rows != 0u; rows &= rows - 1u) {
                    const int r = __builtin_ctz(rows);
                    float rv[DSUB];
#pragma unroll
                    for (int t = 0; t < DSUB; ++t)
                        rv[t] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v[t]), r));
                    float b = __builtin_inff();
                    int bi = 0;
#pragma unroll 1
                    for (int k = 0; k < kCentroids / 64; ++k) {
                        const float d = distance(rv, cb + (64 * k + lane) * DSUB);
                        if (d < b) {
                            b = d;
                            bi = 64 * k + lane;
                        }
                    }
#pragma unroll
                    for (int off = 32; off >= 1; off >>= 1) {
                        const float ob = __shfl_xor(b, off, 64);
                        const int obi = __shfl_xor(bi, off, 64);
                        const bool take = ob < b || (ob == b && obi < bi);
                        b = take ? ob : b;
                        bi = take ? obi : bi;
                    }
                    if ((lane & 31) == r) winner = bi;
                }
            }
        }
        return winner;
    }
};

}  // namespace psc
