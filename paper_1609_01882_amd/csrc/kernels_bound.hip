// Flat search by bounds: which pairs can be among a query's k best is decided on the matrix cores, in 6-bit floating
// point, and only those few are tested and scored (Section 3.3 two-step strategy with the steps' order turned round: the
// answer -- the k best by distance among the codes within ht -- is the same).
//
// With c(code) the concatenated centroids of a code (relative to the mean centroids, in units of u) and q the query
// likewise, the distance is |q|^2 + |c|^2 - 2 q.c.  Both are rounded to 6-bit floats Q, R (E2M3, a power of two per 32
// coordinates), and acc = Q.R - |c|^2 / 2 comes from the matrix cores for every pair: K = 64 coordinates an instruction,
// at 3.5 times the rate of bfloat16.  acc is a sum over the sub-quantizers, acc = sum_j B[j][code_j], like the distance
// D = sum_j lut[j][code_j] itself.  So for every lambda >= 0 a code with D <= thr has
//     acc >= sum_j min_c (B[j][c] + lambda lut[j][c]) - lambda thr = S(lambda) - lambda thr,
// whatever the rounding of Q and R was: the bound is taken from the very numbers that are compared.  A larger lambda looks
// only at centroids that a code within thr can have at all, which is what makes the bound sharp; eight of them are
// tried and the best is used.  SIFT-like vectors of 128 dimensions in 64-bit codes, 500k of them, thr the 13th nearest: 41
// codes per query pass (a simulation with 8-bit integers, 1M codes, thr the 10th nearest: 2247 with lambda = 1 alone, 44 with
// all of them).  8-bit integers would let a quarter as many pass, at half the products' rate.
//
// thr comes from a sample of the codes, scored whole, and is sharpened by a round over some thirty times as many codes (or
// several such rounds), before all are looked at: the distance of the r-th best of a part, r being so many that among R times
// as many codes at least k are as near in all but 1 of 10^7 cases, if the order of the codes is a random one (the parts
// are single codes at odd strides: in a database in the order of its clusters they are still fair).  Whether there were k is checked; a
// query where there were not, whose lists overflow, or whose tables are not finite, is marked, and a scan over marked
// queries alone follows (ScanArgs::redo): the answer does not depend on any of this.
// What passes the bound is tested (Hamming distance) and scored from the same tables and in the same order of
// additions as everywhere, and the k best of what is no farther than thr are selected.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "bound_queue.h"
#include "common.h"
#include "entry.h"

namespace psc {
namespace {

constexpr int kBlock = 128;          // codes of a block: four turns of a wave
constexpr int kLambdas = 8;
__device__ const float kLambda[kLambdas] = {1.0f, 1.04f, 1.1f, 1.18f, 1.35f, 1.7f, 2.5f, 5.0f};
// Places per query, on the average of a tile, for the codes that pass its bound in a round (two words each: 485 MiB from 5120
// queries on).  Mixtures take as long with 6144 or 24576 (777 x 1M 0.999 and 0.999 of the time, 10k x 10M 1.02 and 0.99, runs
// differing by as much).  Gaussian vectors in 128-bit codes, 20 .. 5000 queries x 100k .. 3.2M: with 6144 more are given up
// that need not be, 0.78 of the time without bounds in geometric mean, 0.755 so.  With 24576 batches go on that are given up
// later: 4000 x 4M 64-bit codes of 1000 kinds, ht 24 7450 us, 3070 so, random ones 3430 and 2400 (but 1000 x 1M 543, 1128 so).
constexpr int kNear = 12288;
constexpr int kRun = 8;              // rows a thread of bound_rank_kernel takes of a run at a time
constexpr int kMaxItems = 4096;      // work items (tile, slice) of a round
constexpr int kBoundPool = 2048;     // those of them that are tested and nearer than thr
constexpr int kBoundMaxK = 256;
constexpr int kLeastSample = 4096, kMaxSample = 65536;  // codes of the sample
constexpr int kMostStep = 5;         // a round looks at most at 2^this times as many codes as all before
constexpr int kSampleKeys = 2048;    // keys of the sample's pool
// Rows that a query may list in a round over so many codes.  More are ranked by one workgroup, 2.6 ns a row, in longer than
// 16 take to scan all codes for a query that is marked (4000 queries x 4M codes, half of them alike, 128 bits, nothing
// filtered: 5500 us with all of them ranked, 5000 with this; 3000 x 200k 935 and 592).
inline double most_listed(double codes) { return 2.0 * kNear + codes / 32.0; }
constexpr int kMarkWords = 64;       // of `marks`: the count, and from here on `few` words for the scan of each, then which they are
constexpr float kLeast = -1e29f;     // below every product, above every invalid row's
constexpr float kInvalid = 1e30f;    // "half square" of a row past the end

// Padded sub-vector DP = 8, 16 or 32 coordinates; lane half h of a matrix instruction holds the sub-quantizers
// h M/2 .. h M/2 + M/2 - 1, 32 coordinates (a block: BPJ sub-quantizers) to a step.
template <int M, int DP>
struct Shape {
    static constexpr int BPJ = 32 / DP;             // sub-quantizers per block
    static constexpr int NS = M * DP / 64;          // steps of 64 coordinates
    static constexpr int ENT = DP == 8 ? 8 : DP == 16 ? 16 : 32;  // bytes of a centroid in LDS
    static constexpr int QG = NS <= 2 ? 8 : 4;      // groups of 32 queries a wave holds
    static constexpr int QUEUE = kQueuePlaces<QG>;  // entries of a wave's queue
};

template <int M, int DP>
struct BoundLds {
    using S = Shape<M, DP>;
    unsigned char img[M * 256 * S::ENT];
    uint32_t queue[4][S::QUEUE];  // what passed the bound: place in the slice << 8 | query of the tile
    uint32_t share[256];          // how many of a query (then: where they go)
    uint32_t part[4];
    uint32_t listed;
    float least[S::QG * 32];      // the bound on acc
};

struct BoundArgs {
    const uint8_t *codes;
    const void *img;          // centroids in 6-bit floats, as they lie in LDS
    const uint32_t *qimg;     // queries likewise, [group][step][6][64]
    const uint32_t *qscale;   // [group][64]: exponents of their blocks, a byte per step
    const float *s;           // [nq][kLambdas]
    const uint64_t *thr;      // [nq] codes with keys up to it are wanted (~0: all)
    uint32_t *redo;           // [nq]
    const uint32_t *unfit;    // of every eighth query of the batch those that would list too much (marked ones twice)
    uint32_t *raw;            // [tiles * slices][cap] what passed the bound, as it came
    uint32_t *near;           // [tiles * slices][cap] the rows of those codes, by query
    uint32_t *first;          // [tiles * slices][257] where a query's rows begin
    int cap;
    int n, nq, groups, tiles, slices;
    int stride, codes_in, blocks;  // of the round: every stride-th code, ceil(n / stride) of them, in blocks
    float half_unit;          // 1 / (2 u^2)
    uint32_t scale_lo, scale_hi;  // exponents of the centroids' blocks, a byte per step, lane halves 0 and 1
    float norm_grid;          // DP = 8: unit of the 16-bit half squares
};

// A work item (tile, slice): its first query, its queries, its blocks (every slices-th of the round's: whatever the order
// of the database, the items have about the same to list).
struct BoundItem {
    int g0, ng, q0, nvq, slice, blocks;
};
__device__ __forceinline__ BoundItem bound_item(const BoundArgs &a, int item)
{
    BoundItem w;
    const int tile = item / a.slices;
    w.slice = item - tile * a.slices;
    w.g0 = (int)((int64_t)tile * a.groups / a.tiles);
    w.ng = (int)((int64_t)(tile + 1) * a.groups / a.tiles) - w.g0;
    w.q0 = w.g0 * 32;
    w.nvq = min(a.nq - w.q0, w.ng * 32);
    w.blocks = (a.blocks - w.slice + a.slices - 1) / a.slices;
    return w;
}
// Database row of a place in a slice.
__device__ __forceinline__ uint32_t row_of(const BoundArgs &a, int slice, uint32_t place)
{
    const uint32_t block = (uint32_t)slice + place / kBlock * (uint32_t)a.slices;
    return (block * kBlock + place % kBlock) * (uint32_t)a.stride;
}

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v6i __attribute__((ext_vector_type(6)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ v8i as_operand(v6i v) { return __builtin_shufflevector(v, v, 0, 1, 2, 3, 4, 5, -1, -1); }

constexpr int kE2M3 = 2;  // operand format of the matrix instruction

__device__ __forceinline__ float largest(float x, float y, float z)
{
    return __builtin_elementwise_maximum(__builtin_elementwise_maximum(x, y), z);
}
template <int STEP>
__device__ __forceinline__ v16f multiply(v6i a, v6i b, v16f c, uint32_t sa, uint32_t sb)
{
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as_operand(a), as_operand(b), c, kE2M3, kE2M3, STEP, (int)sa, STEP, (int)sb);
}

// The least acc a code of query q may have that is to be looked at.
__device__ __forceinline__ float least_product(const BoundArgs &a, int64_t q)
{
    if (a.redo[q] != 0u) return __builtin_inff();
    const uint64_t key = a.thr[q];
    if (key == kNoEntry) return kLeast;
    const float thr = entry_dist(key) * (a.half_unit * 1.00001f);
    float best = kLeast;
#pragma unroll
    for (int i = 0; i < kLambdas; ++i) best = fmaxf(best, a.s[q * kLambdas + i] - kLambda[i] * thr);
    return best;
}

// Codes of a block: half h of the lane's code (rows lane % 32).
template <int M>
struct CodeHalf {
    uint32_t w[M / 8];
};

// 32 codes x up to QG * 32 queries a turn and wave.  What bounds it: the matrix cores' products (2 per 1024 pairs and 128
// dimensions) and beside them nine vector instructions per 1024 pairs that find the largest of a lane's 16 products.  The
// queries' operands stay in registers for the whole slice; a code's come from LDS by one gather per sub-quantizer,
// shared by the wave's 256 queries; the half squares are spread over the accumulators by one float32 product, which adds
// up the lane halves' shares as well.  The products of two groups are on their way while those of a third are compared: the
// order is written out, left to itself the compiler waits for each product in turn (the last round of 2000 queries x 10M codes 1985 us,
// 1484 so; with every comparison left out 1220, which is 62 ns a tile of 1024 pairs: the products alone, on operands in
// registers, take 54 at the clock this card holds under them).
// What passes the bound goes to the query's list and is looked at by the next launch, where waves are many and the query's
// tables lie in LDS (here a wave would wait three trips to memory for every 64 codes).
template <int M, int DP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
bound_scan_kernel(BoundArgs a)
{
    using S = Shape<M, DP>;
    constexpr int QG = S::QG, NS = S::NS;
    extern __shared__ __align__(16) unsigned char smem[];
    PSC_LDS BoundLds<M, DP> &s = *(PSC_LDS BoundLds<M, DP> *)smem;
    const int tid = (int)threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // Work in the order (tile, slice), an eighth of it to each XCD (workgroups go round them in turn).
    const int total = a.tiles * a.slices;
    const int share = (total + 7) >> 3;
    const int item = (int)(blockIdx.x & 7u) * share + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= share || item >= total) return;
    const BoundItem it = bound_item(a, item);
    if (*a.unfit * 64u > (uint32_t)a.nq) {  // (uniform; the rounds after this one find the marks)
        for (int i = tid; i < it.nvq; i += 256) a.redo[it.q0 + i] = 1u;
        for (int i = tid; i < 257; i += 256) a.first[(size_t)item * 257 + i] = 0u;
        return;
    }

    for (int e = tid; e < M * 256 * S::ENT / 16; e += 256)
        ((PSC_LDS v4i *)s.img)[e] = ((const v4i *)a.img)[e];
    for (int i = tid; i < QG * 32; i += 256) s.least[i] = i < it.nvq ? least_product(a, it.q0 + i) : __builtin_inff();
    v6i q[QG][NS];
    uint32_t qs[QG];
#pragma unroll
    for (int g = 0; g < QG; ++g) {
        const int gg = it.g0 + (g < it.ng ? g : 0);  // (the bound of groups that are not there is infinite)
        qs[g] = a.qscale[(int64_t)gg * 64 + lane];
#pragma unroll
        for (int t = 0; t < NS; ++t)
#pragma unroll
            for (int i = 0; i < 6; ++i) q[g][t][i] = (int)a.qimg[(((int64_t)gg * NS + t) * 6 + i) * 64 + lane];
    }
    const uint32_t cs = half ? a.scale_hi : a.scale_lo;
    for (int i = tid; i < 256; i += 256) s.share[i] = 0u;
    if (tid == 0) s.listed = 0u;
    __syncthreads();
    float least[QG];
    auto load_least = [&]() {
#pragma unroll
        for (int g = 0; g < QG; ++g) least[g] = ((volatile PSC_LDS float *)s.least)[g * 32 + (lane & 31)];
    };
    load_least();
    bool any = false;
#pragma unroll
    for (int g = 0; g < QG; ++g) any = any || least[g] < __builtin_inff();
    __syncthreads();  // (the waves have read the same: none has marked a query yet)
    if (ballot64(any) == 0ull) {  // every query of the tile is marked
        for (int i = tid; i < 257; i += 256) a.first[(size_t)item * 257 + i] = 0u;
        return;
    }

    const uint32_t bytes = (uint32_t)a.n * (uint32_t)M;  // (< 2^31)
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.codes, 0, (int)bytes, 0x00020000);
    // the wave's blocks: every fourth of the item's, asked for a block ahead
    int block_at = (it.slice + wave * a.slices) * kBlock;
    auto next_base = [&]() {
        const int base = block_at;
        block_at += 4 * a.slices * kBlock;
        return base;
    };
    const uint32_t step = (uint32_t)a.stride * (uint32_t)M;
    auto load = [&](int base, CodeHalf<M> (&c)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // (past the end: zeros, or where 32 bits wrap some row's code; spread() leaves such rows out either way)
            const int at = (int)((uint32_t)(base + 32 * i + (lane & 31)) * step + (uint32_t)(half * (M / 2)));
            if constexpr (M == 8) {
                c[i].w[0] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, at, 0, 0);
            } else {
                const v2i v = __builtin_amdgcn_raw_buffer_load_b64(rsrc, at, 0, 0);
                c[i].w[0] = (uint32_t)v[0];
                c[i].w[1] = (uint32_t)v[1];
            }
        }
    };
    PSC_LDS unsigned char *const img = s.img + half * (M / 2) * 256 * S::ENT;
    // the operand of a block and the lane half's share of the half square
    auto decode = [&](const CodeHalf<M> &c, v6i (&op)[NS]) {
        auto entry = [&](int j) { return img + j * 256 * S::ENT + ((c.w[j >> 2] >> (8 * (j & 3))) & 0xffu) * S::ENT; };
        if constexpr (DP == 16) {
            float sq = 0.f;
#pragma unroll
            for (int t = 0; t < NS; ++t) {
                const v4i e = *(PSC_LDS v4i *)entry(2 * t), o = *(PSC_LDS v4i *)entry(2 * t + 1);
                op[t][0] = e[0];
                op[t][1] = e[1];
                op[t][2] = e[2];
                op[t][3] = o[2];
                op[t][4] = o[0];
                op[t][5] = o[1];
                sq += __int_as_float(e[3]) + __int_as_float(o[3]);
            }
            return sq;
        } else if constexpr (DP == 32) {
            float sq = 0.f;
#pragma unroll
            for (int t = 0; t < NS; ++t) {
                const v4i e = *(PSC_LDS v4i *)entry(t), o = *(PSC_LDS v4i *)(entry(t) + 16);
                op[t][0] = e[0];
                op[t][1] = e[1];
                op[t][2] = e[2];
                op[t][3] = e[3];
                op[t][4] = o[0];
                op[t][5] = o[1];
                sq += __int_as_float(o[2]);
            }
            return sq;
        } else {
            uint32_t sq = 0u;
#pragma unroll
            for (int t = 0; t < NS; ++t)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const v2i e = *(PSC_LDS v2i *)entry(4 * t + 2 * p), o = *(PSC_LDS v2i *)entry(4 * t + 2 * p + 1);
                    op[t][3 * p] = e[0];
                    op[t][3 * p + 1] = (int)(((uint32_t)e[1] & 0xffffu) | ((uint32_t)o[0] & 0xffff0000u));
                    op[t][3 * p + 2] = o[1];
                    sq += ((uint32_t)e[1] >> 16) + ((uint32_t)o[0] & 0xffffu);
                }
            return (float)sq * a.norm_grid;
        }
    };

    // What passed the bound: from the wave's queue, 64 at a time, to the item's list in memory.
    PSC_LDS uint32_t *const queue = s.queue[wave];
    uint32_t *const raw = a.raw + (size_t)item * a.cap;
    int fill = 0;
    auto drain = [&](int left) {
        __builtin_amdgcn_wave_barrier();
        bool full = false;
        while (fill > left) {
            const int n = fill < 64 ? fill : 64;
            fill -= n;
            const uint32_t e = lane < n ? queue[fill + lane] : 0u;
            uint32_t at = 0u;
            if (lane == 0) at = __hip_atomic_fetch_add(&s.listed, (uint32_t)n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + (uint32_t)lane;
            if (lane < n && at < (uint32_t)a.cap) {
                raw[at] = e;
                __hip_atomic_fetch_add(&s.share[e & 255u], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            } else if (lane < n) {  // no room: the query is left to the scan of marked queries
                const int qi = (int)(e & 255u);
                ((volatile PSC_LDS float *)s.least)[qi] = __builtin_inff();
                __hip_atomic_store(&a.redo[it.q0 + qi], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                full = true;
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (ballot64(full) != 0ull) load_least();
    };

    const int blocks = (it.blocks - wave + 3) >> 2;
    auto scan = [&](auto groups) {  // for a known number of groups
        constexpr int NG = decltype(groups)::value;
        constexpr int HALF = (NS + 1) / 2;  // steps before the comparisons of the group two before, the others after them
        v6i op[NS];
        v16f acc[3], start;
        auto steps = [&](auto half, int g) {
            v16f v = half ? acc[g % 3] : start;
            if constexpr (!half) {
                v = multiply<0>(op[0], q[g][0], v, cs, qs[g]);
                if constexpr (HALF > 1) v = multiply<1>(op[1], q[g][1], v, cs, qs[g]);
            } else {
                if constexpr (NS == 2) v = multiply<1>(op[1], q[g][1], v, cs, qs[g]);
                if constexpr (NS == 4) {
                    v = multiply<2>(op[2], q[g][2], v, cs, qs[g]);
                    v = multiply<3>(op[3], q[g][3], v, cs, qs[g]);
                }
            }
            acc[g % 3] = v;
        };
        constexpr std::integral_constant<bool, false> lower{};
        constexpr std::integral_constant<bool, true> upper{};
        auto spread = [&](float sq, int row) {  // the half squares in every product's place
            sq = row + (lane & 31) < a.codes_in ? sq : kInvalid;
            const v16f z = {};
            return __builtin_amdgcn_mfma_f32_32x32x2f32(-sq, 1.0f, z, 0, 0, 0);
        };
        // One turn: the products of 32 codes with all groups, while the next turn's codes are decoded.
        auto turn = [&](uint32_t place0, const CodeHalf<M> &next, int next_row) {
            v6i op1[NS];
            const float sq1 = decode(next, op1);
            steps(lower, 0);
            steps(lower, 1);
            steps(upper, 0);
            steps(upper, 1);
            asm volatile("" ::"v"(acc[0]), "v"(acc[1]));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (g + 2 < NG) steps(lower, g + 2);
                __builtin_amdgcn_sched_barrier(0);
                const v16f &v = acc[g % 3];
                float mx[5];
#pragma unroll
                for (int r = 0; r < 5; ++r) mx[r] = largest(v[3 * r], v[3 * r + 1], v[3 * r + 2]);
                const uint64_t hit = ballot64(largest(largest(mx[0], mx[1], v[15]), mx[2], largest(mx[3], mx[4], mx[4])) >= least[g]);
                __builtin_amdgcn_sched_barrier(0);
                // (issued before the branch, not where they are used behind it)
                if (g + 2 < NG) {
                    steps(upper, g + 2);
                    asm volatile("" ::"v"(acc[(g + 2) % 3]));
                } else if (g + 2 == NG) {
                    start = spread(sq1, next_row);
                    asm volatile("" ::"v"(start));
                }
                if (hit != 0ull) {
                    const uint32_t place = place0 | (uint32_t)half << 10 | (uint32_t)(g << 5 | (lane & 31));
                    auto check = [&](int r) {
                        const bool pass = v[r] >= least[g];
                        const uint64_t m = ballot64(pass);
                        if (m != 0ull) {  // (row 8 (r / 4) + 4 half + r % 4)
                            if (pass) queue[fill + prefix_count(m)] = place | (uint32_t)((8 * (r >> 2) + (r & 3)) << 8);
                            fill += __builtin_popcountll(m);
                        }
                    };
                    queue_group<QG>([&](int t) { return ballot64(mx[t] >= least[g]) != 0ull; }, check,
                                    [&]() { if (fill >= 64) drain(63); });
                }
            }
#pragma unroll
            for (int t = 0; t < NS; ++t) op[t] = op1[t];
        };
        CodeHalf<M> ahead[4];  // the next block's, asked for four turns before
        int base = next_base();
        load(base, ahead);
        start = spread(decode(ahead[0], op), base);
        for (int b = 0; b < blocks; ++b) {
            CodeHalf<M> c = ahead[1], c2 = ahead[2], c3 = ahead[3];
            const int base_ahead = next_base();
            load(base_ahead, ahead);
            const uint32_t place = (uint32_t)(b * 4 + wave) << 15;
#pragma unroll 1
            for (int i = 0; i < 3; ++i) {
                turn(place | (uint32_t)i << 13, c, base + 32 * (i + 1));
                c = c2;
                c2 = c3;
            }
            turn(place | 3u << 13, ahead[0], base_ahead);  // (apart: only here are the next block's codes waited for)
            base = base_ahead;
        }
    };
    switch ((it.ng + 1) / 2) {
    case 1: scan(std::integral_constant<int, 2>{}); break;
    case 2: scan(std::integral_constant<int, 4>{}); break;
    case 3: if constexpr (QG > 4) scan(std::integral_constant<int, 6>{}); break;
    default: if constexpr (QG > 4) scan(std::integral_constant<int, 8>{}); break;
    }
    drain(0);
    __syncthreads();
    // The list by query: where each query's rows begin, and the rows there.
    const uint32_t listed = min(s.listed, (uint32_t)a.cap), mine = s.share[tid];
    uint32_t upto = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(upto, off, 64);
        if (lane >= off) upto += o;
    }
    if (lane == 63) s.part[wave] = upto;
    __syncthreads();
    for (int w = 0; w < wave; ++w) upto += s.part[w];
    s.share[tid] = upto - mine;
    a.first[(size_t)item * 257 + tid] = upto - mine;
    if (tid == 255) a.first[(size_t)item * 257 + 256] = upto;
    __syncthreads();
    uint32_t *const near = a.near + (size_t)item * a.cap;
    for (uint32_t i = tid; i < listed; i += 256u) {
        const uint32_t e = raw[i];
        near[__hip_atomic_fetch_add(&s.share[e & 255u], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)] = row_of(a, it.slice, e >> 8);
    }
}

// Smallest of v over the wave, in every lane.
__device__ __forceinline__ float wave_min_f32(float v)
{
    auto step = [&](int o) { v = fminf(v, __int_as_float(o)); };
    step(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, false));   // lane ^ 1
    step(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xf, 0xf, false));   // lane ^ 2
    step(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xf, 0xf, false));  // mirror in 8
    step(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xf, 0xf, false));  // mirror in 16
    auto row = [&](int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
    return fminf(fminf(row(0), row(16)), fminf(row(32), row(48)));
}

struct PrepareArgs {
    const float *x;        // [nq][dim]
    const float *mu;       // [dim] mean centroids
    const float *lut;      // [nq][M][256]
    const float *rounded;  // [M][256][DP] the centroids as the matrix cores see them
    const float *norms;    // [M][256] half squares
    const float *sizes;    // [M] largest |coordinate| of `rounded`, [M] largest half square
    float per_unit;        // 1 / u
    float half_unit;
    uint32_t *qimg, *qscale;
    float *s;
    uint64_t *thr;
    uint32_t *redo;
    int dim, dsub, nq;
    uint32_t *unfit;  // set to zero
    uint32_t *marks;  // (BoundLayout; null: set by an earlier launch of the call)
    int few;
    // workgroups past those of the queries gather the sample: every stride-th code
    int query_groups;
    const uint8_t *codes;
    uint8_t *sample;
    int samples, stride;
};

// The queries in 6-bit floats and S(lambda).  A workgroup takes four queries, so that the centroids (128 KB at 128
// dimensions, from L2) are read a quarter as often; a wave takes every fourth sub-quantizer, four centroids to a lane.
template <int M, int DP>
__global__ void __launch_bounds__(256)
bound_prepare_kernel(PrepareArgs a)
{
    using S = Shape<M, DP>;
    typedef float v4f __attribute__((ext_vector_type(4)));
    constexpr int NB = 2 * S::NS;  // blocks
    constexpr int Q = 4;
    __shared__ __align__(16) float rounded[Q][M * DP];
    __shared__ uint32_t most[Q][NB];
    __shared__ int exponent[Q][NB];
    __shared__ uint8_t code[Q][NB][32];
    __shared__ float sums[4][Q][kLambdas], sizes[4][Q][kLambdas], reach[Q][M];
    __shared__ uint32_t bad[Q];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if ((int)blockIdx.x >= a.query_groups) {
        typedef uint32_t words __attribute__((ext_vector_type(M / 4)));
        const int p = ((int)blockIdx.x - a.query_groups) * 256 + tid;
        if (p == 0) *a.unfit = 0u;
        if (a.marks != nullptr) {
            if (p == 0) *a.marks = 0u;
            for (int i = p; i < a.few; i += ((int)gridDim.x - a.query_groups) * 256) a.marks[kMarkWords + i] = kPresetWord;
        }
        if (p < a.samples) ((words *)a.sample)[p] = ((const words *)a.codes)[(size_t)p * a.stride];
        return;
    }
    const int64_t q0 = (int64_t)blockIdx.x * Q;
    const int here = (int)max((int64_t)0, min((int64_t)Q, (int64_t)a.nq - q0));  // (none: the rest of the last group)
    if (tid < Q * NB) most[tid / NB][tid % NB] = 0u;
    if (tid < Q) bad[tid] = 0u;
    for (int e = tid; e < Q * NB * 32; e += 256) (&code[0][0][0])[e] = 0;
    for (int e = tid; e < Q * M * DP; e += 256) (&rounded[0][0])[e] = 0.f;
    __syncthreads();
    const int j = tid / a.dsub, at = tid - j * a.dsub;  // (threads below dim)
    const int jl = j % (M / 2), block = jl / S::BPJ * 2 + j / (M / 2);
    float x[Q] = {};
    if (tid < a.dim) {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            if (i < here) {
                x[i] = (a.x[(q0 + i) * a.dim + tid] - a.mu[tid]) * a.per_unit;
                atomicMax(&most[i][block], __float_as_uint(fabsf(x[i])));
            }
        }
    }
    __syncthreads();
    if (tid < Q * NB) {
        // the smallest power of two that brings the block's largest coordinate to 7.5 or less
        const uint32_t b = most[tid / NB][tid % NB];
        const int e = (int)(b >> 23) - 129 + ((b & 0x7fffffu) > 0x700000u ? 1 : 0);
        if (e > 60) bad[tid / NB] = 1u;  // (infinities and what is not a number among them)
        exponent[tid / NB][tid % NB] = max(min(e, 60), -60);
    }
    __syncthreads();
    if (tid < a.dim) {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const int e = exponent[i][block];
            const float y = fminf(ldexpf(fabsf(x[i]), -e), 7.5f);
            const float step = y < 2.f ? 0.125f : y < 4.f ? 0.25f : 0.5f;
            const float w = rintf(y / step) * step;
            const int w8 = (int)(w * 8.f);
            const int c = w8 < 16 ? w8 : w8 < 32 ? 16 + ((w8 - 16) >> 1) : 24 + ((w8 - 32) >> 2);
            code[i][block][(jl % S::BPJ) * DP + at] = (uint8_t)(c | (x[i] < 0.f ? 32 : 0));
            rounded[i][j * DP + at] = ldexpf(x[i] < 0.f ? -w : w, e);
        }
    }
    __syncthreads();
    for (int f = tid; f < Q * NB * 6; f += 256) {
        const int i = f / (NB * 6), b = f % (NB * 6) / 6, d = f % 6;
        uint32_t word = 0u;
        for (int p = (32 * d) / 6; p < 32 && 6 * p < 32 * d + 32; ++p) {
            const int shift = 6 * p - 32 * d;
            word |= shift >= 0 ? (uint32_t)code[i][b][p] << shift : (uint32_t)code[i][b][p] >> -shift;
        }
        const int64_t q = q0 + i;  // (past the last query: places of its group that are there)
        a.qimg[(((q >> 5) * S::NS + (b >> 1)) * 6 + d) * 64 + (b & 1) * 32 + (q & 31)] = word;
    }
    if (tid < 2 * Q) {
        const int i = tid >> 1, h = tid & 1;
        uint32_t word = 0u;
#pragma unroll
        for (int t = 0; t < S::NS; ++t) word |= (uint32_t)(127 + exponent[i][2 * t + h]) << (8 * t);
        a.qscale[((q0 + i) >> 5) * 64 + h * 32 + ((q0 + i) & 31)] = word;
    }
    if (tid < Q * M) {
        const int i = tid / M, jj = tid % M;
        float sum = 0.f;
        for (int t = 0; t < DP; ++t) sum += fabsf(rounded[i][jj * DP + t]);
        reach[i][jj] = sum * a.sizes[jj] + a.sizes[M + jj];
    }
    float sum[Q][kLambdas], size[Q][kLambdas];
#pragma unroll
    for (int i = 0; i < Q; ++i)
#pragma unroll
        for (int l = 0; l < kLambdas; ++l) sum[i][l] = size[i][l] = 0.f;
    for (int jj = wave; jj < M; jj += 4) {
        float mn[Q][kLambdas];
        bool number[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            number[i] = true;
#pragma unroll
            for (int l = 0; l < kLambdas; ++l) mn[i][l] = __builtin_inff();
        }
#pragma unroll 1
        for (int r = 0; r < 4; ++r) {
            const int c = lane + 64 * r;
            const v4f *cen = (const v4f *)(a.rounded + (size_t)(jj * 256 + c) * DP);
            float dot[Q] = {}, entry[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i) entry[i] = i < here ? a.lut[((q0 + i) * M + jj) * 256 + c] : 0.f;
#pragma unroll
            for (int t = 0; t < DP / 4; ++t) {
                const v4f v = cen[t];
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    const v4f y = *(const v4f *)&rounded[i][jj * DP + 4 * t];
#pragma unroll
                    for (int u = 0; u < 4; ++u) dot[i] = __builtin_fmaf(v[u], y[u], dot[i]);
                }
            }
            const float half_square = a.norms[jj * 256 + c];
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                const float b = dot[i] - half_square, l = entry[i] * a.half_unit;
                number[i] = number[i] && l < FLT_MAX;
#pragma unroll
                for (int k = 0; k < kLambdas; ++k) mn[i][k] = fminf(mn[i][k], __builtin_fmaf(kLambda[k], l, b));
            }
        }
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            if (!number[i]) bad[i] = 1u;
#pragma unroll
            for (int l = 0; l < kLambdas; ++l) {
                const float m = wave_min_f32(mn[i][l]);
                sum[i][l] += m;
                size[i][l] += fabsf(m);
            }
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int i = 0; i < Q; ++i)
#pragma unroll
            for (int l = 0; l < kLambdas; ++l) {
                sums[wave][i][l] = sum[i][l];
                sizes[wave][i][l] = size[i][l];
            }
    }
    __syncthreads();
    if (tid < Q * kLambdas && tid / kLambdas < here) {
        // Less what rounding may have done to the sums here and to those of the matrix cores: 2^-16 of the largest that
        // the products can add up to in size (they are sums of up to 512 float32 terms), 2^-20 of the terms added here.
        const int i = tid / kLambdas, l = tid % kLambdas;
        float all = 0.f;
        for (int jj = 0; jj < M; ++jj) all += reach[i][jj];
        const float total = sums[0][i][l] + sums[1][i][l] + sums[2][i][l] + sums[3][i][l];
        const float size4 = sizes[0][i][l] + sizes[1][i][l] + sizes[2][i][l] + sizes[3][i][l];
        const float bound = total - 0x1p-16f * all - 0x1p-20f * size4;
        a.s[(q0 + i) * kLambdas + l] = bound;
        if (!(fabsf(bound) < 1e25f) || !(all < 1e25f)) bad[i] = 1u;
    }
    __syncthreads();
    if (tid < here) {
        a.thr[q0 + tid] = kNoEntry;
        a.redo[q0 + tid] = bad[tid];
    }
}

// The kk-th smallest of the workgroup's keys, PER to a thread (256 threads), those not there ~0 (no key is): a radix
// search from the highest bit in which the keys differ.
struct SelectScratch {
    uint32_t hist[256];
    uint32_t lo[4], hi[4];
    uint32_t bin, below, kept, tied;
};
template <int PER>
__device__ __forceinline__ uint32_t kth_smallest(PSC_LDS SelectScratch &s, const uint32_t (&e)[PER], int regs, uint32_t kk)
{
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t lo = ~0u, hi = 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i)
        if (i < regs) {
            lo = min(lo, e[i]);
            hi = e[i] != ~0u ? max(hi, e[i]) : hi;
        }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor(lo, off, 64));
        hi = max(hi, (uint32_t)__shfl_xor(hi, off, 64));
    }
    if (lane == 0) {
        s.lo[wave] = lo;
        s.hi[wave] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        lo = min(lo, s.lo[w]);
        hi = max(hi, s.hi[w]);
    }
    if (lo == hi) return lo;
    const int top = 32 - __builtin_clz(lo ^ hi);
    int width = top < 8 ? top : 8, shift = top - width;
    uint32_t prefix = top == 32 ? 0u : lo >> top, need = kk;
    while (true) {
        s.hist[tid] = 0u;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (i < regs && e[i] != ~0u) {
                const uint32_t d = e[i] >> shift;
                if ((shift + width == 32 ? 0u : d >> width) == prefix)
                    __hip_atomic_fetch_add(&s.hist[d & ((1u << width) - 1u)], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        __syncthreads();
        if (wave == 0) {
            uint32_t h[4], sum = 0u;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                h[i] = s.hist[4 * lane + i];
                sum += h[i];
            }
            uint32_t incl = sum;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t o = __shfl_up(incl, off, 64);
                if (lane >= off) incl += o;
            }
            uint32_t cum = incl - sum;
            if (cum < need && incl >= need) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (cum < need && cum + h[i] >= need) {
                        s.bin = 4u * (uint32_t)lane + (uint32_t)i;
                        s.below = cum;
                    }
                    cum += h[i];
                }
            }
        }
        __syncthreads();
        need -= s.below;
        prefix = (prefix << width) | s.bin;
        if (shift == 0) return prefix;
        width = shift < 8 ? shift : 8;
        shift -= width;
        __syncthreads();  // (bin and below are read)
    }
}

// The sample, tested and scored; the key of the rank-th best distance bounds what follows.  One workgroup per query, four codes
// to a thread and turn; codes that pass the test wait in a queue of their wave until there are 64.  Bound by the trip to L2 for
// a turn's codes and by how many workgroups run at a time, which LDS is to limit: with codes two turns ahead and a pool of 2048
// keys (one turn and 4096) 1000 queries x 15900 codes of 128 bits take 27 us, 86 before, 3000 x 13300 54 and 99.  Left to
// itself the compiler takes registers for four workgroups of 64-bit codes where LDS has room for seven: 1200 queries x 200k,
// ht 28 36 us, 25 so.
constexpr int kSampleRoom = 1024 + 4 * 64;  // keys of a turn: its codes and those that waited
template <int M>
struct SampleLds {
    float lut[M * 256];
    uint32_t pool[kSampleKeys];
    uint32_t queue[4][128 * (M / 4)];
    SelectScratch sel;
    uint32_t count;
};
template <int M>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(M == 8 ? 7 : 4)))
bound_sample_kernel(const uint8_t *__restrict__ codes, const uint8_t *__restrict__ qcodes, const float *__restrict__ luts,
                    int total, uint32_t bias, int rank, int checked, uint32_t most_near, uint32_t most_tied, uint32_t most_alone,
                    uint32_t *__restrict__ unfit, uint32_t *__restrict__ redo, uint64_t *__restrict__ thr)
{
    constexpr int WPC = M / 4;
    typedef uint32_t words __attribute__((ext_vector_type(WPC)));
    __shared__ __align__(16) SampleLds<M> shared;
    PSC_LDS SampleLds<M> &s = *(PSC_LDS SampleLds<M> *)&shared;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // The queries that are asked come first; once enough of them have said so the others have nothing to do here.
    const int asked = ((int)gridDim.x + 7) >> 3, other = (int)blockIdx.x - asked;
    const int64_t q = other < 0 ? (int64_t)blockIdx.x * 8 : other + other / 7 + 1;
    if (redo[q] != 0u) return;  // (uniform)
    if (other >= 0) {
        if (tid == 0) s.count = __hip_atomic_load(unfit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        const uint32_t said = s.count;
        __syncthreads();
        if (said * 64u > gridDim.x) return;
    }
    for (int e = tid; e < M * 64; e += 256) ((PSC_LDS v4i *)s.lut)[e] = ((const v4i *)(luts + q * (M * 256)))[e];
    uint32_t qw[WPC];
#pragma unroll
    for (int w = 0; w < WPC; ++w) qw[w] = __builtin_amdgcn_readfirstlane(((const uint32_t *)qcodes)[q * WPC + w]);
    if (tid == 0) s.count = 0u;
    uint32_t bound = ~0u;  // (inclusive; the same in every thread)
    auto load = [&](int t, words (&c)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int p = t + 256 * i + tid;
            c[i] = p < total ? ((const words *)codes)[p] : words(0u);
        }
    };
    words cur[2][4];  // (two turns ahead)
    load(0, cur[0]);
    load(1024, cur[1]);
    __syncthreads();
    PSC_LDS words *const queue = (PSC_LDS words *)s.queue[wave];
    int fill = 0;
    auto score = [&](int c) {  // the newest c queued codes
        __builtin_amdgcn_wave_barrier();
        fill -= c;
        const words v = lane < c ? queue[fill + lane] : words(0u);
        __builtin_amdgcn_wave_barrier();
        float d = s.lut[v[0] & 0xffu];
#pragma unroll
        for (int j = 1; j < M; ++j) d += s.lut[j * 256 + ((v[j >> 2] >> (8 * (j & 3))) & 0xffu)];
        const uint32_t key = dist_key(d);
        const bool take = lane < c && key <= bound;
        const uint64_t m = ballot64(take);
        uint32_t base = 0u;
        if (lane == 0 && m) base = __hip_atomic_fetch_add(&s.count, (uint32_t)__builtin_popcountll(m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
        if (take) s.pool[base + (uint32_t)prefix_count(m)] = key;  // (kSampleRoom places are kept)
    };
    // the `rank` smallest to the front of the pool's c keys, the largest of them; `more`: how many others are as small
    uint32_t more = 0u;
    auto select = [&](int c) {
        uint32_t e[kSampleKeys / 256];
        const int regs = (c + 255) >> 8;
#pragma unroll
        for (int i = 0; i < kSampleKeys / 256; ++i) e[i] = tid + 256 * i < c ? s.pool[tid + 256 * i] : ~0u;
        const uint32_t kth = kth_smallest(s.sel, e, regs, (uint32_t)rank);
        if (tid == 0) s.sel.kept = s.sel.tied = 0u;
        __syncthreads();
        uint32_t same = 0u;
#pragma unroll
        for (int i = 0; i < kSampleKeys / 256; ++i) {
            if (i < regs && e[i] < kth) s.pool[__hip_atomic_fetch_add(&s.sel.kept, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)] = e[i];
            same += (uint32_t)__builtin_popcountll(ballot64(i < regs && e[i] == kth));
        }
        if (lane == 0) __hip_atomic_fetch_add(&s.sel.tied, same, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __syncthreads();
        const int below = (int)s.sel.kept;
        more = (kth == bound ? more : 0u) + (uint32_t)below + s.sel.tied - (uint32_t)rank;
        if (tid < rank - below) s.pool[below + tid] = kth;
        if (tid == 0) s.count = (uint32_t)rank;
        return kth;
    };
    auto turn = [&](int t, words (&next)[4]) {
        words c[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) c[i] = next[i];
        load(t + 2048, next);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t h = bias;
#pragma unroll
            for (int w = 0; w < WPC; ++w) h += (uint32_t)__popc(c[i][w] ^ qw[w]);
            const bool pass = (int32_t)h >= 0 && t + 256 * i + tid < total;
            const uint64_t m = ballot64(pass);
            if (pass) queue[fill + prefix_count(m)] = c[i];
            fill += __builtin_popcountll(m);
            if (fill >= 64) score(64);
        }
        __syncthreads();
        const int have = (int)s.count;
        __syncthreads();
        if (have > kSampleKeys - kSampleRoom) {
            bound = select(have);
            __syncthreads();
        }
    };
    for (int t = 0; t < total; t += 2048) {
        turn(t, cur[0]);
        if (t + 1024 < total) turn(t + 1024, cur[1]);
    }
    if (fill > 0) score(fill);
    __syncthreads();
    const int have = (int)s.count;
    __syncthreads();
    uint64_t key = kNoEntry;
    if (have >= rank) key = (uint64_t)select(have) << 32 | 0xffffffffull;
    // Equal distances are all listed, and where fewer than `rank` pass the test everything is.  A query that would list a good
    // share of the codes so is left to the other scan at once; one in eight says so of the batch.  It counts twice: from a
    // sixteenth of the queries marked on (few_marked) the other scan goes through all codes for them anyhow (3000 queries x
    // 200k codes of 1000 kinds, 128 bits, ht 48, a seventh marked: 1015 us where each counted once).
    const bool alone = have < rank || (uint32_t)rank + more > most_alone;
    if (tid == 0) {
        thr[q] = key;
        if (alone) redo[q] = 1u;
        if ((q & 7) == 0 && (alone || (checked == 0 && (uint32_t)rank + more > most_tied)))
            __hip_atomic_fetch_add(unfit, alone ? 2u : 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (checked == 0 || alone || (q & 7) != 0) return;
    // How many codes are as near, whether they pass the test or not: those are what the rounds will list.  Where the
    // numbering of the centroids says nothing about distance they are many times those that pass; a batch of which an
    // eighth is so (every eighth query is asked) is left to the other scan before anything is listed (bound_scan_kernel).
    __syncthreads();
    if (tid == 0) s.count = 0u;
    __syncthreads();
    const uint32_t within = (uint32_t)(key >> 32);
    uint32_t near = 0u;
#pragma unroll 4
    for (int p = tid; p < checked; p += 256) {
        const words c = ((const words *)codes)[p];
        float d = s.lut[c[0] & 0xffu];
#pragma unroll
        for (int j = 1; j < M; ++j) d += s.lut[j * 256 + ((c[j >> 2] >> (8 * (j & 3))) & 0xffu)];
        near += dist_key(d) <= within ? 1u : 0u;
    }
    if (near != 0u) __hip_atomic_fetch_add(&s.count, near, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
    if (tid == 0 && s.count > most_near) __hip_atomic_fetch_add(unfit, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Below which key (exclusive) the kk smallest of a wave's keys lie (barriers between the waves of a workgroup would cost
// 13 us for 1000 keys).  The search: the smallest distance at or below which k keys lie, bit by bit with the keys in registers, until exactly k
// lie below the value tried; among equal distances the same search over the ids.
template <int PER>
__device__ __forceinline__ uint64_t wave_select(const uint64_t (&e)[PER], int kk)
{
    // (more than kk keys; those not there are ~0)
    auto below = [&](uint64_t v) {
        int c = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) c += __builtin_popcountll(ballot64(e[i] < v));
        return c;
    };
    auto below_high = [&](uint32_t v) {
        int c = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) c += __builtin_popcountll(ballot64((uint32_t)(e[i] >> 32) < v));
        return c;
    };
    uint32_t lo = ~0u, hi = 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const uint32_t d = (uint32_t)(e[i] >> 32);
        lo = min(lo, d);
        hi = e[i] != kNoEntry ? max(hi, d) : hi;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor(lo, off, 64));
        hi = max(hi, (uint32_t)__shfl_xor(hi, off, 64));
    }
    lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
    hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)hi);
    const int top = lo == hi ? 0 : 32 - __builtin_clz(lo ^ hi);
    uint32_t d = top == 32 ? 0u : lo >> top << top;
    for (int b = top - 1; b >= 0; --b) {
        const uint32_t mid = d | 1u << b;
        const int c = below_high(mid);
        if (c == kk) return (uint64_t)mid << 32;  // (exclusive)
        if (c < kk) d = mid;
    }
    uint64_t v = (uint64_t)d << 32;  // the kk-th key has this distance
    for (int b = 31; b >= 0; --b) {
        const uint64_t mid = v | 1ull << b;
        const int c = below(mid);
        if (c == kk) return mid;
        if (c < kk) v = mid;
    }
    return v + 1u;
}

struct RankArgs {
    const uint8_t *codes, *qcodes;
    const float *lut;
    const uint32_t *near, *first_row;  // (BoundArgs::near, first)
    int cap, groups, tiles, slices;
    uint32_t *redo;
    uint32_t *unfit;
    uint64_t *thr;
    uint32_t bias;  // 0x7fffffff - ht
    int k, rank;    // rank: whose distance bounds the next round
    float ratio;    // the next round's codes to this one's
    uint32_t most;  // rows that are ranked; a query that lists more is marked (most_listed)
    int64_t *ids;
    float *dists;
    // of the last round: where its marks are counted and listed (BoundLayout), unless the batch is unfit (all are marked then)
    uint32_t *marks;
    int few, first, nq;
};
template <int M>
struct RankLds {
    float lut[M * 256];
    uint64_t pool[kBoundPool];
    uint64_t best[kBoundMaxK];
    uint32_t rows[256 * kRun];
    uint32_t part[4];
    uint32_t count;
};
// After a round: what passed the bounds of a query is tested and scored from the tables in LDS, by a workgroup per query;
// its first wave selects the rank-th best, whose key bounds the next round, or (LAST) writes the k best to their ranks.
template <int M, bool LAST>
__global__ void __launch_bounds__(256)
bound_rank_kernel(RankArgs a)
{
    constexpr int WPC = M / 4;
    typedef uint32_t words __attribute__((ext_vector_type(WPC)));
    __shared__ __align__(16) RankLds<M> shared;
    PSC_LDS RankLds<M> &s = *(PSC_LDS RankLds<M> *)&shared;
    PSC_LDS uint64_t *const sel = s.best;
    const int tid = (int)threadIdx.x, lane = tid & 63, k = a.k;
    const int64_t q = blockIdx.x;
    auto list_mark = [&]() {  // (by one thread)
        if (*a.unfit * 64u > (uint32_t)a.nq) return;
        const uint32_t at = __hip_atomic_fetch_add(a.marks, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (at < (uint32_t)a.few) a.marks[kMarkWords + a.few + at] = (uint32_t)a.first + (uint32_t)q;
    };
    if (a.redo[q] != 0u) {  // (uniform)
        if (LAST && tid == 0) list_mark();
        return;
    }
    const uint64_t wanted = a.thr[q];
    const int group = (int)(q >> 5);
    int tile = (int)((int64_t)group * a.tiles / a.groups);  // (that of tile g0 .. g0 + ng - 1 of bound_item)
    while ((int)((int64_t)(tile + 1) * a.groups / a.tiles) <= group) ++tile;
    const int slot = (int)q - (int)((int64_t)tile * a.groups / a.tiles) * 32;
    for (int e = tid; e < M * 64; e += 256) ((PSC_LDS v4i *)s.lut)[e] = ((const v4i *)(a.lut + q * (M * 256)))[e];
    uint32_t qw[WPC];
#pragma unroll
    for (int w = 0; w < WPC; ++w) qw[w] = __builtin_amdgcn_readfirstlane(((const uint32_t *)a.qcodes)[q * WPC + w]);
    if (tid == 0) s.count = 0u;
    // `lanes` threads read a slice's run (every lanes-th row each), up to kRun rows of it at a time; what all of them read
    // fills `rows`.
    const int lanes = a.slices <= 32 ? 8 : a.slices <= 64 ? 4 : a.slices <= 128 ? 2 : 1;
    int slice = tid / lanes;
    uint32_t at = 0u, end = 0u, listed = 0u;
    size_t item = 0;
    while (true) {
        while (at >= end && slice < a.slices) {
            item = (size_t)tile * a.slices + slice;
            at = a.first_row[item * 257 + slot] + (uint32_t)(tid % lanes);
            end = a.first_row[item * 257 + slot + 1];
            slice += 256 / lanes;
        }
        const uint32_t take = at < end ? min((end - at + (uint32_t)lanes - 1u) / (uint32_t)lanes, (uint32_t)kRun) : 0u;
        uint32_t upto = take;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = __shfl_up(upto, off, 64);
            if (lane >= off) upto += o;
        }
        __syncthreads();  // (`part` and `rows` are read)
        if (lane == 63) s.part[tid >> 6] = upto;
        __syncthreads();
        const uint32_t total = s.part[0] + s.part[1] + s.part[2] + s.part[3];
        if (total == 0u) break;  // (uniform)
        listed += total;
        if (listed > a.most) break;  // (uniform)
        for (int w = 0; w < (tid >> 6); ++w) upto += s.part[w];
        const uint32_t *run = a.near + item * a.cap + at;
        uint32_t mine[kRun];
#pragma unroll
        for (uint32_t i = 0; i < (uint32_t)kRun; ++i) mine[i] = i < take ? run[i * (uint32_t)lanes] : 0u;
#pragma unroll
        for (uint32_t i = 0; i < (uint32_t)kRun; ++i)
            if (i < take) s.rows[upto - take + i] = mine[i];
        at += take * (uint32_t)lanes;
        __syncthreads();
        words c[kRun];
        uint32_t id[kRun];
#pragma unroll
        for (int u = 0; u < kRun; ++u) {
            const uint32_t p = 256u * u + (uint32_t)tid;
            id[u] = p < total ? s.rows[p] : ~0u;
            c[u] = id[u] != ~0u ? ((const words *)a.codes)[id[u]] : words(0u);
        }
#pragma unroll
        for (int u = 0; u < kRun; ++u) {
            if (256u * u >= total) break;  // (uniform)
            uint32_t h = a.bias;
#pragma unroll
            for (int w = 0; w < WPC; ++w) h += (uint32_t)__popc(c[u][w] ^ qw[w]);
            float d = s.lut[c[u][0] & 0xffu];
#pragma unroll
            for (int j = 1; j < M; ++j) d += s.lut[j * 256 + ((c[u][j >> 2] >> (8 * (j & 3))) & 0xffu)];
            const uint64_t key = pack_entry(d, id[u]);
            const bool better = id[u] != ~0u && (int32_t)h >= 0 && key <= wanted;
            const uint64_t m = ballot64(better);
            if (m == 0ull) continue;
            uint32_t base = 0u;
            if (lane == 0) base = __hip_atomic_fetch_add(&s.count, (uint32_t)__builtin_popcountll(m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base) + (uint32_t)prefix_count(m);
            if (better && base < (uint32_t)kBoundPool) s.pool[base] = key;
        }
    }
    __syncthreads();
    if (tid >= 64) return;
    const int pooled = (int)s.count;
    if (pooled > kBoundPool || listed > a.most) {
        if (lane == 0) {
            a.redo[q] = 1u;
            if (LAST) list_mark();
        }
        return;
    }
    const int wants = LAST ? k : a.rank;
    // the `wants` best of the pool, a run of it at a time
    int kept = 0;
    auto merge = [&](auto size, int from, int len) {
        constexpr int PER = decltype(size)::value;
        uint64_t e[PER];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int p = lane + 64 * i;
            e[i] = p < kept ? sel[p] : p - kept < len ? s.pool[from + p - kept] : kNoEntry;
        }
        __builtin_amdgcn_wave_barrier();
        const uint64_t cut = kept + len > wants ? wave_select<PER>(e, wants) : kNoEntry;
        int at = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const uint64_t m = ballot64(e[i] < cut);
            if (e[i] < cut) sel[at + prefix_count(m)] = e[i];
            at += __builtin_popcountll(m);
        }
        __builtin_amdgcn_wave_barrier();
        kept = at;
    };
    for (int from = 0; from < pooled;) {
        const int left = pooled - from;
        if (kept + left <= 8 * 64) {
            merge(std::integral_constant<int, 8>{}, from, left);
            from = pooled;
        } else {
            const int len = min(left, 20 * 64 - kept);
            merge(std::integral_constant<int, 20>{}, from, len);
            from += len;
        }
    }
    if constexpr (LAST) {
        // The pool holds all there is up to thr: the k best, unless fewer are that near.
        if (kept < k && wanted != kNoEntry) {
            if (lane == 0) {
                a.redo[q] = 1u;
                list_mark();
            }
            return;
        }
        __builtin_amdgcn_wave_barrier();
        for (int p = lane; p < k; p += 64) {
            if (p < kept) {
                const uint64_t key = sel[p];
                int rank = 0;
                for (int i = 0; i < kept; ++i) rank += sel[i] < key ? 1 : 0;
                a.ids[q * k + rank] = (int64_t)entry_id(key);
                a.dists[q * k + rank] = entry_dist(key);
            } else {
                a.ids[q * k + p] = (int64_t)-1;
                a.dists[q * k + p] = __builtin_inff();
            }
        }
    } else {
        if (kept < a.rank) return;  // (thr stays as it is)
        uint64_t most = 0ull;
        __builtin_amdgcn_wave_barrier();
        for (int p = lane; p < kept; p += 64) most = sel[p] > most ? sel[p] : most;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const uint64_t o = __shfl_xor(most, off, 64);
            most = o > most ? o : most;
        }
        if (lane == 0) a.thr[q] = most;
        if ((q & 7) != 0) return;
        // What the next round will list, codes at equal distances among them (bound_sample_kernel).
        uint32_t near = 0u;
        for (int p = lane; p < pooled; p += 64) near += (uint32_t)(s.pool[p] >> 32) <= (uint32_t)(most >> 32) ? 1u : 0u;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) near += (uint32_t)__shfl_xor((int)near, off, 64);
        if (lane == 0 && (float)near * a.ratio * (float)listed / (float)pooled > (float)kNear)
            __hip_atomic_fetch_add(a.unfit, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

int padded_length(int m, int dsub)
{
    const int dp = dsub <= 8 ? 8 : dsub <= 16 ? 16 : 32;
    return dsub <= 32 && m * dp <= 256 ? dp : 0;
}
int entry_bytes(int dp) { return dp == 8 ? 8 : dp == 16 ? 16 : 32; }

// v (at most 7.5 in size) to the nearest E2M3 number.
float round_e2m3(float v, uint8_t *code)
{
    const float y8 = 8.f * std::fabs(v);
    const int step = y8 < 16.f ? 1 : y8 < 32.f ? 2 : 4;
    const int w8 = std::min((int)(y8 / (float)step + 0.5f) * step, 60);
    *code = (uint8_t)((w8 < 16 ? w8 : w8 < 32 ? 16 + (w8 - 16) / 2 : 24 + (w8 - 32) / 4) | (v < 0.f ? 32 : 0));
    return v < 0.f ? -0.125f * (float)w8 : 0.125f * (float)w8;
}

size_t round256(size_t v) { return (v + 255) / 256 * 256; }

struct BoundLayout {
    size_t marks, unfit, qimg, qscale, s, thr, sample, raw, near, first, total;
};
// How many marked queries are few: scanned by themselves these take less than the tiles that have one (up to 16 queries and
// the whole database each: at a sixteenth, two tiles of three).
int few_marked(int64_t nq) { return (int)std::min<int64_t>((nq + 15) / 16, 1024); }
BoundLayout bound_layout(int m, int dsub, int64_t nq_all)
{
    const int ns = m * padded_length(m, dsub) / 64;
    const int64_t nq = std::min(nq_all, kBoundChunk);
    const size_t groups = (size_t)(nq + 31) / 32;
    BoundLayout l;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += round256(bytes);
        return at;
    };
    l.marks = take((kMarkWords + 2 * (size_t)few_marked(nq_all)) * 4);
    l.unfit = take(4);
    l.qimg = take(groups * ns * 6 * 64 * 4);
    l.qscale = take(groups * 64 * 4);
    l.s = take((size_t)nq * kLambdas * 4);
    l.thr = take((size_t)nq * 8);
    l.sample = take((size_t)kMaxSample * m);
    l.raw = take(groups * 32 * kNear * 4);
    l.near = take(groups * 32 * kNear * 4);
    l.first = take((size_t)kMaxItems * 257 * 4);
    l.total = o;
    return l;
}

int floor_log2(int64_t v)
{
    int l = 0;
    while (v >= 2) {
        v >>= 1;
        ++l;
    }
    return l;
}

// The rank whose distance bounds a round over R times as many codes, so that fewer than k of them are as near in less than 1 of
// 10^7 cases.  After the sample, whose codes need not be among the round's: k - 1 of the round's and all `rank` of the
// sample's are the nearest of both; so too after a round whose stride is no multiple of the next one's (2^a - 1 divides
// 2^b - 1 where a divides b).  After a round over a part of the next one's codes: at least `rank` of the next one's k best were
// among them; at most k.
int rank_after_sample(int k, double ratio)
{
    // Binomial(k + r - 1, p) >= r: less with every r by C(k + r - 1, r) p^r (1 - p)^k
    const double p = 1.0 / (1.0 + ratio);
    double term = std::pow(1.0 - p, k), tail = 1.0;
    int r = 0;
    do {
        tail -= term;
        term *= (double)(k + r) / (double)(r + 1) * p;
        ++r;
    } while (tail > 1e-7);
    return r;
}
int rank_after_round(int k, double ratio)
{
    // Binomial(k, p) >= r
    const double p = 1.0 / ratio;
    double term = std::pow(1.0 - p, k), tail = 1.0;
    int r = 0;
    do {
        tail -= term;
        term *= (double)(k - r) / (double)(r + 1) * (p / (1.0 - p));
        ++r;
    } while (r < k && tail > 1e-7);
    return r;
}

// Sample and rounds for n codes, of which a share `keep` passes the Hamming test at least.
BoundRounds plan_rounds(int64_t n, int k, double keep)
{
    BoundRounds r;
    // The widest step whose lists fit a pool: rank 2^step keys, give or take 2^step sqrt(rank).
    int most = 1;
    while (most < kMostStep) {
        const double rank = rank_after_sample(k, std::ldexp(1.1, most + 1));
        if (std::ldexp(1.1 * (rank + 5.0 * std::sqrt(rank)), most + 1) > kBoundPool) break;
        ++most;
    }
    // The sample: half as many codes again that pass as the rank asks for; no fewer than kLeastSample, and up to twice as
    // many if that saves a round.
    const double sample = std::max((double)kLeastSample, 1.5 * rank_after_sample(k, std::ldexp(1.0, most)) / keep);
    if ((double)n < 4.0 * sample) return r;
    const int fewest = (floor_log2((int64_t)((double)n / std::max(2.0 * kLeastSample, sample))) + most - 1) / most;
    const int top = std::min(floor_log2((int64_t)((double)n / sample)), std::max(1, fewest) * most);
    if ((n >> top) > kMaxSample / 2) return r;
    r.rounds = (top + most - 1) / most;
    auto odd = [](int log) { return log == 0 ? 1 : (1 << log) - 1; };
    int left = top;
    r.stride[0] = odd(top);
    for (int i = 0; i < r.rounds; ++i) {
        left -= (left + r.rounds - i - 1) / (r.rounds - i);  // (the wider steps first)
        r.stride[i + 1] = odd(left);
        const double ratio = (double)r.stride[i] / r.stride[i + 1];
        r.rank[i] = i > 0 && r.stride[i] % r.stride[i + 1] == 0 ? rank_after_round(k, ratio) : rank_after_sample(k, ratio);
    }
    return r;
}

}  // namespace

size_t bound_image_floats(int m, int dsub)
{
    const int dp = padded_length(m, dsub);
    if (dp == 0) return 0;
    return (size_t)m * kCentroids * (entry_bytes(dp) / 4 + dp + 1) + 2 * (size_t)m;
}

bool build_bound_image(const float *centred, int m, int dsub, float *image, BoundCodebook *cb)
{
    *cb = BoundCodebook{};
    const int dp = padded_length(m, dsub);
    if (dp == 0) return false;
    const int bpj = 32 / dp, ns = m * dp / 64, ent = entry_bytes(dp);
    const size_t rows = (size_t)m * kCentroids;
    float most = 0.f;
    for (size_t e = 0; e < rows * dsub; ++e) {
        if (!(std::fabs(centred[e]) < 1e15f)) return false;
        most = std::max(most, std::fabs(centred[e]));
    }
    if (!(most > 1e-15f)) return false;
    const float unit = most / 7.5f;
    const double per_unit = 1.0 / (double)unit;
    std::memset(image, 0, bound_image_floats(m, dsub) * sizeof(float));
    unsigned char *entries = (unsigned char *)image;
    float *rounded = image + rows * (ent / 4), *norms = rounded + rows * dp, *sizes = norms + rows;
    // exponents of the blocks: the largest coordinate of each between 3.75 and 7.5
    int exponent[16];
    auto block_of = [&](int j) { return (j % (m / 2)) / bpj * 2 + j / (m / 2); };
    float block_most[16] = {};
    for (int j = 0; j < m; ++j)
        for (size_t e = 0; e < (size_t)kCentroids * dsub; ++e)
            block_most[block_of(j)] = std::max(block_most[block_of(j)], std::fabs(centred[(size_t)j * kCentroids * dsub + e]) / unit);
    for (int b = 0; b < 2 * ns; ++b) {
        int e = 0;
        while (e > -20 && std::ldexp(block_most[b], -(e - 1)) <= 7.5f) --e;
        exponent[b] = e;
    }
    for (int h = 0; h < 2; ++h)
        for (int t = 0; t < ns; ++t) cb->scale[h] |= (uint32_t)(127 + exponent[2 * t + h]) << (8 * t);
    float down[16], up[16];
    for (int b = 0; b < 2 * ns; ++b) {
        up[b] = std::ldexp(1.f, exponent[b]);
        down[b] = 1.f / (unit * up[b]);
    }
    std::vector<uint8_t> code(rows * dp);
    for (int j = 0; j < m; ++j)
        for (size_t r = (size_t)j * kCentroids; r < ((size_t)j + 1) * kCentroids; ++r)
            for (int t = 0; t < dsub; ++t) {
                const float v = std::max(-7.5f, std::min(7.5f, centred[r * dsub + t] * down[block_of(j)]));
                rounded[r * dp + t] = round_e2m3(v, &code[r * dp + t]) * up[block_of(j)];
                sizes[j] = std::max(sizes[j], std::fabs(rounded[r * dp + t]));
            }
    // What is taken from the product: the half square, less what the rounding of the centroid takes from its product with
    // a query close to it (q.(c - R) is near c.(c - R) for those that matter: a third as many codes pass the bound).
    float norm_most = 0.f;
    for (int j = 0; j < m; ++j)
        for (int c = 0; c < kCentroids; ++c) {
            const size_t r = (size_t)j * kCentroids + c;
            double sq = 0.0, off = 0.0;
            for (int t = 0; t < dsub; ++t) {
                const double v = (double)centred[r * dsub + t] * per_unit;
                sq += v * v;
                off += v * (v - rounded[r * dp + t]);
            }
            norms[r] = (float)std::max(0.5 * sq - off, 0.0);
            norm_most = std::max(norm_most, norms[r]);
        }
    cb->norm_grid = 1.f;
    if (dp == 8) {  // 16 bits of them: whole multiples of a power of two
        int e = -20;
        while (std::ldexp(65535.f, e) < norm_most) ++e;
        cb->norm_grid = std::ldexp(1.f, e);
        for (size_t r = 0; r < rows; ++r) norms[r] = std::min(65535.f, std::nearbyint(norms[r] / cb->norm_grid)) * cb->norm_grid;
    }
    for (int j = 0; j < m; ++j) {
        for (int c = 0; c < kCentroids; ++c) {
            const size_t r = (size_t)j * kCentroids + c;
            sizes[m + j] = std::max(sizes[m + j], norms[r]);
            uint32_t bits[6] = {};
            for (int t = 0; t < dp; ++t) {
                const uint64_t v = (uint64_t)code[r * dp + t] << (6 * t % 32);
                bits[6 * t / 32] |= (uint32_t)v;
                if (v >> 32) bits[6 * t / 32 + 1] |= (uint32_t)(v >> 32);
            }
            uint32_t *out = (uint32_t *)(entries + r * ent), norm;
            std::memcpy(&norm, &norms[r], 4);
            if (dp == 32) {
                for (int i = 0; i < 6; ++i) out[i] = bits[i];
                out[6] = norm;
            } else if (dp == 16) {  // (the odd sub-quantizer of a pair: its first word where the other's half square lands)
                if (j % 2 == 0) {
                    for (int i = 0; i < 3; ++i) out[i] = bits[i];
                } else {
                    out[0] = bits[1];
                    out[1] = bits[2];
                    out[2] = bits[0];
                }
                out[3] = norm;
            } else {
                const uint32_t n16 = (uint32_t)(norms[r] / cb->norm_grid);
                if (j % 2 == 0) {
                    out[0] = bits[0];
                    out[1] = (bits[1] & 0xffffu) | n16 << 16;
                } else {  // 48 bits that follow the even one's
                    out[0] = bits[0] << 16 | n16;
                    out[1] = bits[0] >> 16 | bits[1] << 16;
                }
            }
        }
    }
    cb->per_unit = 1.f / unit;
    cb->half_unit = (float)(1.0 / (2.0 * (double)unit * unit));
    cb->usable = true;
    return true;
}

namespace {
bool sizes_fit(int m, int dsub, int64_t nq, int64_t n, int k)
{
    return padded_length(m, dsub) != 0 && nq >= kBoundMinQueries && n >= kBoundMinCodes && n * m <= 0x7fffffffLL && k <= kBoundMaxK;
}
}  // namespace

// The time of a search by bounds against that of launch_scan's kernels with the tables' (12 us more), both estimated; in
// microseconds, fitted to 337 searches (16 .. 1500 queries x 100k .. 3M codes, k = 10 and 100, five thresholds): taken where
// it was slower by more than 5 % in 3 of them, 0.692 of the time before in geometric mean, 0.681 if the faster one were
// always taken.  That was on mixtures, and what the data is cannot be told beforehand: Gaussian vectors, of which many codes
// are as near as those that pass the test, are given up after the sample.
// Thresholds that let fewer than 1 random pair of 500 through (64 bits: below 21, 128 bits: below 48) are left to the
// Hamming filter: the k-th best among so few is far, and less is gained where the bounds hold than lost where they do not.
// With / without the bounds, k = 100, mixture and Gaussian vectors: 3000 queries x 200k 64 bits ht 20 340 / 461 and 500 /
// 388 us, ht 21 327 / 464 and 489 / 393, ht 24 347 / 606 and 613 / 530; 128 bits ht 47 379 / 467 and 399 / 281, ht 48
// 358 / 479 and 419 / 318, ht 50 377 / 526 and 510 / 419; 1000 x 1M 128 bits ht 46 307 / 402 and 329 / 256, ht 48 329 /
// 419 and 364 / 298.
// Filtered searches of 128-bit codes have a time of their own beside that of the others, whichever is longer, fitted to 292
// (20 .. 5000 queries x 100k .. 3.2M, k = 10 .. 200, ht 48, 56, 60): on mixtures 0.45 of the time before in geometric mean,
// more than 4 % slower in 2; on Gaussian vectors 0.66, more than 8 % slower in 62.  E.g. with / without, mixture and Gaussian:
// 2500 x 100k, k = 200, ht 60 333 / 531 and 429 / 547 us, 5000 x 1.6M, k = 10, ht 48 1156 / 1497 and 1351 / 1258, both taken;
// 1200 x 200k, k = 10, ht 48 184 / 207 and 239 / 161, 600 x 200k, k = 200, ht 48 178 / 130 and 415 / 122, neither.
// Past the sizes of the fit: 4000 x 4M 64 bits ht 24 1.80 / 2.46 ms (Gaussian 2.37 / 2.28), 128 bits ht 48 2.03 / 3.20 (2.71
// / 2.58), 10k x 10M 9.98 / 14.1 and 10.6 / 25.3; of 64-bit codes more than some 30M have too many at every distance:
// 3000 x 100M 45.0 / 43.0 ms (ht 24), 206 / 203 (nothing filtered), given up in the rounds.
// (The plan of the rounds comes last: it takes longer than the estimates.)
bool bound_search_pays(int m, int dsub, int64_t nq, int64_t n, int ht, int k, size_t ws_bytes, BoundRounds *plan)
{
    if (!sizes_fit(m, dsub, nq, n, k)) return false;
    const double keep = ht >= 8 * m ? 1.0 : random_code_survival(8 * m, ht);
    if (keep < 0.002) return false;
    const double padded = (double)((nq + 31) / 32 * 32), steps = m * padded_length(m, dsub) / 64, size = std::log2((double)n / 1e5);
    double bounds = 65.0 + 9.6 * size + 0.042 * (double)nq * (1.0 + k / 100.0) + 0.5 * steps * 9.75e-8 * padded * (double)n + 0.7 * m;
    if (m == 16 && ht < 128)
        bounds = std::max(bounds, 65.0 + 11.5 * size + 0.14 * k + (0.058 + 2.2e-4 * k) * (double)nq + 0.5 * steps * 1.13e-7 * padded * (double)n);
    if (bounds >= 0.9 * (estimated_scan_time(m, nq, n, k, ht, ws_bytes) + 12.0)) return false;
    *plan = plan_rounds(n, k, keep);
    return plan->rounds != 0;
}

size_t bound_scratch_bytes(int m, int dsub, int64_t nq) { return padded_length(m, dsub) != 0 ? bound_layout(m, dsub, nq).total : 0; }

size_t bound_workspace_bytes(int m, int dsub, int64_t nq, int64_t n, int k)
{
    // (the thresholds at which the other kernels take longest: nothing filtered, and the last before the dense route)
    const size_t any = (size_t)1 << 60;
    BoundRounds plan;
    for (int ht : {8 * m, m == 8 ? 29 : 61})
        if (bound_search_pays(m, dsub, nq, n, ht, k, any, &plan)) return bound_scratch_bytes(m, dsub, nq);
    return 0;
}

namespace {

template <int M, int DP>
int run_bound(const BoundSearch &b, int64_t q_first, int nq, const BoundLayout &l, const BoundRounds &plan, hipStream_t s)
{
    using S = Shape<M, DP>;
    static std::atomic<bool> configured{false};  // the dynamic-LDS ceiling, once
    const size_t lds = sizeof(BoundLds<M, DP>);
    if (!configured.load(std::memory_order_acquire)) {
        PSC_HIP_TRY(hipFuncSetAttribute((const void *)bound_scan_kernel<M, DP>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        configured.store(true, std::memory_order_release);
    }
    char *w = (char *)b.ws;
    const size_t rows = (size_t)M * kCentroids;
    const float *entries = b.image, *rounded = entries + rows * (S::ENT / 4), *norms = rounded + rows * DP, *sizes = norms + rows;
    const float *lut = b.lut + (size_t)q_first * rows;
    const uint8_t *qcodes = b.qcodes + (size_t)q_first * M;
    uint32_t *redo = b.redo + q_first;
    uint64_t *thr = (uint64_t *)(w + l.thr);

    PrepareArgs p;
    p.x = b.q + (size_t)q_first * b.dim;
    p.mu = b.mu;
    p.lut = lut;
    p.rounded = rounded;
    p.norms = norms;
    p.sizes = sizes;
    p.per_unit = b.cb.per_unit;
    p.half_unit = b.cb.half_unit;
    p.qimg = (uint32_t *)(w + l.qimg);
    p.qscale = (uint32_t *)(w + l.qscale);
    p.s = (float *)(w + l.s);
    p.thr = thr;
    p.redo = redo;
    p.dim = b.dim;
    p.dsub = b.dsub;
    p.nq = nq;
    p.query_groups = (nq + 31) / 32 * 8;
    p.codes = b.codes;
    p.sample = (uint8_t *)(w + l.sample);
    p.unfit = (uint32_t *)(w + l.unfit);
    p.few = few_marked(b.nq);
    uint32_t *const marks = (uint32_t *)(w + l.marks);
    p.marks = q_first == 0 ? marks : nullptr;
    p.stride = plan.stride[0];
    p.samples = (int)((b.n + p.stride - 1) / p.stride);
    hipLaunchKernelGGL((bound_prepare_kernel<M, DP>), dim3((unsigned)(p.query_groups + (p.samples + 255) / 256)), dim3(256), 0, s, p);
    PSC_HIP_TRY(hipGetLastError());

    const int ht = std::min(b.ht, 8 * M);
    const uint32_t bias = 0x7fffffffu - (uint32_t)ht;
    // A query is unfit if three times the codes of the first round that are as near (of which the test lets some through:
    // counted over part of the sample; without a test they are those at equal distances) are more than its share of the lists.
    const int checked = ht < 8 * M ? std::min(p.samples, 2048) : 0;
    const double ratio = (double)plan.stride[0] / plan.stride[1], codes_in = (double)b.n / plan.stride[1];
    const uint32_t most_near = (uint32_t)((double)checked / p.samples * kNear / (3.0 * ratio)) + 8u;
    const uint32_t most_tied = (uint32_t)(kNear / (3.0 * ratio)) + 8u, most_alone = (uint32_t)(most_listed(codes_in) / ratio);
    hipLaunchKernelGGL((bound_sample_kernel<M>), dim3((unsigned)nq), dim3(256), 0, s, p.sample, qcodes, lut, p.samples,
                       bias, plan.rank[0], checked, most_near, most_tied, most_alone, p.unfit, redo, thr);
    PSC_HIP_TRY(hipGetLastError());

    BoundArgs a;
    a.codes = b.codes;
    a.img = entries;
    a.qimg = p.qimg;
    a.qscale = p.qscale;
    a.s = p.s;
    a.thr = thr;
    a.redo = redo;
    a.unfit = p.unfit;
    a.raw = (uint32_t *)(w + l.raw);
    a.near = (uint32_t *)(w + l.near);
    a.first = (uint32_t *)(w + l.first);
    a.n = (int)b.n;
    a.nq = nq;
    a.groups = (nq + 31) / 32;
    a.tiles = (a.groups + S::QG - 1) / S::QG;
    a.half_unit = b.cb.half_unit;
    a.scale_lo = b.cb.scale[0];
    a.scale_hi = b.cb.scale[1];
    a.norm_grid = b.cb.norm_grid;
    RankArgs r;
    r.codes = b.codes;
    r.qcodes = qcodes;
    r.lut = lut;
    r.near = a.near;
    r.first_row = a.first;
    r.groups = a.groups;
    r.tiles = a.tiles;
    r.redo = redo;
    r.thr = thr;
    r.unfit = p.unfit;
    r.bias = bias;
    r.k = b.k;
    r.ids = b.ids + (size_t)q_first * b.k;
    r.dists = b.dists + (size_t)q_first * b.k;
    r.marks = marks;
    r.few = p.few;
    r.first = (int)q_first;
    r.nq = nq;
    for (int i = 0; i < plan.rounds; ++i) {
        const bool last = i + 1 == plan.rounds;
        a.stride = plan.stride[i + 1];
        a.codes_in = (int)((b.n + a.stride - 1) / a.stride);
        a.blocks = (a.codes_in + kBlock - 1) / kBlock;
        // Two workgroups a compute unit, and no more: the items are alike, and a workgroup's start and its sorting of what it
        // listed take as long as 2000 codes.  A place in a
        // slice has 24 bits.
        a.slices = (int)std::max<int64_t>((a.blocks + (1 << 17) - 1) >> 17, std::min<int64_t>((a.blocks + 3) / 4, 512 / a.tiles));
        const int total = a.tiles * a.slices;
        PSC_REQUIRE(total <= kMaxItems, "too many work items");
        a.cap = (int)((int64_t)a.groups * 32 * kNear / total);
        hipLaunchKernelGGL((bound_scan_kernel<M, DP>), dim3((unsigned)((total + 7) / 8 * 8)), dim3(256), lds, s, a);
        PSC_HIP_TRY(hipGetLastError());
        r.cap = a.cap;
        r.slices = a.slices;
        r.most = (uint32_t)most_listed((double)a.codes_in);
        r.rank = last ? 0 : plan.rank[i + 1];
        r.ratio = last ? 1.f : (float)a.stride / (float)plan.stride[i + 2];
        if (last) hipLaunchKernelGGL((bound_rank_kernel<M, true>), dim3((unsigned)nq), dim3(256), 0, s, r);
        else hipLaunchKernelGGL((bound_rank_kernel<M, false>), dim3((unsigned)nq), dim3(256), 0, s, r);
        PSC_HIP_TRY(hipGetLastError());
    }
    char route[96];
    snprintf(route, sizeof route, "bound_scan_kernel m=%d tq=%d waves=4 slices=%d tiles=%lld", M, S::QG * 32, a.slices,
             (long long)a.tiles * a.slices);
    note_scan_route(route);
    return PSC_OK;
}

}  // namespace

int launch_bound_search(const BoundSearch &b, MarkedQueries *marked, hipStream_t s)
{
    const int dp = padded_length(b.m, b.dsub);
    const BoundRounds &plan = b.plan;
    PSC_REQUIRE(dp != 0 && plan.rounds > 0, "sizes without a bound search");
    const BoundLayout l = bound_layout(b.m, b.dsub, b.nq);
    uint32_t *marks = (uint32_t *)((char *)b.ws + l.marks);
    marked->few = few_marked(b.nq);
    marked->redo = b.redo;
    marked->count = marks;
    marked->arrived = marks + kMarkWords;
    marked->which = (const int32_t *)(marks + kMarkWords + marked->few);
    marked->scratch = (char *)b.ws + l.raw;  // (the lists are read by then)
    marked->scratch_bytes = l.total - l.raw;
    for (int64_t q = 0; q < b.nq; q += kBoundChunk) {
        const int nq = (int)std::min(kBoundChunk, b.nq - q);
        int rc = PSC_EINVAL;
        if (b.m == 8 && dp == 8) rc = run_bound<8, 8>(b, q, nq, l, plan, s);
        if (b.m == 8 && dp == 16) rc = run_bound<8, 16>(b, q, nq, l, plan, s);
        if (b.m == 8 && dp == 32) rc = run_bound<8, 32>(b, q, nq, l, plan, s);
        if (b.m == 16 && dp == 8) rc = run_bound<16, 8>(b, q, nq, l, plan, s);
        if (b.m == 16 && dp == 16) rc = run_bound<16, 16>(b, q, nq, l, plan, s);
        if (rc != PSC_OK) return rc;
    }
    return PSC_OK;
}

}  // namespace psc
