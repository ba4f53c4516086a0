// Inverted-file variant (Section 2 "Non-exhaustive search", Section 4.3): coarse quantizer,
// selection of the lists to probe, and the device-side bookkeeping that turns the
// (query, probed list) jobs into list-major tiles for the fused scan.
//
// A query probes the nprobe coarse centroids nearest to it (squared L2 in float32, lower list
// number on equal distance; the three distance kernels -- plain, a handful of rows, matrix cores
// -- add the coordinates up in different orders, so they can rank two centroids that are equally
// near within float32 rounding differently).  Jobs are then grouped by list so
// that the codes of a list are streamed once per tile of up to TQ queries that probe it.
#include "common.h"

namespace psc {
namespace {

constexpr int kRows = 16;  // rows per workgroup in the distance kernels
// Up to this many rows (queries) the coarse stage runs the kernels built for latency: many
// workgroups per row instead of many rows per workgroup (from 256 rows the distances come from the
// matrix-core kernel where it is built for the dimension; the selection keeps a workgroup per row).
constexpr int64_t kFewRowsMax = 512;

// dist[r][c] = || x_r - cent_c ||^2 for a tile of kRows rows and 256 centroids per workgroup.
// Rows sit in LDS (read as broadcasts), each thread walks its own centroid row.
__global__ void __launch_bounds__(256)
coarse_dist_kernel(const float *__restrict__ x, int64_t n, int dim, const float *__restrict__ cent,
                   int nlist, float *__restrict__ dist)
{
    extern __shared__ __align__(16) float rows[];  // [kRows][dim]
    const int64_t r0 = (int64_t)blockIdx.x * kRows;
    for (int e = threadIdx.x; e < kRows * dim; e += 256) {
        const int64_t r = r0 + e / dim;
        rows[e] = r < n ? x[r * dim + e % dim] : 0.f;
    }
    __syncthreads();
    const int c = blockIdx.y * 256 + threadIdx.x;
    if (c >= nlist) return;
    const float *crow = cent + (int64_t)c * dim;
    float acc[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) acc[r] = 0.f;
    for (int d = 0; d < dim; d += 4) {
        const float4 cv = *(const float4 *)(crow + d);
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const float4 xv = *(const float4 *)(rows + r * dim + d);
            float t = xv.x - cv.x;
            acc[r] = fmaf(t, t, acc[r]);
            t = xv.y - cv.y;
            acc[r] = fmaf(t, t, acc[r]);
            t = xv.z - cv.z;
            acc[r] = fmaf(t, t, acc[r]);
            t = xv.w - cv.w;
            acc[r] = fmaf(t, t, acc[r]);
        }
    }
#pragma unroll
    for (int r = 0; r < kRows; ++r)
        if (r0 + r < n) dist[(r0 + r) * nlist + c] = acc[r];
}

// The same distances for a handful of rows (a single query is the case that matters): one
// workgroup = 32 centroids x up to kFewRows rows, 8 lanes to a centroid, each lane taking every
// eighth group of 4 coordinates, so that the centroid rows are read in 128-byte pieces by many
// workgroups at once instead of one row per thread.  The 8 partial sums are added pairwise, so a
// distance can differ from coarse_dist_kernel's in its last bits.
constexpr int kFewRows = 4;

__global__ void __launch_bounds__(256)
coarse_dist_few_kernel(const float *__restrict__ x, int64_t n, int dim, const float *__restrict__ cent,
                       int nlist, float *__restrict__ dist)
{
    extern __shared__ __align__(16) float rows[];  // [kFewRows][dim]
    const int64_t r0 = (int64_t)blockIdx.y * kFewRows;
    for (int e = threadIdx.x; e < kFewRows * dim; e += 256) {
        const int64_t r = r0 + e / dim;
        rows[e] = r < n ? x[r * dim + e % dim] : 0.f;
    }
    __syncthreads();
    const int sub = threadIdx.x & 7;
    const int c = blockIdx.x * 32 + (threadIdx.x >> 3);
    float acc[kFewRows];
#pragma unroll
    for (int r = 0; r < kFewRows; ++r) acc[r] = 0.f;
    if (c < nlist) {
        const float *crow = cent + (int64_t)c * dim;
        for (int d = sub * 4; d < dim; d += 32) {
            const float4 cv = *(const float4 *)(crow + d);
#pragma unroll
            for (int r = 0; r < kFewRows; ++r) {
                const float4 xv = *(const float4 *)(rows + r * dim + d);
                float t = xv.x - cv.x;
                acc[r] = fmaf(t, t, acc[r]);
                t = xv.y - cv.y;
                acc[r] = fmaf(t, t, acc[r]);
                t = xv.z - cv.z;
                acc[r] = fmaf(t, t, acc[r]);
                t = xv.w - cv.w;
                acc[r] = fmaf(t, t, acc[r]);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < kFewRows; ++r) {
        acc[r] += __shfl_xor(acc[r], 1, 64);
        acc[r] += __shfl_xor(acc[r], 2, 64);
        acc[r] += __shfl_xor(acc[r], 4, 64);
        if (sub == 0 && c < nlist && r0 + r < n) dist[(r0 + r) * nlist + c] = acc[r];
    }
}

__device__ __forceinline__ uint64_t order_key(float d, uint32_t idx)
{
    const uint32_t u = __float_as_uint(d + 0.0f);
    const uint32_t key = u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
    return ((uint64_t)key << 32) | idx;
}

__device__ __forceinline__ uint64_t wave_min_u64(uint64_t v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const uint64_t o = __shfl_xor(v, off, 64);
        v = o < v ? o : v;
    }
    return v;
}

// Sum of v over the wave, in every lane (row-local steps on the data-parallel path, the four row
// sums through scalar registers).
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, false);   // lane ^ 1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, false);   // lane ^ 2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, false);  // mirror in 8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, false);  // mirror in 16
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 0) + (uint32_t)__builtin_amdgcn_readlane((int)v, 16) +
           (uint32_t)__builtin_amdgcn_readlane((int)v, 32) + (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
}

// The nprobe nearest lists of a row, one wave per row, the row's nlist <= 64 KPL distance keys
// in registers (lane l holds lists l, l + 64, ...).
//  1. the nprobe-th smallest distance key, bit by bit: a bit of the answer is 0 iff at least
//     nprobe keys lie below (the bits found so far, this bit set);
//  2. selected = keys below it, plus the lowest-numbered lists among the keys equal to it;
//  3. the selected (key, list) pairs go to LDS and every one is written to its rank.
template <int KPL>
__global__ void __launch_bounds__(256)
select_probes_wave_kernel(const float *__restrict__ dist, int64_t n, int nlist, int nprobe,
                          const int32_t *__restrict__ settled, int32_t *__restrict__ probed)
{
    extern __shared__ __align__(16) uint64_t sel[];  // [4][nprobe]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t r = (int64_t)blockIdx.x * 4 + wave;
    if (r >= n) return;
    if (settled && settled[r] >= 0) return;  // (the waves of a workgroup meet at no barrier)
    uint64_t *mine = sel + (size_t)wave * nprobe;
    uint32_t dk[KPL];
#pragma unroll
    for (int i = 0; i < KPL; ++i) {
        const int c = i * 64 + lane;
        // (real keys stay below the filler of the places past the last list, whatever the distance)
        dk[i] = c < nlist ? min((uint32_t)(order_key(dist[r * nlist + c], 0u) >> 32), 0xfffffffeu) : 0xffffffffu;
    }
    uint32_t pivot = 0;
    for (int b = 31; b >= 0; --b) {
        const uint32_t mid = pivot | (1u << b);
        uint32_t cnt = 0;
#pragma unroll
        for (int i = 0; i < KPL; ++i) cnt += dk[i] < mid ? 1u : 0u;
        if (wave_sum_u32(cnt) < (uint32_t)nprobe) pivot = mid;
    }
    uint32_t below = 0;
#pragma unroll
    for (int i = 0; i < KPL; ++i) below += dk[i] < pivot ? 1u : 0u;
    int take = nprobe - (int)wave_sum_u32(below);  // how many of the keys equal to the pivot belong
    int at = 0;                                     // selected so far
#pragma unroll
    for (int i = 0; i < KPL; ++i) {
        const bool eq = dk[i] == pivot;
        const uint64_t eqm = __ballot(eq);
        const int before = __builtin_popcountll(eqm & ((1ull << lane) - 1ull));
        const bool chosen = dk[i] < pivot || (eq && before < take);
        take -= __builtin_popcountll(eqm);
        const uint64_t cm = __ballot(chosen);
        if (chosen) mine[at + __builtin_popcountll(cm & ((1ull << lane) - 1ull))] = ((uint64_t)dk[i] << 32) | (uint32_t)(i * 64 + lane);
        at += __builtin_popcountll(cm);
    }
    __builtin_amdgcn_wave_barrier();
    for (int e = lane; e < nprobe; e += 64) {
        const uint64_t key = mine[e];
        int rank = 0;
        for (int j = 0; j < nprobe; ++j) rank += mine[j] < key ? 1 : 0;
        probed[r * nprobe + rank] = (int32_t)(uint32_t)key;
    }
}

// The same selection by a whole workgroup of 16 waves per row, for a handful of rows (a single
// query is the case that matters): thread t holds lists t, t + 1024, ...  The nprobe-th smallest
// (distance, list) pair is found by a radix search over the bits of the distance key and, only if
// several lists share that distance, bit by bit over the 14 bits of the list number, with one
// workgroup-wide count per bit (per-wave sums through LDS, two buffers in turn so that one barrier
// per bit is enough).  Bound by its chain of barriers: 34 of them counting bit by bit, 9 to 15 now.  The
// pairs up to it are exactly the nprobe lists; each goes to its rank.
template <int KPL>
__global__ void __launch_bounds__(1024)
select_probes_block_kernel(const float *__restrict__ dist, int nlist, int nprobe, const int32_t *__restrict__ settled,
                           int32_t *__restrict__ probed)
{
    __shared__ uint32_t part[2][16];
    __shared__ uint64_t sel[1024];
    __shared__ uint32_t nsel;
    __shared__ uint32_t hist[256], found[3];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t r = blockIdx.x;
    if (settled && settled[r] >= 0) return;  // (the whole workgroup: one row)
    uint32_t dk[KPL];
#pragma unroll
    for (int i = 0; i < KPL; ++i) {
        const int c = i * 1024 + tid;
        dk[i] = c < nlist ? min((uint32_t)(order_key(dist[r * nlist + c], 0u) >> 32), 0xfffffffeu) : 0xffffffffu;
    }
    if (tid == 0) nsel = 0u;
    int turn = 0;
    // number of keys for which `below(i)` holds, over the whole workgroup
    auto count = [&](auto below) {
        uint32_t cnt = 0;
#pragma unroll
        for (int i = 0; i < KPL; ++i) cnt += below(i) ? 1u : 0u;
        cnt = wave_sum_u32(cnt);
        if (lane == 0) part[turn][wave] = cnt;
        __syncthreads();
        uint32_t total = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) total += part[turn][w];
        turn ^= 1;
        return total;
    };
    // The pivot: a key with nprobe keys at or below it, of which those at the nprobe-th smallest distance
    // are the largest.  The bits in which the keys differ are searched eight at a time, by a histogram of
    // the keys that share the bits found so far; a search ends as soon as a whole bin is taken.
    uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
    for (int i = 0; i < KPL; ++i) {
        if (i * 1024 + tid >= nlist) continue;
        lo = min(lo, dk[i]);
        hi = max(hi, dk[i]);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, off, 64));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, off, 64));
    }
    if (lane == 0) {
        part[0][wave] = lo;
        part[1][wave] = hi;
    }
    if (tid < 256) hist[tid] = 0u;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        lo = min(lo, part[0][w]);
        hi = max(hi, part[1][w]);
    }
    uint32_t pivot = lo;  // (all keys equal)
    if (lo != hi) {
        const int top = 32 - __builtin_clz(lo ^ hi);
        int width = top < 8 ? top : 8, shift = top - width;
        uint32_t prefix = top == 32 ? 0u : lo >> top, need = (uint32_t)nprobe;
        while (true) {
#pragma unroll
            for (int i = 0; i < KPL; ++i) {
                const uint32_t d = dk[i] >> shift;
                if (i * 1024 + tid < nlist && (shift + width == 32 ? 0u : d >> width) == prefix)
                    atomicAdd(&hist[d & ((1u << width) - 1u)], 1u);
            }
            __syncthreads();
            if (wave == 0) {
                uint32_t h[4], sum = 0u;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    h[i] = hist[4 * lane + i];
                    sum += h[i];
                }
                uint32_t incl = sum;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const uint32_t o = (uint32_t)__shfl_up((int)incl, off, 64);
                    if (lane >= off) incl += o;
                }
                uint32_t cum = incl - sum;
                if (cum < need && incl >= need) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (cum < need && cum + h[i] >= need) {
                            found[0] = 4u * lane + i;
                            found[1] = cum;
                            found[2] = h[i];
                        }
                        cum += h[i];
                    }
                }
            }
            __syncthreads();
            const uint32_t inside = found[2];
            need -= found[1];
            prefix = (prefix << width) | found[0];
            if (inside == need || shift == 0) {
                pivot = min(((prefix + 1u) << shift) - 1u, 0xfffffffeu);  // (below the places past the last list)
                break;
            }
            width = shift < 8 ? shift : 8;
            shift -= width;
            if (tid < 256) hist[tid] = 0u;
            __syncthreads();
        }
    }
    __syncthreads();  // (`part` and `found` are read)
    // lists at the pivot distance: all of them belong unless they are too many; then the
    // lowest-numbered ones do, up to list number `last`
    const uint32_t below = count([&](int i) { return dk[i] < pivot; });
    const uint32_t upto = count([&](int i) { return dk[i] <= pivot; });
    uint32_t last = 0xffffffffu;
    if (upto > (uint32_t)nprobe) {
        const uint32_t want = (uint32_t)nprobe - below;  // >= 1
        uint32_t lp = 0;
        for (int b = 13; b >= 0; --b) {
            const uint32_t mid = lp | (1u << b);
            if (count([&](int i) { return dk[i] == pivot && (uint32_t)(i * 1024 + tid) < mid; }) < want) lp = mid;
        }
        last = lp;
    }
#pragma unroll
    for (int i = 0; i < KPL; ++i) {
        const uint32_t c = (uint32_t)(i * 1024 + tid);
        if (dk[i] < pivot || (dk[i] == pivot && c <= last)) {
            const uint32_t slot = atomicAdd(&nsel, 1u);
            if (slot < 1024u) sel[slot] = ((uint64_t)dk[i] << 32) | c;  // (exactly nprobe <= 1024 pass)
        }
    }
    __syncthreads();
    if (tid < nprobe) {
        const uint64_t key = sel[tid];
        int rank = 0;
        for (int j = 0; j < nprobe; ++j) rank += sel[j] < key ? 1 : 0;
        probed[r * nprobe + rank] = (int32_t)(uint32_t)key;
    }
}

// More than 4096 lists.  One workgroup per row: nprobe times take the smallest remaining
// (distance, list) key.
__global__ void __launch_bounds__(256)
select_probes_kernel(const float *__restrict__ dist, int nlist, int nprobe, const int32_t *__restrict__ settled,
                     int32_t *__restrict__ probed)
{
    extern __shared__ __align__(16) uint64_t keys[];  // [nlist]
    __shared__ uint64_t wave_best[4];
    const int64_t r = blockIdx.x;
    if (settled && settled[r] >= 0) return;  // (the whole workgroup: one row)
    for (int c = threadIdx.x; c < nlist; c += 256) keys[c] = order_key(dist[r * nlist + c], (uint32_t)c);
    __syncthreads();
    for (int p = 0; p < nprobe; ++p) {
        uint64_t best = ~0ull;
        for (int c = threadIdx.x; c < nlist; c += 256) {
            const uint64_t v = keys[c];
            best = v < best ? v : best;
        }
        best = wave_min_u64(best);
        if ((threadIdx.x & 63) == 0) wave_best[threadIdx.x >> 6] = best;
        __syncthreads();
        uint64_t b = wave_best[0];
#pragma unroll
        for (int w = 1; w < 4; ++w) b = wave_best[w] < b ? wave_best[w] : b;
        const uint32_t sel = (uint32_t)b;
        if (threadIdx.x == 0) {
            probed[r * nprobe + p] = (int32_t)sel;
            keys[sel] = ~0ull;
        }
        __syncthreads();
    }
}

// Nearest centroid per row: the same distance arithmetic as coarse_dist_kernel, with a running
// (distance, number) minimum per thread over all centroid blocks and one reduction per row.
__global__ void __launch_bounds__(256)
nearest_centroid_kernel(const float *__restrict__ x, int64_t n, int dim, const float *__restrict__ cent,
                        int nlist, int32_t *__restrict__ assign)
{
    extern __shared__ __align__(16) float rows[];  // [kRows][dim], then 4*kRows uint64 for the reduction
    const int64_t r0 = (int64_t)blockIdx.x * kRows;
    for (int e = threadIdx.x; e < kRows * dim; e += 256) {
        const int64_t r = r0 + e / dim;
        rows[e] = r < n ? x[r * dim + e % dim] : 0.f;
    }
    __syncthreads();
    uint64_t best[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) best[r] = ~0ull;
    for (int c = threadIdx.x; c < nlist; c += 256) {
        const float *crow = cent + (int64_t)c * dim;
        float acc[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) acc[r] = 0.f;
        for (int d = 0; d < dim; d += 4) {
            const float4 cv = *(const float4 *)(crow + d);
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                const float4 xv = *(const float4 *)(rows + r * dim + d);
                float t = xv.x - cv.x;
                acc[r] = fmaf(t, t, acc[r]);
                t = xv.y - cv.y;
                acc[r] = fmaf(t, t, acc[r]);
                t = xv.z - cv.z;
                acc[r] = fmaf(t, t, acc[r]);
                t = xv.w - cv.w;
                acc[r] = fmaf(t, t, acc[r]);
            }
        }
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const uint64_t key = order_key(acc[r], (uint32_t)c);
            best[r] = key < best[r] ? key : best[r];
        }
    }
    __syncthreads();  // rows no longer needed: reuse LDS for the cross-wave reduction
    uint64_t *red = (uint64_t *)rows;
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const uint64_t b = wave_min_u64(best[r]);
        if ((threadIdx.x & 63) == 0) red[(threadIdx.x >> 6) * kRows + r] = b;
    }
    __syncthreads();
    if (threadIdx.x < kRows && r0 + threadIdx.x < n) {
        uint64_t b = red[threadIdx.x];
        for (int w = 1; w < 4; ++w) b = red[w * kRows + threadIdx.x] < b ? red[w * kRows + threadIdx.x] : b;
        assign[r0 + threadIdx.x] = (int32_t)(uint32_t)b;
    }
}

// ---------------------------------------------------------------------------------------------
// Nearest centroid on the matrix cores in float32 (the multi-index's halves, and of the assignment
// step of Section 4.3's index and the coarse k-means what the search on bfloat16 parts below does not
// take or leaves undecided): arg-min over c of || x - c ||^2 = arg-min of || c' ||^2 - 2 x'.c' with
// x' = x - mu, c' = c - mu (mu: any common reference point, here the mean centroid; centring keeps
// the terms small and with them the rounding error of the expansion, about 1e-7 of the distance).
// The cross term is a dense [rows x DIM] . [DIM x nlist] contraction in full float32
// (v_mfma_f32_32x32x2f32, operand layout as in the table kernel: A[i][k] with i = lane % 32,
// k = lane / 32; D[i][j] in 16 registers, register v = row 8 * (v / 4) + 4 * (lane / 32) + v % 4,
// column j = lane % 32).
// One workgroup = 4 waves x 32 rows; the rows sit in registers for the whole kernel (DIM / 2 per
// lane), the centroids stream through LDS in tiles of 32 (double-buffered, centred and their
// norms taken while staging), and every lane keeps the running minimum of its 16 outputs.  Ties
// go to the lower centroid number, as in the plain kernel; the two kernels can differ where two
// centroids are equally near within float32 rounding.
// ---------------------------------------------------------------------------------------------
typedef float f32x16 __attribute__((ext_vector_type(16)));

// DIST: instead of the arg-min, all distances || x - c ||^2 = || x' ||^2 + || c' ||^2 - 2 x'.c' are
// written (dist [n][nlist], clamped at 0), and the grid's second dimension splits the centroid
// tiles into groups of kDistTilesPerGroup so that a small batch of rows still fills the chip.
constexpr int kDistTilesPerGroup = 8;

// One turn of a workgroup: the 128 rows row_at(0), row_at(1), ... (n or more: no such row).
template <int DIM, bool DIST, typename RowAt>
__device__ __forceinline__ void
nearest_centroid_turn(const float *__restrict__ x, int64_t n, const float *__restrict__ cent,
                      const float *__restrict__ mu, int nlist, const RowAt &row_at, int32_t *__restrict__ assign,
                      float *__restrict__ dist)
{
    static_assert(DIM % 8 == 0 && DIM <= 128, "rows are held in registers");
    constexpr int KS = DIM / 2;
    constexpr int LD = DIM + 2;  // row pitch of a staged tile: lanes (half, col) hit 64 different banks
    __shared__ float tile[2][32 * LD];
    __shared__ float cnorm[2][32];
    __shared__ float xnorm[4][32];
    const int tid = (int)threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int half = lane >> 5, col = lane & 31;

    float a[KS];
    {
        const int64_t r = row_at(wave * 32 + col);
        const float *xr = x + (r < n ? r : n - 1) * DIM;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) a[kk] = xr[2 * kk + half] - mu[2 * kk + half];
    }
    if constexpr (DIST) {  // || x' ||^2 of row `col`: this lane's coordinates plus the other half's
        float xn = 0.f;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) xn = fmaf(a[kk], a[kk], xn);
        xn += __shfl_xor(xn, 32, 64);
        if (half == 0) xnorm[wave][col] = xn;
        __builtin_amdgcn_wave_barrier();
    }
    // staging: thread -> centroid tid / 8 of the tile, coordinates (tid % 8) * 4 + 32 * i
    const int sc = tid >> 3, sp = (tid & 7) * 4;
    auto stage = [&](int t, int buf) {
        const int c = t * 32 + sc;
        float nrm = 0.f;
#pragma unroll
        for (int i = 0; i < DIM / 32; ++i) {
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (c < nlist) {
                v = *(const float4 *)(cent + (int64_t)c * DIM + sp + 32 * i);
                const float4 m = *(const float4 *)(mu + sp + 32 * i);
                v.x -= m.x;
                v.y -= m.y;
                v.z -= m.z;
                v.w -= m.w;
            }
            float *d = &tile[buf][sc * LD + sp + 32 * i];
            d[0] = v.x;
            d[1] = v.y;
            d[2] = v.z;
            d[3] = v.w;
            nrm = fmaf(v.x, v.x, nrm);
            nrm = fmaf(v.y, v.y, nrm);
            nrm = fmaf(v.z, v.z, nrm);
            nrm = fmaf(v.w, v.w, nrm);
        }
        nrm += __shfl_xor(nrm, 1, 64);
        nrm += __shfl_xor(nrm, 2, 64);
        nrm += __shfl_xor(nrm, 4, 64);
        if ((tid & 7) == 0) cnorm[buf][sc] = c < nlist ? nrm : __builtin_inff();
    };
    float bestv[16];
    int besti[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        bestv[v] = __builtin_inff();
        besti[v] = 0;
    }
    const int tiles_all = (nlist + 31) / 32;
    const int tbeg = DIST ? (int)blockIdx.y * kDistTilesPerGroup : 0;
    const int ntiles = DIST ? (tiles_all < tbeg + kDistTilesPerGroup ? tiles_all : tbeg + kDistTilesPerGroup) : tiles_all;
    stage(tbeg, tbeg & 1);
    __syncthreads();
    for (int t = tbeg; t < ntiles; ++t) {
        const int buf = t & 1;
        if (t + 1 < ntiles) stage(t + 1, buf ^ 1);
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        const float *b = &tile[buf][col * LD + half];
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[kk], b[2 * kk], acc, 0, 0, 0);
        const float cn = cnorm[buf][col];
        const int ci = t * 32 + col;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float d = fmaf(-2.0f, acc[v], cn);  // (+inf for the padding of the last tile)
            if constexpr (DIST) {
                const int i = 8 * (v / 4) + 4 * half + v % 4;
                const int64_t r = row_at(wave * 32 + i);
                if (r < n && ci < nlist) {
                    const float full = d + xnorm[wave][i];
                    dist[r * nlist + ci] = full > 0.f ? full : 0.f;
                }
            } else if (d < bestv[v]) {
                bestv[v] = d;
                besti[v] = ci;
            }
        }
        __syncthreads();
    }
    if constexpr (DIST) return;
    // the 32 lanes of a half hold the 32 columns of each of its 16 rows: smallest (value, number)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        float bv = bestv[v];
        int bi = besti[v];
#pragma unroll
        for (int off = 16; off >= 1; off >>= 1) {
            const float ov = __shfl_xor(bv, off, 64);
            const int oi = __shfl_xor(bi, off, 64);
            if (ov < bv || (ov == bv && oi < bi)) {
                bv = ov;
                bi = oi;
            }
        }
        const int64_t r = row_at(wave * 32 + 8 * (v / 4) + 4 * half + v % 4);
        if (col == 0 && r < n) assign[r] = bi;
    }
}

template <int DIM, bool DIST>
__global__ void __launch_bounds__(256)
nearest_centroid_mfma_kernel(const float *__restrict__ x, int64_t n, const float *__restrict__ cent,
                             const float *__restrict__ mu, int nlist, int32_t *__restrict__ assign,
                             float *__restrict__ dist)
{
    const int64_t r0 = (int64_t)blockIdx.x * 128;
    nearest_centroid_turn<DIM, DIST>(x, n, cent, mu, nlist, [&](int i) { return r0 + i; }, assign, dist);
}

// The same for the rows that hold kUndecided in `assign` only: a workgroup gathers those of its `chunk`
// rows (at most kMarkedChunk) and takes them 128 at a time.  Without any it is a read of `assign`.
constexpr int32_t kUndecided = -1;
constexpr int kMarkedChunk = 4096;

template <int DIM>
__global__ void __launch_bounds__(256)
nearest_centroid_marked_kernel(const float *__restrict__ x, int64_t n, const float *__restrict__ cent,
                               const float *__restrict__ mu, int nlist, int chunk, int32_t *__restrict__ assign)
{
    __shared__ uint16_t marked[kMarkedChunk];
    __shared__ int nmarked;
    const int64_t first = (int64_t)blockIdx.x * chunk;
    if (threadIdx.x == 0) nmarked = 0;
    __syncthreads();
    for (int e = (int)threadIdx.x; e < chunk && first + e < n; e += 256)
        if (assign[first + e] == kUndecided) marked[atomicAdd(&nmarked, 1)] = (uint16_t)e;
    __syncthreads();
    const int count = nmarked;
    for (int turn = 0; turn < count; turn += 128)
        nearest_centroid_turn<DIM, false>(x, n, cent, mu, nlist,
                                          [&](int i) { return turn + i < count ? first + marked[turn + i] : n; },
                                          assign, (float *)nullptr);
}

// ---------------------------------------------------------------------------------------------
// Nearest centroid with the search on float16 products and the decision in float32.  The float32
// products above run at 1/16 of the rate of float16 ones.  With a = s (x - mu), b = s (c - mu) (s a power
// of two, the longest b between 2^8 and 2^9), rounded to float16 as a = A + e, b = B + f,
//     v(c) = (|a|^2 - 2 a.e) + (|b|^2 - 2 b.f) - 2 A.B
// is |a - b|^2 but for 2 (a - b).(e - f) + 2 e.f: what rounding does to a and b along themselves
// is in the two brackets, and what is left is as small as the distance.  So with d = |a - b|, E = |e| + |f|,
//     | v - d^2 | <= 2 d E + 2 |e||f| + u (|a|^2 + |b|^2) + w v,
// u = 2^-16 (the brackets come in as three bfloat16 parts each; a rounding per addition), w = 2^-(22 - b) for
// the b low bits of the mantissa that carry the tile number.  |e| is each row's own; |f| is at most the
// largest of all centroids, and at most r (|b| + 2), r the largest |f| / (|b| + 2), with |b| <= |a| + d (so one
// long centroid does not widen it for all).  With c1 the centroid of the smallest value, this gives
// D >= d1; the nearest is no farther, and its value is within twice the bound at D of the smallest.  Mostly
// one centroid is; otherwise the distances of those that are (the close calls) are taken by direct
// differences in float32 and the smallest wins, lower number on ties.
//
// A lane keeps the two smallest v of its columns.  If a lane's second is a close call too, all
// centroids of that lane are compared; if that happens in more than a few lanes, or too many lanes have a
// close call, the tiles are gone through again and every value within reach is listed.  That is the
// dearer the more there are: a workgroup whose rows have more than kManyNear lanes each with a close call
// after an eighth of the tiles gives up, and so does a row with kMostLanes at the end, one with a coordinate
// that float16 does not hold (64 times the longest centroid), or all if the centroids' squared lengths are no
// float32; nearest_centroid_marked_kernel takes those.
//
// The centroids' operands are laid out once per quantizer (centroid_operands_kernel): per tile of 32
// centroids DIM / 16 of 1 KB and one with the norms.  One workgroup = 4 waves x G groups of 32 rows; the rows'
// operands sit in registers, tiles go through LDS, two in turn; a wave's operands of the next tile are read and the
// values of one group looked at while the products of the next group are under way.  DIM / 16 + 1 products of
// 32 cycles per 32 x 32 outputs stand against 48 vector instructions (tile number into the mantissa, minimum,
// median) and (DIM / 16 + 1) KB read from LDS, which serve all G groups.  1M x 4096 at 128 dimensions: 1.19 ms
// (2.64 with three bfloat16 products a coordinate, 10.6 by the float32 products alone); the products alone take
// 0.68 at the rate registers give (1.73 PFLOP/s); with half of the vector instructions 1.00.  300k rows x 4096:
// with one of the centroids 30 times as far out 0.40 (before: 0.88), squared lengths log-normal 0.45 (0.90), every
// centroid twice 0.88 (1.75), clusters of spread 4 / 2 / 1 / 0.3 around 100 centres in 0 .. 100: 0.43 / 0.54 /
// 0.89 / 3.08 (0.91 / 1.12 / 3.54 / 3.13).
// ---------------------------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// v in three bfloat16 parts at p[0 .. 2] (2^-24 of it are left out)
__device__ __forceinline__ void three_parts(float v, __bf16 *p)
{
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        p[i] = (__bf16)v;  // nearest even
        v -= (float)p[i];  // (exact)
    }
}

// Nearest float16, 0 where that is no normal number (whatever the matrix cores make of those).
__device__ __forceinline__ _Float16 half_of(float v)
{
    return __builtin_fabsf(v) < 6.103515625e-5f ? (_Float16)0.f : (_Float16)v;
}

// Largest of n floats that are not negative, by one wave, as bits: these are ordered as the floats are, one
// that is not a number above all others.
__device__ __forceinline__ uint32_t largest_bits(const float *p, int n)
{
    uint32_t top = 0u;
    for (int i = (int)threadIdx.x & 63; i < n; i += 64) top = max(top, __float_as_uint(p[i]));
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) top = max(top, (uint32_t)__shfl_xor((int)top, off, 64));
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)top);
}

// The power of two s by the bits of the largest squared length: s sqrt(top) in [2^8, 2^9).
__device__ __forceinline__ float scale_of(uint32_t top)
{
    if (top == 0u || top >= 0x7f800000u) return 1.f;
    const int e = (int)(top >> 23) - 127;  // top < 2^(e + 1)
    return __uint_as_float((uint32_t)(127 + 9 - ((e + 2) >> 1)) << 23);
}

// Per tile, rounded up: the largest squared length (before scaling) ...
template <int DIM>
__global__ void __launch_bounds__(64)
centroid_lengths_kernel(const float *__restrict__ cent, const float *__restrict__ mu, int nlist,
                        float *__restrict__ tile_max2)
{
    const int lane = threadIdx.x, half = lane >> 5, c = blockIdx.x * 32 + (lane & 31);
    double norm = 0.0;
    if (c < nlist) {
#pragma unroll
        for (int i = 0; i < DIM / 8; ++i) {
            const float4 a = *(const float4 *)(cent + (int64_t)c * DIM + 8 * i + 4 * half);
            const float4 b = *(const float4 *)(mu + 8 * i + 4 * half);
            const float e[4] = {a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w};
#pragma unroll
            for (int p = 0; p < 4; ++p) norm += (double)e[p] * (double)e[p];
        }
    }
    norm += __shfl_xor(norm, 32, 64);
    uint32_t top = __float_as_uint((float)norm * 1.0001f);
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) top = max(top, (uint32_t)__shfl_xor((int)top, off, 64));
    if (lane == 0) tile_max2[blockIdx.x] = __uint_as_float(top);
}

// ... and, scaled, the largest |f| and |f| / (|b| + 2), with the operands.
template <int DIM>
__global__ void __launch_bounds__(64)
centroid_operands_kernel(const float *__restrict__ cent, const float *__restrict__ mu, int nlist,
                         const float *__restrict__ tile_max2, u32x4 *__restrict__ image,
                         float *__restrict__ tile_rest, float *__restrict__ tile_ratio)
{
    constexpr int KS = DIM / 16;
    const int tile = blockIdx.x, lane = threadIdx.x, half = lane >> 5, c = tile * 32 + (lane & 31);
    float4 v[2 * KS], mean[2 * KS];
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i) {
        const int d = 16 * (i >> 1) + 8 * half + 4 * (i & 1);
        v[i] = c < nlist ? *(const float4 *)(cent + (int64_t)c * DIM + d) : make_float4(0.f, 0.f, 0.f, 0.f);
        mean[i] = c < nlist ? *(const float4 *)(mu + d) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    const float scale = scale_of(largest_bits(tile_max2, (int)gridDim.x));
    u32x4 *out = image + (int64_t)tile * (KS + 1) * 64;
    double norm = 0.0, rest2 = 0.0, along = 0.0;
#pragma unroll
    for (int t = 0; t < KS; ++t) {
        f16x8 h;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const float4 a = v[2 * t + i], m = mean[2 * t + i];
            const float e[4] = {a.x - m.x, a.y - m.y, a.z - m.z, a.w - m.w};
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const float b = e[p] * scale;  // (exact, or below 2^-80)
                h[4 * i + p] = half_of(b);
                const float f = b - (float)h[4 * i + p];
                norm += (double)b * (double)b;
                rest2 += (double)f * (double)f;
                along += (double)b * (double)f;
            }
        }
        out[t * 64 + lane] = __builtin_bit_cast(u32x4, h);
    }
    norm += __shfl_xor(norm, 32, 64);
    rest2 += __shfl_xor(rest2, 32, 64);
    along += __shfl_xor(along, 32, 64);
    __bf16 n[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) n[i] = (__bf16)0.f;
    if (half == 0) {  // (places past the last centroid: farther than anything finite)
        three_parts(c < nlist ? (float)(norm - 2.0 * along) : 1e30f, n);
#pragma unroll
        for (int i = 3; i < 6; ++i) n[i] = (__bf16)1.f;
    }
    bf16x8 ops;
#pragma unroll
    for (int i = 0; i < 8; ++i) ops[i] = n[i];
    out[KS * 64 + lane] = __builtin_bit_cast(u32x4, ops);
    const float rest = __builtin_amdgcn_sqrtf((float)rest2) * 1.0001f;
    uint32_t most = __float_as_uint(rest);
    uint32_t ratio = __float_as_uint(rest * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf((float)norm) * 0.9999f + 2.f) * 1.0001f);
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) {
        most = max(most, (uint32_t)__shfl_xor((int)most, off, 64));
        ratio = max(ratio, (uint32_t)__shfl_xor((int)ratio, off, 64));
    }
    if (lane == 0) {
        tile_rest[tile] = __uint_as_float(most);
        tile_ratio[tile] = __uint_as_float(ratio);
    }
}

constexpr int kHalfWaves = 4;
// Rows from which a wave takes two groups: below, twice the workgroups weigh more (one group / two, us, 4096
// lists of 128 dimensions: 20k rows 90 / 107, 50k 122 / 123, 100k 192 / 182, 1M 1341 / 1188; 1024 of 64, 20k 25 / 33,
// 100k 49 / 47, 500k 164 / 155).
constexpr int64_t kTwoGroupRows = 100'000;
constexpr int kPairList = 512;    // pairs a wave lists before it takes their distances
constexpr int kManyNear = 3;      // (some 25 close calls a row in all: listing them takes about as long as the
                                  //  float32 products)
constexpr int kMostLanes = 28;    // of 32
constexpr int kDeepLanes = 16;    // of a workgroup's rows: comparing all centroids of so many lanes takes as long
                                  // as going through the tiles again
template <int DIM, int G>
__global__ void __launch_bounds__(kHalfWaves * 64) __attribute__((amdgpu_waves_per_eu(G == 1 ? 3 : 2)))
nearest_centroid_half_kernel(const float *__restrict__ x, int64_t n, const float *__restrict__ cent,
                             const float *__restrict__ mu, const u32x4 *__restrict__ image,
                             const float *__restrict__ tile_max2, int nlist, int tile_bits,
                             int32_t *__restrict__ assign)
{
    constexpr int KS = DIM / 16;
    constexpr int kThreads = kHalfWaves * 64;
    constexpr int kRows = 32 * G;            // of a wave
    constexpr int kOps = (KS + 1) * 64;      // 16-byte entries of a tile
    constexpr int kTurns = (kOps + kThreads - 1) / kThreads;
    __shared__ __align__(16) u32x4 tile[2][kTurns * kThreads];
    __shared__ float row_norm[kHalfWaves][kRows], row_rest[kHalfWaves][kRows];  // |a|^2, |e|
    __shared__ float limit[kHalfWaves][kRows];  // what counts as a close call
    __shared__ unsigned long long nearest[kHalfWaves][kRows];  // (distance, number) of the best listed pair
    __shared__ uint16_t near_tile[kHalfWaves][kRows][32];      // of the lanes whose smallest value is a close call
    __shared__ uint32_t pairs[kHalfWaves][kPairList];          // row << 16 | centroid
    __shared__ int tally[2];
    const int tid = (int)threadIdx.x, wave = tid >> 6, lane = tid & 63, half = lane >> 5, col = lane & 31;
    const int64_t r0 = ((int64_t)blockIdx.x * kHalfWaves + wave) * kRows;
    const int ntiles = (nlist + 31) / 32;
    const uint32_t top = largest_bits(tile_max2, ntiles);
    const float scale = scale_of(top);
    // (rest_max is not a number where the centroids' lengths are none: nothing is then within reach)
    const float cmax2 = __uint_as_float(top) * scale * scale;
    const float rest_max = top < 0x7f800000u ? __uint_as_float(largest_bits(tile_max2 + ntiles, ntiles)) : __builtin_nanf("");
    const float ratio = __uint_as_float(largest_bits(tile_max2 + 2 * ntiles, ntiles));
    constexpr float kSum = 1.52587890625e-5f;
    const float kTag = __uint_as_float((uint32_t)(127 - 22 + tile_bits) << 23);

    f16x8 xh[G][KS];
    bf16x8 one[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int64_t r = r0 + 32 * g + col;
        const float *xr = x + (r < n ? r : n - 1) * DIM + 8 * half;
        float norm = 0.f, rest2 = 0.f, along = 0.f;
#pragma unroll
        for (int t = 0; t < KS; ++t) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float v = (xr[16 * t + i] - mu[16 * t + 8 * half + i]) * scale;
                xh[g][t][i] = half_of(-2.f * v);
                const float rest = fmaf(-2.f, v, -(float)xh[g][t][i]);  // (-2 e)
                norm = fmaf(v, v, norm);
                rest2 = fmaf(rest, rest, rest2);
                along = fmaf(v, rest, along);
            }
        }
        norm += __shfl_xor(norm, 32, 64);
        rest2 += __shfl_xor(rest2, 32, 64);
        along += __shfl_xor(along, 32, 64);
        __bf16 p[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) p[i] = (__bf16)(half == 0 && i < 3 ? 1.f : 0.f);
        if (half == 0) {
            three_parts(norm + along, p + 3);
            row_norm[wave][32 * g + col] = norm;
            row_rest[wave][32 * g + col] = __builtin_amdgcn_sqrtf(rest2) * 0.5005f;
            nearest[wave][32 * g + col] = ~0ull;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) one[g][i] = p[i];
    }
    if (tid < 2) tally[tid] = 0;
    u32x4 hold[kTurns];
    auto fetch = [&](int t) {
#pragma unroll
        for (int i = 0; i < kTurns; ++i)
            hold[i] = image[(int64_t)t * kOps + min(i * kThreads + tid, kOps - 1)];
    };
    auto put = [&](int buf) {
#pragma unroll
        for (int i = 0; i < kTurns; ++i)
            tile[buf][i * kThreads + tid] = hold[i];
    };
    float best[G][16], next[G][16];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int v = 0; v < 16; ++v) best[g][v] = next[g][v] = __builtin_inff();
    // Tiles [from, to): see(t, group, values).  The operands of the first are held and the tile after it waits in
    // LDS, as do those of `to` and the tile after that at the end.  The values of one group are looked at while
    // the products of the next are under way.
    u32x4 op[KS + 1];
    auto sweep = [&](int from, int to, auto &&see) {
        f32x16 last;
#pragma unroll
        for (int v = 0; v < 16; ++v) last[v] = 1e30f;  // (beyond every reach)
        for (int t = from; t < to; ++t) {
            fetch(min(t + 2, ntiles - 1));
            const u32x4 *b = tile[(t + 1) & 1];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                f32x16 acc;
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[v] = 0.f;
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(one[g], __builtin_bit_cast(bf16x8, op[KS]), acc, 0, 0, 0);
#pragma unroll
                for (int s = 0; s < KS; ++s)
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(xh[g][s], __builtin_bit_cast(f16x8, op[s]), acc, 0, 0, 0);
                if (g == G - 1) {
                    op[KS] = b[KS * 64 + lane];
#pragma unroll
                    for (int s = 0; s < KS; ++s) op[s] = b[s * 64 + lane];
                }
                see(g > 0 ? t : max(t - 1, 0), g > 0 ? g - 1 : G - 1, last);
                asm volatile("" : "+v"(acc));
                last = acc;
#pragma unroll
                for (int s = 0; s < KS + 1; ++s) {
                    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                    if (g == G - 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x2, (48 + KS) / (KS + 1), 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            put(t & 1);
            __syncthreads();
        }
        see(to > 0 ? to - 1 : 0, G - 1, last);
    };
    uint32_t keep = ~((1u << tile_bits) - 1u);
    float low = -__builtin_inff();
    asm("" : "+v"(keep), "+v"(low));
    auto two_smallest = [&](int t, int g, const f32x16 &acc) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float d = __uint_as_float((__float_as_uint(acc[v]) & keep) | (uint32_t)t);
            next[g][v] = __builtin_amdgcn_fmed3f(d, best[g][v], next[g][v]);
            best[g][v] = __builtin_amdgcn_fmed3f(d, best[g][v], low);  // (the smaller of the two)
            asm volatile("" : "+v"(best[g][v]), "+v"(next[g][v]));     // (here, not after the products)
        }
    };
    // limit[]: the largest value of a close call for each row, by the smallest of its values.  Halving the
    // registers with every step across the lanes leaves lane (half, c) with the row of register c of its half.
    auto set_limits = [&]() {
        float least[16 * G];
#pragma unroll
        for (int i = 0; i < 16 * G; ++i) least[i] = best[i >> 4][i & 15];
#pragma unroll
        for (int r = 8 * G; r >= 1; r >>= 1)
#pragma unroll
            for (int i = 0; i < r; ++i) {
                const bool up = (lane & r) != 0;
                const float mine = up ? least[i + r] : least[i], other = up ? least[i] : least[i + r];
                least[i] = fminf(mine, __shfl_xor(other, r, 64));
            }
        if (G == 1) least[0] = fminf(least[0], __shfl_xor(least[0], 16, 64));
        const int reg = lane & (16 * G - 1), row = 32 * (reg >> 4) + 8 * (reg >> 2 & 3) + 4 * half + (reg & 3);
        const float x2 = row_norm[wave][row], e = row_rest[wave][row], len = __builtin_amdgcn_sqrtf(x2);
        const float seen = fmaxf(least[0], 0.f) + kTag * __builtin_fabsf(least[0]);
        auto farthest = [&](float f, float b2) {  // D from d^2 <= seen + 2 d (e + f) + 2 e f + u (x2 + b2)
            return (e + f + __builtin_amdgcn_sqrtf((e + f) * (e + f) + seen + 2.f * e * f + kSum * (x2 + b2))) * 1.001f;
        };
        const float reach_len = len + farthest(rest_max, cmax2);
        const float f = fminf(rest_max, ratio * (reach_len + 2.f)), b2 = fminf(cmax2, reach_len * reach_len);
        const float d = farthest(f, b2);
        const float reach = least[0] + 2.002f * (2.f * d * (e + f) + 2.f * e * f + kSum * (x2 + b2) + 2.f * kTag * d * d);
        // (rows that float16 does not hold have an |e| that is no finite number)
        limit[wave][row] = x2 < 1e20f && e < 1e20f && rest_max < 1e20f ? reach : __builtin_nanf("");
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    auto row_of = [&](int g, int v) { return 32 * g + 8 * (v / 4) + 4 * half + v % 4; };

    auto begin = [&]() {
        fetch(0);
        put(0);
        fetch(min(1, ntiles - 1));
        put(1);
        __syncthreads();
#pragma unroll
        for (int s = 0; s < KS + 1; ++s) op[s] = tile[0][s * 64 + lane];
        __syncthreads();  // (the first turn of a sweep writes there)
    };
    begin();
    const int early = ntiles >= 16 ? ntiles / 8 : 0;
    sweep(0, early, two_smallest);
    if (early > 0) {
        int lanes = 0;
        set_limits();
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                lanes += __builtin_popcountll(__ballot(best[g][v] <= limit[wave][row_of(g, v)]));
        if (lane == 0) atomicAdd(&tally[0], lanes);
        __syncthreads();
        if (tally[0] > kManyNear * kRows * kHalfWaves) {
            if (lane < kRows && r0 + lane < n) assign[r0 + lane] = kUndecided;
            return;
        }
    }
    sweep(early, ntiles, two_smallest);

    // The distances of the listed pairs, four at a time, 16 lanes to a pair.
    int npairs = 0;
    auto settle = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int l16 = lane & 15;
#pragma unroll 4
        for (int i = lane >> 4; i - (lane >> 4) < npairs; i += 4) {
            const uint32_t e = pairs[wave][i < npairs ? i : npairs - 1];  // (the last one again: the same key)
            const int row = (int)(e >> 16), c = (int)(e & 0xffffu);
            typedef float row4 __attribute__((ext_vector_type(4), aligned(4)));  // (rows of the caller's start anywhere)
            const row4 *xr = (const row4 *)(x + (r0 + row) * DIM);
            const float4 *cr = (const float4 *)(cent + (int64_t)c * DIM);
            float d = 0.f;
#pragma unroll
            for (int p = 0; p < (DIM / 4 + 15) / 16; ++p) {
                if (16 * p + l16 >= DIM / 4) continue;
                const row4 xv = xr[16 * p + l16];
                const float4 cv = cr[16 * p + l16];
                const float dx = xv.x - cv.x, dy = xv.y - cv.y, dz = xv.z - cv.z, dw = xv.w - cv.w;
                d = fmaf(dx, dx, d);
                d = fmaf(dy, dy, d);
                d = fmaf(dz, dz, d);
                d = fmaf(dw, dw, d);
            }
#pragma unroll
            for (int off = 8; off >= 1; off >>= 1) d += __shfl_xor(d, off, 64);
            if (l16 == 0) atomicMin(&nearest[wave][row], (unsigned long long)order_key(d, (uint32_t)c));
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        npairs = 0;
    };
    auto list_pairs = [&](bool take, int row, int c) {
        take = take && c < nlist;  // (the places past the last centroid are no centroids)
        const uint64_t m = __ballot(take);
        if (npairs + __builtin_popcountll(m) > kPairList) settle();
        const int at = npairs + __builtin_popcountll(m & ((1ull << lane) - 1ull));
        if (take) pairs[wave][at] = (uint32_t)row << 16 | (uint32_t)c;
        npairs += __builtin_popcountll(m);
    };

    // Lane r < kRows gathers of row r which lanes' smallest, and second smallest, value is a close call.
    uint32_t near = 0u, deep = 0u;
    set_limits();
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = row_of(g, v), upper = 32 * g + 8 * (v / 4) + v % 4;
            const float reach = limit[wave][row];
            const uint64_t near2 = __ballot(best[g][v] <= reach), deep2 = __ballot(next[g][v] <= reach);
            if (best[g][v] <= reach) near_tile[wave][row][col] = (uint16_t)(__float_as_uint(best[g][v]) & ~keep);
            near = lane == upper ? (uint32_t)near2 : lane == upper + 4 ? (uint32_t)(near2 >> 32) : near;
            deep = lane == upper ? (uint32_t)deep2 : lane == upper + 4 ? (uint32_t)(deep2 >> 32) : deep;
        }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    int decided = kUndecided;  // lane r: what is known of row r
    const bool is_row = lane < kRows && r0 + lane < n;
    const int count = __builtin_popcount(near);
    const bool again = is_row && deep != 0u && count < kMostLanes;
    if (is_row && deep == 0u && count == 1) {
        const int at = __builtin_ctz(near), winner = (int)near_tile[wave][lane][at] * 32 + at;
        if (winner < nlist) decided = winner;
    }
    if (again) atomicAdd(&tally[1], __builtin_popcount(deep));
    if (lane < kRows && !again) limit[wave][lane] = __builtin_nanf("");  // (no value is within it)
    for (uint64_t rows = __ballot(is_row && deep == 0u && count > 1); rows != 0; rows &= rows - 1u) {
        const int row = __builtin_ctzll(rows);
        const uint32_t lanes = (uint32_t)__builtin_amdgcn_readlane((int)near, row);
        list_pairs(half == 0 && (lanes >> col & 1u) != 0u, row, (int)near_tile[wave][row][col] * 32 + col);
    }
    __syncthreads();
    if (tally[1] > kDeepLanes) {
        asm("" : "+s"(image));  // (addresses kept from above would go to scratch memory)
        float lim[G][16];
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int v = 0; v < 16; ++v) lim[g][v] = limit[wave][row_of(g, v)];
        begin();
        sweep(0, ntiles, [&](int t, int g, const f32x16 &acc) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const bool close = __uint_as_float((__float_as_uint(acc[v]) & keep) | (uint32_t)t) <= lim[g][v];
                if (__ballot(close) != 0) list_pairs(close, row_of(g, v), t * 32 + col);
            }
        });
    } else {
        for (uint64_t rows = __ballot(again); rows != 0; rows &= rows - 1u) {
            const int row = __builtin_ctzll(rows);
            const uint32_t lanes = (uint32_t)__builtin_amdgcn_readlane((int)near, row);
            uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)deep, row);
            list_pairs(half == 0 && ((lanes & ~all) >> col & 1u) != 0u, row, (int)near_tile[wave][row][col] * 32 + col);
            for (; all != 0u; all &= all - 1u)
                for (int t = 0; t < ntiles; t += 64)
                    list_pairs(t + lane < ntiles, row, (t + lane) * 32 + __builtin_ctz(all));
        }
    }
    settle();
    if (is_row)
        assign[r0 + lane] = nearest[wave][lane] != ~0ull ? (int32_t)(uint32_t)nearest[wave][lane] : decided;
}

// ---------------------------------------------------------------------------------------------
// Job bookkeeping.  Jobs in query-major order are cut into blocks of kJobBlockQ queries; a
// stable counting sort by list number (block histograms -> column prefix -> in-order scatter)
// gives every list its jobs in ascending query order, reproducibly.
// ---------------------------------------------------------------------------------------------
constexpr int kJobBlockQ = 16;

__global__ void zero_i32_kernel(int32_t *p, int64_t n)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) p[e] = 0;
}

// Sort key of job (q, p): its list, with the jobs of a query's `pilot` nearest lists ahead of all
// others (keys [0, nlist) before keys [nlist, 2 nlist)).  Workgroups start in tile order, so the
// nearest lists of every query are scanned first and their k-th best distances are published
// before the bulk of the lists is looked at, which then rejects most survivors at the threshold
// test instead of inserting them into lists.
__device__ __forceinline__ int job_key(int list, int p, int nlist, int pilot) { return list + (p >= pilot ? nlist : 0); }

__global__ void job_hist_kernel(const int32_t *__restrict__ probed, int64_t nq, int nprobe, int nlist, int pilot,
                                int32_t *__restrict__ hist)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= nq * nprobe) return;
    const int64_t q = j / nprobe;
    const int p = (int)(j - q * nprobe);
    atomicAdd(&hist[(q / kJobBlockQ) * (2 * nlist) + job_key(probed[j], p, nlist, pilot)], 1);
}

// hist[b][l] -> number of jobs of list l in blocks before b; totals[l] = jobs of list l.
__global__ void job_column_prefix_kernel(int32_t *__restrict__ hist, int64_t nblk, int nlist,
                                         int32_t *__restrict__ totals)
{
    const int l = blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= nlist) return;
    int32_t run = 0;
    int64_t b = 0;
    for (; b + 16 <= nblk; b += 16) {  // sixteen loads in flight instead of one (the walk is latency-bound)
        int32_t c[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) c[i] = hist[(b + i) * nlist + l];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            hist[(b + i) * nlist + l] = run;
            run += c[i];
        }
    }
    for (; b < nblk; ++b) {
        const int32_t c = hist[b * nlist + l];
        hist[b * nlist + l] = run;
        run += c;
    }
    totals[l] = run;
}

// One workgroup: list_begin = exclusive prefix of totals; tile_begin = exclusive prefix of
// ceil(totals / tq).  `totals` aliases list_begin (read before written, element-wise by owner).
__global__ void __launch_bounds__(1024)
job_list_prefix_kernel(int32_t *__restrict__ list_begin, int32_t *__restrict__ tile_begin, int nlist, int tq)
{
    __shared__ int32_t pj[1024], pt[1024];
    const int t = threadIdx.x;
    const int per = (nlist + 1023) / 1024;
    const int lo = t * per, hi = min(nlist, lo + per);
    int32_t sj = 0, st = 0;
    for (int l = lo; l < hi; ++l) {
        sj += list_begin[l];
        st += (list_begin[l] + tq - 1) / tq;
    }
    pj[t] = sj;
    pt[t] = st;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int32_t aj = t >= off ? pj[t - off] : 0, at = t >= off ? pt[t - off] : 0;
        __syncthreads();
        pj[t] += aj;
        pt[t] += at;
        __syncthreads();
    }
    int32_t bj = pj[t] - sj, bt = pt[t] - st;  // exclusive
    for (int l = lo; l < hi; ++l) {
        const int32_t c = list_begin[l];
        list_begin[l] = bj;
        tile_begin[l] = bt;
        bj += c;
        bt += (c + tq - 1) / tq;
    }
    if (t == 1023) {
        list_begin[nlist] = pj[1023];
        tile_begin[nlist] = pt[1023];
    }
}

// One workgroup per block of kJobBlockQ queries, queries taken in order: job (q, p) goes to
// list_begin[l] + (jobs of l in earlier blocks) + (jobs of l earlier in this block).
__global__ void __launch_bounds__(256)
job_scatter_kernel(const int32_t *__restrict__ probed, int64_t nq, int nprobe, int nlist, int pilot,
                   int32_t *__restrict__ hist, const int32_t *__restrict__ list_begin,
                   int32_t *__restrict__ job_q, int32_t *__restrict__ job_list, int32_t *__restrict__ job_slot)
{
    const int64_t b = blockIdx.x;
    int32_t *run = hist + b * (2 * nlist);
    for (int qi = 0; qi < kJobBlockQ; ++qi) {
        const int64_t q = b * kJobBlockQ + qi;
        if (q >= nq) break;
        for (int p = threadIdx.x; p < nprobe; p += 256) {  // the lists of one query are distinct
            const int l = probed[q * nprobe + p];
            const int key = job_key(l, p, nlist, pilot);
            // the only writer of run[key] in this turn; the atomic keeps it coherent across turns
            const int32_t at = list_begin[key] + atomicAdd(&run[key], 1);
            job_q[at] = (int32_t)q;
            job_list[at] = l;
            job_slot[at] = (int32_t)(q * nprobe + p);
        }
        __syncthreads();
    }
}

struct TileRec {
    int32_t job_begin, njobs, list, pad;
};

__global__ void job_tiles_kernel(const int32_t *__restrict__ list_begin, const int32_t *__restrict__ tile_begin,
                                 int nlist, int tq, TileRec *__restrict__ tiles)
{
    const int key = blockIdx.x * blockDim.x + threadIdx.x;
    if (key >= 2 * nlist) return;
    const int l = key < nlist ? key : key - nlist;
    const int32_t jb = list_begin[key], cnt = list_begin[key + 1] - jb;
    int32_t t = tile_begin[key];
    for (int32_t o = 0; o < cnt; o += tq, ++t) tiles[t] = TileRec{jb + o, min(tq, cnt - o), l, 0};
}

// Few jobs: no grouping by list.  Every job becomes a tile of its own, the jobs of every query's
// nearest list first, then all second nearest, ...: tile t = (query t % nq, probe t / nq).
__global__ void direct_jobs_kernel(const int32_t *__restrict__ probed, int nq, int nprobe,
                                   int32_t *__restrict__ job_q, int32_t *__restrict__ job_list,
                                   int32_t *__restrict__ job_slot, TileRec *__restrict__ tiles,
                                   int32_t *__restrict__ ntiles)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int njobs = nq * nprobe;
    if (t == 0) *ntiles = njobs;
    if (t >= njobs) return;
    const int p = t / nq, q = t - p * nq;
    const int l = probed[q * nprobe + p];
    job_q[t] = q;
    job_list[t] = l;
    job_slot[t] = q * nprobe + p;
    tiles[t] = TileRec{t, 1, l, 0};
}

// The lists' share of the residual tables: see launch_list_tables.  One workgroup per (list,
// sub-quantizer), thread c owns centroid c.
__global__ void __launch_bounds__(256)
list_tables_kernel(const float *__restrict__ cb, int dim, int m, const float *__restrict__ coarse, int nlist,
                   float *__restrict__ out)
{
    extern __shared__ float gt[];  // (g_l - o)_j
    const int l = blockIdx.x, j = blockIdx.y, c = threadIdx.x;
    const int dsub = dim / m;
    for (int t = threadIdx.x; t < dsub; t += 256)
        gt[t] = coarse[(int64_t)l * dim + j * dsub + t] - coarse[(int64_t)nlist * dim + j * dsub + t];
    __syncthreads();
    const float *crow = cb + ((int64_t)j * 256 + c) * dsub;
    float acc = 0.f;
    for (int t = 0; t < dsub; ++t) acc = fmaf(gt[t], crow[t], acc);
    out[((int64_t)l * m + j) * 256 + c] = 2.0f * acc;
}

// Copy per-job rows (job-sorted) back to (query, probe) order.
__global__ void unsort_rows_kernel(const uint8_t *__restrict__ src, const int32_t *__restrict__ job_slot,
                                   int64_t njobs, int row_bytes, uint8_t *__restrict__ dst)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= njobs * row_bytes) return;
    const int64_t j = e / row_bytes;
    dst[(int64_t)job_slot[j] * row_bytes + e % row_bytes] = src[e];
}

}  // namespace

int launch_list_tables(const float *cb_dev, int dim, int m, const float *coarse_dev, int nlist,
                       float *list_tab_dev, hipStream_t s)
{
    PSC_REQUIRE(dim % m == 0 && nlist >= 1, "bad shape");
    hipLaunchKernelGGL(list_tables_kernel, dim3((unsigned)nlist, (unsigned)m), dim3(256),
                       (size_t)(dim / m) * sizeof(float), s, cb_dev, dim, m, coarse_dev, nlist, list_tab_dev);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

int launch_unsort_rows(const uint8_t *src_dev, const int32_t *job_slot_dev, int64_t njobs, int row_bytes,
                       uint8_t *dst_dev, hipStream_t s)
{
    const int64_t total = njobs * row_bytes;
    if (total == 0) return PSC_OK;
    hipLaunchKernelGGL(unsort_rows_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, src_dev,
                       job_slot_dev, njobs, row_bytes, dst_dev);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

static int check_dim(int dim, int nlist)
{
    PSC_REQUIRE(dim > 0 && dim % 4 == 0 && dim <= 1024, "coarse quantizer needs dim %% 4 == 0 and dim <= 1024, got %d", dim);
    PSC_REQUIRE(nlist >= 1 && nlist <= 16384, "nlist must be in [1, 16384], got %d", nlist);
    return PSC_OK;
}

template <int DIM>
static int run_coarse_dist_mfma(const float *x_dev, int64_t n, const float *cent_dev, const float *mu_dev, int nlist,
                                float *dist_dev, hipStream_t s)
{
    const int tiles = (nlist + 31) / 32;
    dim3 grid((unsigned)((n + 127) / 128), (unsigned)((tiles + kDistTilesPerGroup - 1) / kDistTilesPerGroup));
    hipLaunchKernelGGL((nearest_centroid_mfma_kernel<DIM, true>), grid, dim3(256), 0, s, x_dev, n, cent_dev, mu_dev,
                       nlist, (int32_t *)nullptr, dist_dev);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

// mu_dev: reference point [dim] of the matrix-core kernel (the mean centroid), which takes batches
// of 256 rows and more in the dimensions it is built for; everything else takes the plain kernel.
int launch_coarse_distances(const float *x_dev, int64_t n, int dim, const float *cent_dev, int nlist,
                            const float *mu_dev, float *dist_dev, hipStream_t s)
{
    int rc = check_dim(dim, nlist);
    if (rc != PSC_OK) return rc;
    if (n == 0) return PSC_OK;
    if (mu_dev && n >= 256 && (n + 127) / 128 <= 0x7fffffffLL) {
        switch (dim) {
        case 32: return run_coarse_dist_mfma<32>(x_dev, n, cent_dev, mu_dev, nlist, dist_dev, s);
        case 64: return run_coarse_dist_mfma<64>(x_dev, n, cent_dev, mu_dev, nlist, dist_dev, s);
        case 96: return run_coarse_dist_mfma<96>(x_dev, n, cent_dev, mu_dev, nlist, dist_dev, s);
        case 128: return run_coarse_dist_mfma<128>(x_dev, n, cent_dev, mu_dev, nlist, dist_dev, s);
        default: break;
        }
    }
    if (n <= kFewRowsMax) {
        dim3 grid((unsigned)((nlist + 31) / 32), (unsigned)((n + kFewRows - 1) / kFewRows));
        hipLaunchKernelGGL(coarse_dist_few_kernel, grid, dim3(256), (size_t)kFewRows * dim * sizeof(float), s, x_dev, n,
                           dim, cent_dev, nlist, dist_dev);
        PSC_HIP_TRY(hipGetLastError());
        return PSC_OK;
    }
    PSC_REQUIRE((n + kRows - 1) / kRows <= 0x7fffffffLL, "too many rows");
    dim3 grid((unsigned)((n + kRows - 1) / kRows), (unsigned)((nlist + 255) / 256));
    hipLaunchKernelGGL(coarse_dist_kernel, grid, dim3(256), (size_t)kRows * dim * sizeof(float), s, x_dev, n, dim,
                       cent_dev, nlist, dist_dev);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

int launch_select_probes(const float *dist_dev, int64_t n, int nlist, int nprobe, const int32_t *settled_dev,
                         int32_t *probed_dev, hipStream_t s)
{
    PSC_REQUIRE(nprobe >= 1 && nprobe <= nlist && nlist <= 16384, "bad nprobe/nlist");
    if (n == 0) return PSC_OK;
    PSC_REQUIRE(n <= 0x7fffffffLL, "too many rows");
    static bool configured = false;
    if (!configured) {
        PSC_HIP_TRY(hipFuncSetAttribute((const void *)select_probes_kernel,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, 16384 * 8));
        configured = true;
    }
    if (n <= kFewRowsMax) {  // a workgroup per row: the latency of a single query
        if (nlist <= 4096)
            hipLaunchKernelGGL(select_probes_block_kernel<4>, dim3((unsigned)n), dim3(1024), 0, s, dist_dev, nlist,
                               nprobe, settled_dev, probed_dev);
        else
            hipLaunchKernelGGL(select_probes_block_kernel<16>, dim3((unsigned)n), dim3(1024), 0, s, dist_dev, nlist,
                               nprobe, settled_dev, probed_dev);
        PSC_HIP_TRY(hipGetLastError());
        return PSC_OK;
    }
    const dim3 wgrid((unsigned)((n + 3) / 4));
    const size_t wlds = (size_t)4 * nprobe * sizeof(uint64_t);
    if (nlist <= 1024)
        hipLaunchKernelGGL(select_probes_wave_kernel<16>, wgrid, dim3(256), wlds, s, dist_dev, n, nlist, nprobe,
                           settled_dev, probed_dev);
    else if (nlist <= 4096)
        hipLaunchKernelGGL(select_probes_wave_kernel<64>, wgrid, dim3(256), wlds, s, dist_dev, n, nlist, nprobe,
                           settled_dev, probed_dev);
    else
        hipLaunchKernelGGL(select_probes_kernel, dim3((unsigned)n), dim3(256), (size_t)nlist * sizeof(uint64_t), s,
                           dist_dev, nlist, nprobe, settled_dev, probed_dev);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

template <int DIM>
static int run_nearest_centroid_mfma(const float *x_dev, int64_t n, const float *cent_dev, const float *mu_dev,
                                     int nlist, int32_t *assign_dev, hipStream_t s)
{
    hipLaunchKernelGGL((nearest_centroid_mfma_kernel<DIM, false>), dim3((unsigned)((n + 127) / 128)), dim3(256), 0, s,
                       x_dev, n, cent_dev, mu_dev, nlist, assign_dev, (float *)nullptr);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

static size_t centroid_operand_bytes(int nlist, int dim) { return (size_t)((nlist + 31) / 32) * (size_t)(dim / 16 + 1) * 64 * 16; }

size_t centroid_image_bytes(int nlist, int dim)
{
    if (dim != 32 && dim != 64 && dim != 96 && dim != 128) return 0;
    return centroid_operand_bytes(nlist, dim) + (size_t)((nlist + 31) / 32) * 3 * sizeof(float);  // (of the tiles)
}

int launch_centroid_image(const float *cent_dev, const float *mu_dev, int nlist, int dim, void *image_dev, hipStream_t s)
{
    float *tile_max2 = (float *)((char *)image_dev + centroid_operand_bytes(nlist, dim));
    const int ntiles = (nlist + 31) / 32;
    const dim3 grid((unsigned)ntiles), block(64);
#define CALL(D)                                                                                                  \
    do {                                                                                                         \
        hipLaunchKernelGGL((centroid_lengths_kernel<D>), grid, block, 0, s, cent_dev, mu_dev, nlist, tile_max2); \
        hipLaunchKernelGGL((centroid_operands_kernel<D>), grid, block, 0, s, cent_dev, mu_dev, nlist, tile_max2, \
                           (u32x4 *)image_dev, tile_max2 + ntiles, tile_max2 + 2 * ntiles);                      \
    } while (0)
    switch (dim) {
    case 32: CALL(32); break;
    case 64: CALL(64); break;
    case 96: CALL(96); break;
    case 128: CALL(128); break;
    default: set_error("no float16 assignment for dimension %d", dim); return PSC_EINVAL;
    }
#undef CALL
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

// The float32 products are done sooner only where there is next to nothing for either to do (float32 / float16, us:
// 32 lists of 32 dimensions, 1k rows 12 / 13, 20k 13 / 14, 50k 16 / 14, 1M 106 / 83; 128 of 32, 1k rows 16 / 13; 16
// of 128, 1k rows 20 / 15, 1M 417 / 174; 128 of 128, 28 / 14 and 641 / 194).
bool half_assignment_pays(int64_t n, int dim, int nlist) { return (int64_t)nlist * dim > 1024 || n >= 50'000; }

template <int DIM, int G>
static void launch_half(const float *x_dev, int64_t n, const float *cent_dev, int nlist, const float *mu_dev,
                        const u32x4 *image, const float *tile_max2, int bits, int32_t *assign_dev, hipStream_t s)
{
    constexpr int kRowsPer = 32 * G * kHalfWaves;
    hipLaunchKernelGGL((nearest_centroid_half_kernel<DIM, G>), dim3((unsigned)((n + kRowsPer - 1) / kRowsPer)),
                       dim3(kHalfWaves * 64), 0, s, x_dev, n, cent_dev, mu_dev, image, tile_max2, nlist, bits, assign_dev);
}

int launch_nearest_centroid_half(const float *x_dev, int64_t n, int dim, const float *cent_dev, int nlist,
                                 const float *mu_dev, const void *image_dev, int32_t *assign_dev, hipStream_t s)
{
    int rc = check_dim(dim, nlist);
    if (rc != PSC_OK) return rc;
    if (n == 0) return PSC_OK;
    constexpr int kRowsPer = 32 * kHalfWaves;
    PSC_REQUIRE((n + kRowsPer - 1) / kRowsPer <= 0x7fffffffLL, "too many rows");
    const float *tile_max2 = (const float *)((const char *)image_dev + centroid_operand_bytes(nlist, dim));
    int bits = 0;  // of a tile's number
    while ((1 << bits) < (nlist + 31) / 32) ++bits;
    // (512 workgroups of whole turns for the rows left over, once there are as many)
    const int64_t share = (n / 512 + kRowsPer - 1) / kRowsPer * kRowsPer;
    const int chunk = (int)(share < kRowsPer ? kRowsPer : share < kMarkedChunk ? share : kMarkedChunk);
    const dim3 mgrid((unsigned)((n + chunk - 1) / chunk));
    const bool two = n >= kTwoGroupRows;
#define CALL(D)                                                                                                      \
    do {                                                                                                             \
        const u32x4 *image = (const u32x4 *)image_dev;                                                               \
        if (two)                                                                                                     \
            launch_half<D, 2>(x_dev, n, cent_dev, nlist, mu_dev, image, tile_max2, bits, assign_dev, s);             \
        else                                                                                                         \
            launch_half<D, 1>(x_dev, n, cent_dev, nlist, mu_dev, image, tile_max2, bits, assign_dev, s);             \
        hipLaunchKernelGGL((nearest_centroid_marked_kernel<D>), mgrid, dim3(256), 0, s, x_dev, n, cent_dev, mu_dev,  \
                           nlist, chunk, assign_dev);                                                                \
    } while (0)
    switch (dim) {
    case 32: CALL(32); break;
    case 64: CALL(64); break;
    case 96: CALL(96); break;
    case 128: CALL(128); break;
    default: set_error("no float16 assignment for dimension %d", dim); return PSC_EINVAL;
    }
#undef CALL
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

// mu_dev: a reference point [dim] for the matrix-core kernel (the mean centroid); null, or a
// dimension that kernel is not built for, takes the plain kernel.
int launch_nearest_centroid(const float *x_dev, int64_t n, int dim, const float *cent_dev, int nlist,
                            const float *mu_dev, int32_t *assign_dev, hipStream_t s)
{
    int rc = check_dim(dim, nlist);
    if (rc != PSC_OK) return rc;
    if (n == 0) return PSC_OK;
    if (mu_dev && (n + 127) / 128 <= 0x7fffffffLL) {
        switch (dim) {
        case 32: return run_nearest_centroid_mfma<32>(x_dev, n, cent_dev, mu_dev, nlist, assign_dev, s);
        case 64: return run_nearest_centroid_mfma<64>(x_dev, n, cent_dev, mu_dev, nlist, assign_dev, s);
        case 96: return run_nearest_centroid_mfma<96>(x_dev, n, cent_dev, mu_dev, nlist, assign_dev, s);
        case 128: return run_nearest_centroid_mfma<128>(x_dev, n, cent_dev, mu_dev, nlist, assign_dev, s);
        default: break;
        }
    }
    PSC_REQUIRE((n + kRows - 1) / kRows <= 0x7fffffffLL, "too many rows");
    size_t lds = (size_t)kRows * dim * sizeof(float);
    if (lds < 4 * kRows * sizeof(uint64_t)) lds = 4 * kRows * sizeof(uint64_t);
    hipLaunchKernelGGL(nearest_centroid_kernel, dim3((unsigned)((n + kRows - 1) / kRows)), dim3(256), lds, s,
                       x_dev, n, dim, cent_dev, nlist, assign_dev);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

int launch_build_jobs(const int32_t *probed_dev, int64_t nq, int nprobe, int nlist, int pilot, int tq,
                      const IvfJobBuffers &b, hipStream_t s)
{
    const int64_t njobs = nq * nprobe;
    if (njobs <= kDirectJobs) {  // a few queries: latency matters, sharing of code loads does not
        hipLaunchKernelGGL(direct_jobs_kernel, dim3((unsigned)((njobs + 255) / 256)), dim3(256), 0, s, probed_dev,
                           (int)nq, nprobe, b.job_q, b.job_list, b.job_slot, (TileRec *)b.tiles,
                           b.tile_begin + 2 * nlist);
        PSC_HIP_TRY(hipGetLastError());
        return PSC_OK;
    }
    const int64_t nblk = (nq + kJobBlockQ - 1) / kJobBlockQ;
    const int nkeys = 2 * nlist;
    PSC_REQUIRE(njobs < 0x7fffffffLL && nblk * nkeys < ((int64_t)1 << 40), "too many jobs");
    const int64_t hcells = nblk * nkeys;
    hipLaunchKernelGGL(zero_i32_kernel, dim3((unsigned)((hcells + 255) / 256)), dim3(256), 0, s, b.hist, hcells);
    hipLaunchKernelGGL(job_hist_kernel, dim3((unsigned)((njobs + 255) / 256)), dim3(256), 0, s, probed_dev, nq,
                       nprobe, nlist, pilot, b.hist);
    hipLaunchKernelGGL(job_column_prefix_kernel, dim3((unsigned)((nkeys + 255) / 256)), dim3(256), 0, s, b.hist,
                       nblk, nkeys, b.list_begin);
    hipLaunchKernelGGL(job_list_prefix_kernel, dim3(1), dim3(1024), 0, s, b.list_begin, b.tile_begin, nkeys, tq);
    hipLaunchKernelGGL(job_scatter_kernel, dim3((unsigned)nblk), dim3(256), 0, s, probed_dev, nq, nprobe, nlist,
                       pilot, b.hist, b.list_begin, b.job_q, b.job_list, b.job_slot);
    hipLaunchKernelGGL(job_tiles_kernel, dim3((unsigned)((nkeys + 255) / 256)), dim3(256), 0, s, b.list_begin,
                       b.tile_begin, nlist, tq, (TileRec *)b.tiles);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

}  // namespace psc
