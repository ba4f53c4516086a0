// Lloyd k-means on the GPU for the product quantizer (Section 3, opening: one k-means of 256
// centroids per sub-space) and for the coarse quantizer of the inverted file (Section 4.3).
// Offline work, left of the scan: the search path never comes here.
//
// One iteration = assignment (nearest centroid in float32, lowest number on ties) + the sums and
// counts of every cell; the new centroid is sum / count in double precision, rounded to float32.
// Sums are order-dependent in their last bits (atomic adds), so two runs agree to rounding, not
// bit for bit.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <iterator>

#include "common.h"
#include "pq_nearest.h"

namespace psc {

namespace {

// ---------------------------------------------------------------------------------------------
// Product quantizer: grid (row blocks, m).  A workgroup keeps a private copy of its cells' sums
// (float32: a workgroup adds a few members per cell) and counts in LDS, walks its share of the rows
// (one row per thread and turn), and adds its sums to the global ones (double) at the end.  Per row
// it also stores the cell and the distance, for the refill of empty cells.  The centroids, the same
// for every lane, come through the scalar cache: read from LDS, four 16-byte reads per 32 vector
// instructions, they take as long as the arithmetic.  For sub-vectors of 48 and 64, whose operands and sums do not
// fit LDS, and of 1, where nearly every row is a close call (1M rows, 16 sub-quantizers 677 / 1600 us an
// iteration); the others take pq_lloyd_mfma_kernel.  Few rows with sub-vectors of 1 do read the centroids from LDS (STAGED):
// there are not the waves to hide the scalar cache's trips.  An iteration with LDS / scalar cache, us: 8 sub-quantizers,
// 300 rows 56 / 62, 3000 59 / 62, 30k 98 / 99, 1M 382 / 383; 16, 300 54 / 58, 300k 275 / 274, 1M 691 / 674.
// ---------------------------------------------------------------------------------------------
template <int DSUB, bool STAGED>
__global__ void __launch_bounds__(256)
pq_lloyd_step_kernel(const float *__restrict__ cb, int dim, int m, const float *__restrict__ x, int64_t n,
                     uint8_t *__restrict__ cell, float *__restrict__ dmin, double *__restrict__ gsum,
                     uint32_t *__restrict__ gcount, double *__restrict__ gobj)
{
    extern __shared__ float smem[];
    constexpr int LD = DSUB + 1;  // pitch of a cell's sums: a coordinate's additions hit all banks, not a few
    float *sum = smem;                                    // [256][LD]
    uint32_t *cnt = (uint32_t *)(smem + kCentroids * LD);  // [256]
    const int j = blockIdx.y, tid = threadIdx.x;
    const float *__restrict__ from = cb + (int64_t)j * kCentroids * DSUB;
    __shared__ float staged[STAGED ? kCentroids * DSUB : 1];
    if constexpr (STAGED)
        for (int e = tid; e < kCentroids * DSUB; e += 256) staged[e] = from[e];
    const float *cen = STAGED ? staged : from;  // (the same address in every lane)
    for (int e = tid; e < kCentroids * LD; e += 256) sum[e] = 0.f;
    cnt[tid] = 0u;
    __syncthreads();
    double obj = 0.0;
    for (int64_t r = (int64_t)blockIdx.x * 256 + tid; r < n; r += (int64_t)gridDim.x * 256) {
        float v[DSUB];
#pragma unroll
        for (int t = 0; t < DSUB; ++t) v[t] = x[r * dim + j * DSUB + t];
        float best = __builtin_inff();
        int bi = 0;
#pragma unroll 2
        for (int c = 0; c < kCentroids; ++c) {
            float acc = 0.f;
#pragma unroll
            for (int t = 0; t < DSUB; ++t) {
                const float df = v[t] - cen[c * DSUB + t];
                acc = fmaf(df, df, acc);
            }
            if (acc < best) {
                best = acc;
                bi = c;
            }
        }
        cell[r * m + j] = (uint8_t)bi;
        dmin[r * m + j] = best;
        obj += (double)best;
#pragma unroll
        for (int t = 0; t < DSUB; ++t) unsafeAtomicAdd(&sum[bi * LD + t], v[t]);
        atomicAdd(&cnt[bi], 1u);
    }
    __syncthreads();
    for (int e = tid; e < kCentroids * DSUB; e += 256)
        if (cnt[e / DSUB] != 0u)
            unsafeAtomicAdd(&gsum[(int64_t)j * kCentroids * DSUB + e], (double)sum[e / DSUB * LD + e % DSUB]);
    if (cnt[tid] != 0u) atomicAdd(&gcount[j * kCentroids + tid], cnt[tid]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) obj += __shfl_xor(obj, off, 64);
    if ((tid & 63) == 0) unsafeAtomicAdd(&gobj[j], obj);
}

// ---------------------------------------------------------------------------------------------
// The same step with the search on the matrix cores (pq_nearest.h), for sub-vectors whose operands and sums fit
// LDS together.  Workgroup b of sub-quantizer j (block b * m + j) walks every nb-th 32 x waves rows, adds its rows
// to sums in LDS (double precision) and writes them, its counts and its share of the objective to part b
// of the scratch arrays; pq_lloyd_update_kernel adds the parts up in a fixed order.  No launch clears anything and
// nothing but LDS is added to atomically: 196 workgroups a sub-quantizer adding 4096 doubles each to the
// same addresses took most of what the search left.
// `stop`: set by the update when a cell came out empty (iteration + 1): everything after it leaves at once, and
// the host refills the cells and goes on from there.
// Bound by vector issue (2.5 instructions per centroid and row), then by its start and end.  An iteration, before /
// after, us: 8 sub-vectors of 16, 300 rows 81 / 21, 100k 254 / 74, 1M 1508 / 447; of 32 114 / 33, 506 / 111,
// 3546 / 747; 16 of 4, 100k 196 / 77; 8 of 2, 1M 442 / 255.
// ---------------------------------------------------------------------------------------------
template <int DSUB>
struct LloydLds {
    static constexpr int LD = DSUB + 1;  // pitch of a cell's sums: a coordinate's additions hit all banks, not a few
    typename PqNearest<DSUB>::Shared nearest;
    double sum[kCentroids * LD];
    uint32_t cnt[kCentroids];
    double obj;
};
constexpr int kLloydThreads = 512;

template <int DSUB>
__global__ void __launch_bounds__(kLloydThreads) __attribute__((amdgpu_waves_per_eu(PqNearest<DSUB>::kWavesPerEu)))
pq_lloyd_mfma_kernel(const float *__restrict__ cb, int dim, int m, const float *__restrict__ x, int64_t n,
                     uint8_t *__restrict__ cell, float *__restrict__ dmin, double *__restrict__ part_sum,
                     uint32_t *__restrict__ part_count, double *__restrict__ part_obj, const int *__restrict__ stop)
{
    if (*stop != 0) return;
    typedef PqNearest<DSUB> Nearest;
    constexpr int kThreads = kLloydThreads, kWaves = kThreads / 64, LD = LloydLds<DSUB>::LD;
    extern __shared__ __align__(16) unsigned char lloyd_smem[];
    LloydLds<DSUB> &s = *(LloydLds<DSUB> *)lloyd_smem;
    const int j = (int)(blockIdx.x % (unsigned)m), b = (int)(blockIdx.x / (unsigned)m), nb = (int)(gridDim.x / (unsigned)m);
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
    const float *cbj = cb + (int64_t)j * kCentroids * DSUB;
    for (int e = tid; e < kCentroids * LD; e += kThreads) s.sum[e] = 0.0;
    if (tid < kCentroids) s.cnt[tid] = 0u;
    if (tid == 0) s.obj = 0.0;
    Nearest::prepare(s.nearest, cbj);
    double obj = 0.0;
    const int64_t step = (int64_t)nb * (kWaves * 32);
    bool plain = false;  // (wave-uniform) a row to each lane: two turns' rows at once
    for (int64_t r0 = ((int64_t)b * kWaves + wave) * 32; r0 < n;) {
        const int64_t own = r0 + (lane & 31) + (plain && half ? step : 0);
        const bool live = own < n;
        const int64_t r = live ? own : n - 1;
        float v[DSUB];
#pragma unroll
        for (int t = 0; t < DSUB; ++t) v[t] = x[r * dim + j * DSUB + t];
        r0 += plain ? 2 * step : step;
        const bool alone = plain;
        const int c = plain ? Nearest::all_distances(cbj, v) : Nearest::search(s.nearest, cbj, v, live, plain);
        float d = Nearest::distance(v, cbj + c * DSUB);
        if (!(d < __builtin_inff())) d = __builtin_inff();  // (a row that is not a number is at infinity)
        if (!live) continue;
        if (half == 0 || alone) {
            cell[r * m + j] = (uint8_t)c;
            dmin[r * m + j] = d;
            obj += (double)d;
            atomicAdd(&s.cnt[c], 1u);
        }
        double *to = s.sum + c * LD;
        if (alone) {
#pragma unroll
            for (int t = 0; t < DSUB; ++t) unsafeAtomicAdd(to + t, (double)v[t]);
        } else {  // a coordinate each from the row's two lanes
#pragma unroll
            for (int t = 0; t < DSUB; t += 2) unsafeAtomicAdd(to + t + half, (double)(half ? v[t + 1] : v[t]));
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) obj += __shfl_xor(obj, off, 64);
    if (lane == 0) unsafeAtomicAdd(&s.obj, obj);
    __syncthreads();
    double *out = part_sum + ((int64_t)j * nb + b) * (kCentroids * DSUB);
    for (int e = tid; e < kCentroids * DSUB; e += kThreads) out[e] = s.sum[e / DSUB * LD + e % DSUB];
    if (tid < kCentroids) part_count[((int64_t)j * nb + b) * kCentroids + tid] = s.cnt[tid];
    if (tid == 0) part_obj[j * nb + b] = s.obj;
}

// Sums, counts and objective of the step's parts; the new centroid of every cell that has members.
// One thread per coordinate of a cell, 256 to a workgroup (a workgroup sees one sub-quantizer).
__global__ void __launch_bounds__(256)
pq_lloyd_update_kernel(const double *__restrict__ part_sum, const uint32_t *__restrict__ part_count,
                       const double *__restrict__ part_obj, int nb, int dsub, int iteration, double *__restrict__ gsum,
                       uint32_t *__restrict__ gcount, double *__restrict__ gobj, float *__restrict__ cb, int *__restrict__ stop)
{
    const int seen = *(volatile int *)stop;
    if (seen != 0 && seen != iteration + 1) return;
    const int j = (int)blockIdx.y, per = kCentroids * dsub, e = (int)blockIdx.x * 256 + (int)threadIdx.x;
    const int c = e / dsub;
    const double *sums = part_sum + (int64_t)j * nb * per + e;
    const uint32_t *counts = part_count + (int64_t)j * nb * kCentroids + c;
    double sum = 0.0;
    uint32_t cnt = 0u;
#pragma unroll 8
    for (int b = 0; b < nb; ++b) {
        sum += sums[(int64_t)b * per];
        cnt += counts[b * kCentroids];
    }
    gsum[(int64_t)j * per + e] = sum;
    if (cnt != 0u) cb[(int64_t)j * per + e] = (float)(sum / (double)cnt);
    if (e % dsub == 0) {
        gcount[j * kCentroids + c] = cnt;
        if (cnt == 0u) *stop = iteration + 1;
    }
    if (e == 0) {
        double obj = 0.0;
        for (int b = 0; b < nb; ++b) obj += part_obj[j * nb + b];
        gobj[j] = obj;
    }
}

// The 256 starting centroids of every sub-quantizer: sub-vector j of row rows[j][c].
__global__ void __launch_bounds__(256)
pq_gather_start_kernel(const float *__restrict__ x, int dim, int dsub, const int64_t *__restrict__ rows,
                       float *__restrict__ cb)
{
    const int j = blockIdx.x, c = threadIdx.x;
    const float *src = x + rows[j * kCentroids + c] * dim + j * dsub;
    float *dst = cb + ((int64_t)j * kCentroids + c) * dsub;
    for (int t = 0; t < dsub; ++t) dst[t] = src[t];
}

// Refill of an empty cell, step 1: the member of cell `big` of sub-quantizer j that lies farthest
// from its centroid, lowest row on equal distance.  key = (distance bits << 32) | ~row, maximised.
__global__ void __launch_bounds__(256)
pq_farthest_member_kernel(const uint8_t *__restrict__ cell, const float *__restrict__ dmin, int64_t n, int m,
                          int j, int big, unsigned long long *__restrict__ key)
{
    unsigned long long best = 0ull;
    for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < n; r += (int64_t)gridDim.x * 256)
        if (cell[r * m + j] == (uint8_t)big) {
            const unsigned long long k =
                ((unsigned long long)__float_as_uint(dmin[r * m + j]) << 32) | (0xffffffffu - (uint32_t)r);
            best = k > best ? k : best;
        }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const unsigned long long o = __shfl_xor(best, off, 64);
        best = o > best ? o : best;
    }
    if ((threadIdx.x & 63) == 0 && best != 0ull) atomicMax(key, best);
}

// Step 2: row `far` becomes the only member of the empty cell c (the sum and count of the cell
// it leaves stay as they are: that cell's mean still includes it in this iteration).
__global__ void pq_move_member_kernel(const float *__restrict__ x, int dim, int dsub, int m, int j, int64_t far,
                                      int c, uint8_t *__restrict__ cell, float *__restrict__ dmin,
                                      double *__restrict__ gsum, uint32_t *__restrict__ gcount)
{
    const int t = threadIdx.x;
    if (t < dsub) gsum[((int64_t)j * kCentroids + c) * dsub + t] = (double)x[far * dim + j * dsub + t];
    if (t == 0) {
        cell[far * m + j] = (uint8_t)c;
        dmin[far * m + j] = 0.f;
        gcount[j * kCentroids + c] = 1u;
    }
}

// cent[c] = sum[c] / count[c] for the cells that have members; the others keep their centroid.
__global__ void __launch_bounds__(256)
centroid_update_kernel(const double *__restrict__ gsum, const uint32_t *__restrict__ gcount, int64_t ncell,
                       int d, float *__restrict__ cent)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= ncell * d) return;
    const uint32_t cnt = gcount[e / d];
    if (cnt != 0u) cent[e] = (float)(gsum[e] / (double)cnt);
}

// ---------------------------------------------------------------------------------------------
// Coarse quantizer: the assignment comes from the nearest-centroid kernel; this adds every row to
// its cell.  One thread per (row, 4 coordinates), atomics straight to the global sums: the cells
// are too many for private copies, and a row's coordinates go to consecutive addresses.
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
coarse_accumulate_kernel(const float *__restrict__ x, int64_t n, int dim, const int32_t *__restrict__ assign,
                         double *__restrict__ gsum, uint32_t *__restrict__ gcount)
{
    const int q4 = dim / 4;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n * q4) return;
    const int64_t r = e / q4;
    const int t4 = (int)(e - r * q4);
    const int c = assign[r];
    const float4 v = *(const float4 *)(x + r * dim + 4 * t4);
    double *s = gsum + (int64_t)c * dim + 4 * t4;
    unsafeAtomicAdd(s + 0, (double)v.x);
    unsafeAtomicAdd(s + 1, (double)v.y);
    unsafeAtomicAdd(s + 2, (double)v.z);
    unsafeAtomicAdd(s + 3, (double)v.w);
    if (t4 == 0) atomicAdd(&gcount[c], 1u);
}

__global__ void __launch_bounds__(256)
gather_rows_kernel(const float *__restrict__ x, int dim, const int64_t *__restrict__ rows, int64_t nrows,
                   float *__restrict__ out)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= nrows * dim) return;
    const int64_t c = e / dim;
    out[e] = x[rows[c] * dim + (e - c * dim)];
}

// Refill of an empty coarse cell: the lowest-numbered member of cell `big`.
__global__ void __launch_bounds__(256)
coarse_first_member_kernel(const int32_t *__restrict__ assign, int64_t n, int big, unsigned long long *__restrict__ key)
{
    unsigned long long best = 0ull;
    for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < n; r += (int64_t)gridDim.x * 256)
        if (assign[r] == big) {
            const unsigned long long k = (1ull << 32) | (0xffffffffu - (uint32_t)r);
            best = k > best ? k : best;
        }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const unsigned long long o = __shfl_xor(best, off, 64);
        best = o > best ? o : best;
    }
    if ((threadIdx.x & 63) == 0 && best != 0ull) atomicMax(key, best);
}

__global__ void coarse_move_member_kernel(const float *__restrict__ x, int dim, int64_t far, int c,
                                          int32_t *__restrict__ assign, double *__restrict__ gsum,
                                          uint32_t *__restrict__ gcount)
{
    for (int t = threadIdx.x; t < dim; t += blockDim.x) gsum[(int64_t)c * dim + t] = (double)x[far * dim + t];
    if (threadIdx.x == 0) {
        assign[far] = c;
        gcount[c] = 1u;
    }
}

// The mean of the centroids, appended as row ncent: the reference point of the matrix-core
// distance kernel.  One workgroup per coordinate, a fixed order of additions.
__global__ void __launch_bounds__(256)
mean_centroid_kernel(float *__restrict__ cent, int ncent, int dim)
{
    __shared__ double part[4];
    const int t = blockIdx.x;
    double acc = 0.0;
    for (int c = threadIdx.x; c < ncent; c += 256) acc += (double)cent[(int64_t)c * dim + t];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) cent[(int64_t)ncent * dim + t] = (float)((part[0] + part[1] + part[2] + part[3]) / ncent);
}

template <int DSUB, bool STAGED>
int run_pq_step_form(const float *cb, int dim, int m, const float *x, int64_t n, uint8_t *cell, float *dmin,
                double *gsum, uint32_t *gcount, double *gobj, hipStream_t s)
{
    const size_t lds = (size_t)(kCentroids * (DSUB + 2)) * sizeof(float);
    if (lds > 48 * 1024)
        PSC_HIP_TRY(hipFuncSetAttribute((const void *)pq_lloyd_step_kernel<DSUB, STAGED>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    // at most 2048 workgroups (8 to a compute unit), all with the same number of turns
    const int64_t want = (n + 255) / 256, cap = 2048 / m, turns = (want + cap - 1) / cap;
    dim3 grid((unsigned)((want + turns - 1) / turns), (unsigned)m);
    hipLaunchKernelGGL((pq_lloyd_step_kernel<DSUB, STAGED>), grid, dim3(256), lds, s, cb, dim, m, x, n, cell, dmin,
                       gsum, gcount, gobj);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

template <int DSUB>
int run_pq_step(const float *cb, int dim, int m, const float *x, int64_t n, uint8_t *cell, float *dmin,
                double *gsum, uint32_t *gcount, double *gobj, hipStream_t s)
{
    // (up to 30k rows ahead, even up to 300k x 16 and 1M x 8)
    if constexpr (DSUB == 1)
        if (n * m <= 4'000'000) return run_pq_step_form<1, true>(cb, dim, m, x, n, cell, dmin, gsum, gcount, gobj, s);
    return run_pq_step_form<DSUB, false>(cb, dim, m, x, n, cell, dmin, gsum, gcount, gobj, s);
}

}  // namespace

int launch_pq_lloyd_step(const float *cb_dev, int dim, int m, const float *x_dev, int64_t n, uint8_t *cell_dev,
                         float *dmin_dev, double *sum_dev, uint32_t *count_dev, double *obj_dev, hipStream_t s)
{
    const size_t ncell = (size_t)m * kCentroids;
    PSC_HIP_TRY(hipMemsetAsync(sum_dev, 0, ncell * (size_t)(dim / m) * sizeof(double), s));
    PSC_HIP_TRY(hipMemsetAsync(count_dev, 0, ncell * sizeof(uint32_t), s));
    PSC_HIP_TRY(hipMemsetAsync(obj_dev, 0, (size_t)m * sizeof(double), s));
#define CALL(DS) run_pq_step<DS>(cb_dev, dim, m, x_dev, n, cell_dev, dmin_dev, sum_dev, count_dev, obj_dev, s)
    switch (dim / m) {
    case 1: return CALL(1);
    case 48: return CALL(48);
    case 64: return CALL(64);
    default:
        set_error("unsupported sub-vector length %d (supported: 1,2,4,6,8,12,16,24,32,48,64)", dim / m);
        return PSC_EINVAL;
    }
#undef CALL
}

template <int DSUB>
static int run_pq_lloyd(const PqLloydArgs &a, int iteration, hipStream_t s)
{
    const size_t lds = sizeof(LloydLds<DSUB>);
    PSC_HIP_TRY(hipFuncSetAttribute((const void *)pq_lloyd_mfma_kernel<DSUB>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)lds));
    hipLaunchKernelGGL((pq_lloyd_mfma_kernel<DSUB>), dim3((unsigned)(a.parts * a.m)), dim3(kLloydThreads), lds, s, a.cb,
                       a.dim, a.m, a.x, a.n, a.cell, a.dmin, a.part_sum, a.part_count, a.part_obj, a.stop);
    PSC_HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(pq_lloyd_update_kernel, dim3((unsigned)DSUB, (unsigned)a.m), dim3(256), 0, s, a.part_sum, a.part_count,
                       a.part_obj, a.parts, DSUB, iteration, a.sum, a.count, a.obj + (int64_t)iteration * a.m, a.cb, a.stop);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

int pq_lloyd_parts(int dim, int m, int64_t n)
{
    const int dsub = dim / m;
    static constexpr int kLengths[] = {2, 4, 6, 8, 12, 16, 24, 32};  // (launch_pq_lloyd's; the plain step refuses the rest)
    if (std::find(std::begin(kLengths), std::end(kLengths), dsub) == std::end(kLengths)) return 0;
    // as many workgroups as run together (two to a compute unit up to sub-vectors of 16), at least a turn each
    const int rows = 32 * kLloydThreads / 64;
    const int64_t want = (n + rows - 1) / rows, cap = std::max(1, (dsub <= 16 ? 512 : 256) / m), turns = (want + cap - 1) / cap;
    return (int)((want + turns - 1) / turns);
}

int launch_pq_lloyd(const PqLloydArgs &a, int iteration, hipStream_t s)
{
    switch (a.dim / a.m) {
    case 2: return run_pq_lloyd<2>(a, iteration, s);
    case 4: return run_pq_lloyd<4>(a, iteration, s);
    case 6: return run_pq_lloyd<6>(a, iteration, s);
    case 8: return run_pq_lloyd<8>(a, iteration, s);
    case 12: return run_pq_lloyd<12>(a, iteration, s);
    case 16: return run_pq_lloyd<16>(a, iteration, s);
    case 24: return run_pq_lloyd<24>(a, iteration, s);
    case 32: return run_pq_lloyd<32>(a, iteration, s);
    default: set_error("no matrix-core step for sub-vectors of %d", a.dim / a.m); return PSC_EINVAL;
    }
}

int launch_pq_gather_start(const float *x_dev, int dim, int m, const int64_t *rows_dev, float *cb_dev, hipStream_t s)
{
    hipLaunchKernelGGL(pq_gather_start_kernel, dim3((unsigned)m), dim3(kCentroids), 0, s, x_dev, dim, dim / m,
                       rows_dev, cb_dev);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

int launch_pq_refill(const float *x_dev, int64_t n, int dim, int m, int j, int big, int c, uint8_t *cell_dev,
                     float *dmin_dev, double *sum_dev, uint32_t *count_dev, unsigned long long *key_dev,
                     hipStream_t s)
{
    PSC_HIP_TRY(hipMemsetAsync(key_dev, 0, sizeof(unsigned long long), s));
    const int64_t want = (n + 255) / 256;
    hipLaunchKernelGGL(pq_farthest_member_kernel, dim3((unsigned)(want < 1024 ? want : 1024)), dim3(256), 0, s,
                       cell_dev, dmin_dev, n, m, j, big, key_dev);
    PSC_HIP_TRY(hipGetLastError());
    unsigned long long key = 0;
    PSC_HIP_TRY(hipMemcpyAsync(&key, key_dev, sizeof key, hipMemcpyDeviceToHost, s));
    PSC_HIP_TRY(hipStreamSynchronize(s));
    if (key == 0ull) return PSC_OK;  // the cell has no member: nothing to move
    const int64_t far = (int64_t)(0xffffffffu - (uint32_t)(key & 0xffffffffull));
    hipLaunchKernelGGL(pq_move_member_kernel, dim3(1), dim3(64), 0, s, x_dev, dim, dim / m, m, j, far, c,
                       cell_dev, dmin_dev, sum_dev, count_dev);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

int launch_centroid_update(const double *sum_dev, const uint32_t *count_dev, int64_t ncell, int d, float *cent_dev,
                           hipStream_t s)
{
    const int64_t total = ncell * d;
    hipLaunchKernelGGL(centroid_update_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, sum_dev,
                       count_dev, ncell, d, cent_dev);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

int launch_gather_rows(const float *x_dev, int dim, const int64_t *rows_dev, int64_t nrows, float *out_dev,
                       hipStream_t s)
{
    const int64_t total = nrows * dim;
    hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, x_dev, dim,
                       rows_dev, nrows, out_dev);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

int launch_coarse_accumulate(const float *x_dev, int64_t n, int dim, const int32_t *assign_dev, int ncent,
                             double *sum_dev, uint32_t *count_dev, hipStream_t s)
{
    PSC_HIP_TRY(hipMemsetAsync(sum_dev, 0, (size_t)ncent * dim * sizeof(double), s));
    PSC_HIP_TRY(hipMemsetAsync(count_dev, 0, (size_t)ncent * sizeof(uint32_t), s));
    const int64_t total = n * (dim / 4), blocks = (total + 255) / 256;
    if (blocks > 0x7fffffffLL) {
        set_error("too many training rows for one launch");
        return PSC_EINVAL;
    }
    hipLaunchKernelGGL(coarse_accumulate_kernel, dim3((unsigned)blocks), dim3(256), 0, s, x_dev, n, dim, assign_dev,
                       sum_dev, count_dev);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

int launch_coarse_refill(const float *x_dev, int64_t n, int dim, int big, int c, int32_t *assign_dev,
                         double *sum_dev, uint32_t *count_dev, unsigned long long *key_dev, hipStream_t s)
{
    PSC_HIP_TRY(hipMemsetAsync(key_dev, 0, sizeof(unsigned long long), s));
    const int64_t want = (n + 255) / 256;
    hipLaunchKernelGGL(coarse_first_member_kernel, dim3((unsigned)(want < 1024 ? want : 1024)), dim3(256), 0, s,
                       assign_dev, n, big, key_dev);
    PSC_HIP_TRY(hipGetLastError());
    unsigned long long key = 0;
    PSC_HIP_TRY(hipMemcpyAsync(&key, key_dev, sizeof key, hipMemcpyDeviceToHost, s));
    PSC_HIP_TRY(hipStreamSynchronize(s));
    if (key == 0ull) return PSC_OK;
    const int64_t far = (int64_t)(0xffffffffu - (uint32_t)(key & 0xffffffffull));
    hipLaunchKernelGGL(coarse_move_member_kernel, dim3(1), dim3(256), 0, s, x_dev, dim, far, c, assign_dev,
                       sum_dev, count_dev);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

int launch_mean_centroid(float *cent_dev, int ncent, int dim, hipStream_t s)
{
    hipLaunchKernelGGL(mean_centroid_kernel, dim3((unsigned)dim), dim3(256), 0, s, cent_dev, ncent, dim);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

}  // namespace psc
