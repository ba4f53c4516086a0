// The fused polysemous scan (Section 3.3 two-step strategy; Section 4.2 "dual") for gfx950.
//
// One workgroup = one tile of TQ queries x one slice of the database.
//   * the TQ ADC tables (TQ * m * 256 float32) and the TQ running top-k lists live in LDS for
//     the lifetime of the workgroup;
//   * the TQ query codes live in scalar registers;
//   * every wave streams blocks of 64 x CB codes from memory into vector registers (16-byte
//     loads, four blocks per turn with the next four already requested; CB = 32 / TQ codes per
//     lane) and compares each code with all TQ query codes: xor + popcount-accumulate per
//     32-bit word, then one funnel shift that appends the "too far" bit to a 32-bit per-lane
//     mask (one bit per (code, query)): 5 integer instructions per (query, 64-bit code) pair;
//   * lanes that hold survivors append their mask and its position to a per-wave queue in LDS,
//     places assigned with ballot + prefix popcount, so that the expensive step runs on full
//     wavefronts;
//   * whenever the queue holds 64 masks the wave scores one survivor of each of the newest 64:
//     re-reads the codes, gathers m table entries each from LDS, sums them in float32 (j ascending)
//     and compares with the query's current bound on its k-th best distance; masks with survivors
//     left are appended again;
//   * the few candidates that pass are spliced into the query's sorted list in LDS by the whole
//     wave, under a per-query lock (waves of the workgroup share the lists); workgroups of one
//     query tell each other how far their lists have come through a few words in global memory
//     (their k-th best distance, or -- a query cut into many slices -- an earlier entry of each
//     list, from which a bound on the k-th best of all of them follows: ScanArgs::pub_slots).
// Partial lists (one per query and slice) go to the workspace; a second kernel merges them.
//
// Ordering everywhere: (distance, id) ascending, lower id first on equal distance.
#include <atomic>
#include <cfloat>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "common.h"
#include "entry.h"

namespace psc {
namespace {

constexpr int kQueueCap = 95;         // queue entries per wave (8 bytes each, and one to spare; see score_survivors)
constexpr int kMfmaQueueCap = 111;    // the same for the matrix-core filter, whose blocks bring more of them
constexpr int64_t kMaxSliceLen = (int64_t)1 << 27;
// Queue entries of the matrix-core filter: a lane's first code is at most the block's position (a multiple of
// 128, of 256 at 128 bits) + 15 (31), so the bits above hold the lane's group of query slots.
template <int M>
constexpr uint32_t kGroupShift = M == 8 ? 4u : 5u;
template <int M>
constexpr uint32_t kGroupMask = M == 8 ? 3u : 1u;
// Fewer queries than this take the narrower xor/popcount tiles (those scans are bound by memory; 128
// bits, 50M codes, 5 and 8 queries, k = 100: 0.18 to 0.24 ms at ht = 0 .. 48 with either filter).
constexpr int64_t kMfmaMinQueries = 9;
constexpr int kSpinLimit = 1 << 22;   // bounded wait on a list lock (each turn sleeps)
constexpr int kManySlices = 4;        // slices per query from which the lists exchange more than their k-th best

struct IvfTile {
    int32_t job_begin, njobs, list, pad;
};

struct ScanArgs {
    const float *lut;         // [nq][M][256]
    const uint8_t *qcodes;    // [nq][M]
    const uint8_t *codes;     // [n][M]
    int64_t skip_first;       // >= 0: query q never returns database row skip_first + q (graph mode)
    int64_t nq, n;
    int64_t slice_len;
    int nslice;
    int64_t tiles_one;        // flat mode: the first tiles_one query tiles scan the whole database in one piece
    int k, kpad;
    uint32_t bias;            // 0x7fffffff - ht: bit 31 of (bias + distance) <=> distance > ht
    float *part_d;            // [nq][nslice][k]
    int64_t *part_i;          // [nq][nslice][k]
    int *status;              // set non-zero if a bounded wait expired
    // Per query, the smallest k-th-best distance any workgroup working for that query has
    // reached so far, as a sortable key (see dist_key).  Nothing farther than it can be in the
    // query's final top-k, so every workgroup of the query prunes with it: the partial lists
    // of one query behave like one stream instead of one warm-up per slice or list.
    uint32_t *gthr;           // [number of queries][pub_slots] (pub_slots = 1: as described; more: see pub_slots)
    const int32_t *job_q;     // inverted-file mode: query of each job (index into gthr)
    // inverted-file mode (Section 4.3): a tile = up to TQ (query, list) jobs of ONE list, rows
    // job_begin.. of the job-sorted tables / query codes; the scanned range is that list
    const IvfTile *tiles;     // [*ntiles]
    const int *ntiles;        // device-side count (the grid is an upper bound)
    const int64_t *list_off;  // [nlist+1] list boundaries in `codes`
    const int32_t *ext_ids;   // [n] id of each stored code
    const int32_t *job_slot;  // [njobs] partial list (query * nprobe + probe) a job writes
    // Residual tables of the inverted file, not stored per job.  With o the mean coarse
    // centroid, q~ = q - o and g~ = g - o for the coarse centroid g of the tile's list,
    //   ||(q - g)_j - c||^2 = (||c||^2 - 2 q~_j . c)  +  2 g~_j . c  +  ||(q - g)_j||^2
    //                       = lut[query][j][c] + list_tab[list][j][c] + (one number per job and j),
    // which a tile puts together in LDS (the first two, whose sum ||c||^2 - 2 (q - g)_j . c is of
    // the size of the result, before the third).  The query code of a job is the arg-min of those
    // rows.  list_tab == nullptr: `lut` holds one finished table per job, in job order (indexes
    // whose coarse centroids lie so far apart that the sum above would lose too many bits).
    const float *list_tab;    // [nlist][M][256]
    const float *queries;     // [nq][dim] raw query vectors
    const float *coarse;      // [nlist + 1][dim] coarse centroids, then their mean
    uint8_t *job_qcodes;      // [njobs][M] out: query code of each job
    int dim, nlist;
    // A few jobs, one per tile (latency matters): the tile's unused query slots serve the same
    // job, each wave feeding the list of slot wave % TQ, so that a list's lock is shared by a
    // quarter of the waves while the lists fill; the lists are merged when the tile ends.
    int spread_lists = 0;
    // Many slices per query (a handful of queries over a large database: every slice's list
    // would otherwise warm up on its own share only).  gthr then holds pub_slots words per query;
    // a list with pub_r entries or more keeps the key of its pub_r-th best in word slice %
    // pub_slots (atomic minimum over the lists that share the word).  Lists of different words
    // hold different codes, so a value v with pub_kth words at or below it has pub_kth * pub_r
    // >= k codes at or below it: nothing farther than v is in the query's top k.  With one word,
    // pub_r = k and pub_kth = 1 this is the plain exchange of k-th best distances.
    int pub_slots = 1, pub_r = 0, pub_kth = 1;
    // Flat mode: a word per query, non-zero for those this scan is to answer (nullptr: all of them).  Tiles (workgroups
    // of the small scan) without such a query end at once.
    const uint32_t *redo = nullptr;
};

// Flat mode: which queries and which part of the database a workgroup works on.  Query tiles
// 0 .. tiles_one-1 are scanned in one piece each (they fill whole rounds of workgroups that run
// together); the tiles after them are cut into nslice slices each, so that the last, partial
// round finishes in 1/nslice of the time instead of leaving compute units idle.  A query scanned
// in one piece builds one list instead of nslice: fewer insertions and a cheaper merge.
struct FlatTile {
    int slice;
    bool whole;  // one piece: the other slices' places in the partial lists get padding
    int64_t q0, slice_begin, slice_end;
};
__device__ __forceinline__ FlatTile flat_tile(const ScanArgs &a, int64_t tile, int tq)
{
    FlatTile t;
    if (tile < a.tiles_one) {
        t.slice = 0;
        t.whole = true;
        t.q0 = tile * tq;
        t.slice_begin = 0;
        t.slice_end = a.n;
    } else {
        const int64_t u = tile - a.tiles_one;
        t.slice = (int)(u % a.nslice);
        t.whole = false;
        t.q0 = (a.tiles_one + u / a.nslice) * tq;
        t.slice_begin = (int64_t)t.slice * a.slice_len;
        t.slice_end = (t.slice_begin + a.slice_len) < a.n ? (t.slice_begin + a.slice_len) : a.n;
    }
    return t;
}
// Whether a tile of up to 64 queries has one that ScanArgs::redo asks for.
__device__ __forceinline__ bool tile_wanted(const ScanArgs &a, int64_t q0, int nvq)
{
    if (a.redo == nullptr) return true;
    const int lane = (int)(threadIdx.x & 63);
    return __ballot(lane < nvq && a.redo[q0 + lane] != 0u) != 0ull;
}
// Padding for the partial lists a one-piece tile leaves unused (slices 1 .. nslice-1 of its queries).
__device__ __forceinline__ void pad_unused_slices(const ScanArgs &a, int64_t q0, int nvq, int tid, int nthreads)
{
    const int per_q = (a.nslice - 1) * a.k;
    for (int e = tid; e < nvq * per_q; e += nthreads) {
        const int q = e / per_q, r = e - q * per_q;
        const int64_t o = ((q0 + q) * a.nslice + 1) * a.k + r;
        a.part_d[o] = __builtin_inff();
        a.part_i[o] = (int64_t)-1;
    }
}

__device__ __forceinline__ float bcast_f(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ uint32_t bcast_u(uint32_t v, int lane)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

// Shared-memory view of one workgroup.  The pointers carry the LDS address space explicitly so
// that every access is a ds_* instruction.
typedef PSC_LDS float lds_f32;
typedef PSC_LDS volatile float lds_vf32;
typedef PSC_LDS volatile uint32_t lds_vu32;
typedef PSC_LDS uint32_t lds_u32;
typedef PSC_LDS volatile int lds_vi32;
typedef PSC_LDS int lds_i32;

typedef PSC_LDS volatile uint64_t lds_vu64;
typedef PSC_LDS uint64_t lds_u64;

static_assert(kPresetWord == kKeyInf, "init_scan_kernel presets the words too");

template <int M, int TQ>
struct Lds {
    lds_f32 *lut;    // [TQ][M][256]
    lds_vu64 *top;   // [TQ][kpad] sorted ascending
    lds_vf32 *thr;   // [TQ] bound on the query's k-th best distance (+inf while nothing is known)
    lds_i32 *lock;   // [TQ] number of entries in the list, or kLocked while a wave works on it
    lds_i32 *gidx;   // [TQ] the slot's query as an index into the shared thresholds (-1: empty slot)
    lds_i32 *pslot;  // [TQ] word of the query's shared thresholds the slot's list publishes to
    lds_f32 *sterm;  // [TQ][M] inverted file: the per-job, per-sub-quantizer constant of the tables
    lds_u32 *qcw;    // [TQ][M/4] inverted file: the jobs' query codes
    lds_u64 *queue;  // [nwaves][entries]; private to a wave: LDS keeps a wave's accesses in order
    __device__ __forceinline__ Lds(PSC_LDS unsigned char *base, int kpad)
    {
        lut = (lds_f32 *)base;
        top = (lds_vu64 *)(lut + TQ * M * 256);
        thr = (lds_vf32 *)(top + TQ * kpad);
        lock = (lds_i32 *)(thr + TQ);
        gidx = lock + TQ;
        pslot = gidx + TQ;
        sterm = (lds_f32 *)(pslot + TQ);
        qcw = (lds_u32 *)(sterm + TQ * M);
        queue = (lds_u64 *)(qcw + TQ * M / 4);
    }
};

// ---- the Hamming test of Section 3.3, hand-written ------------------------------------------
// For one code (words w) and NQ queries whose code words sit in scalar registers: per pair one
// v_xor and one v_bcnt (population count plus accumulator) per 32-bit word, the accumulator
// starting at `bias` = 0x7fffffff - ht so that its sign bit says "farther than ht", and one
// v_alignbit that shifts that bit into `far`.  5 instructions per 64-bit pair, 9 per 128-bit
// pair; written out because the compiler, left to itself, sometimes regroups the sum into
// (count + count) + bias at the price of one more instruction per pair.
#define PSC_PAIR_W2(QA, QB)                          \
    "v_xor_b32_e32 %[t0], %[" QA "], %[w0]\n\t"       \
    "v_bcnt_u32_b32 %[t0], %[t0], %[b]\n\t"           \
    "v_xor_b32_e32 %[t1], %[" QB "], %[w1]\n\t"       \
    "v_bcnt_u32_b32 %[t0], %[t1], %[t0]\n\t"          \
    "v_alignbit_b32 %[far], %[far], %[t0], 31\n\t"
#define PSC_PAIR_W4(QA, QB, QC, QD)                  \
    "v_xor_b32_e32 %[t0], %[" QA "], %[w0]\n\t"       \
    "v_bcnt_u32_b32 %[t0], %[t0], %[b]\n\t"           \
    "v_xor_b32_e32 %[t1], %[" QB "], %[w1]\n\t"       \
    "v_bcnt_u32_b32 %[t0], %[t1], %[t0]\n\t"          \
    "v_xor_b32_e32 %[t1], %[" QC "], %[w2]\n\t"       \
    "v_bcnt_u32_b32 %[t0], %[t1], %[t0]\n\t"          \
    "v_xor_b32_e32 %[t1], %[" QD "], %[w3]\n\t"       \
    "v_bcnt_u32_b32 %[t0], %[t1], %[t0]\n\t"          \
    "v_alignbit_b32 %[far], %[far], %[t0], 31\n\t"

// four queries, 64-bit codes
__device__ __forceinline__ void hamming_test4(uint32_t &far, const uint32_t (&w)[2], uint32_t bias,
                                              const uint32_t (*q)[2])
{
    uint32_t t0, t1;
    asm(PSC_PAIR_W2("q0a", "q0b") PSC_PAIR_W2("q1a", "q1b") PSC_PAIR_W2("q2a", "q2b") PSC_PAIR_W2("q3a", "q3b")
        : [far] "+v"(far), [t0] "=&v"(t0), [t1] "=&v"(t1)
        : [w0] "v"(w[0]), [w1] "v"(w[1]), [b] "s"(bias), [q0a] "s"(q[0][0]), [q0b] "s"(q[0][1]),
          [q1a] "s"(q[1][0]), [q1b] "s"(q[1][1]), [q2a] "s"(q[2][0]), [q2b] "s"(q[2][1]), [q3a] "s"(q[3][0]),
          [q3b] "s"(q[3][1]));
}
// eight queries, 64-bit codes
__device__ __forceinline__ void hamming_test8(uint32_t &far, const uint32_t (&w)[2], uint32_t bias,
                                              const uint32_t (*q)[2])
{
    uint32_t t0, t1;
    asm(PSC_PAIR_W2("q0a", "q0b") PSC_PAIR_W2("q1a", "q1b") PSC_PAIR_W2("q2a", "q2b") PSC_PAIR_W2("q3a", "q3b")
            PSC_PAIR_W2("q4a", "q4b") PSC_PAIR_W2("q5a", "q5b") PSC_PAIR_W2("q6a", "q6b") PSC_PAIR_W2("q7a", "q7b")
        : [far] "+v"(far), [t0] "=&v"(t0), [t1] "=&v"(t1)
        : [w0] "v"(w[0]), [w1] "v"(w[1]), [b] "s"(bias), [q0a] "s"(q[0][0]), [q0b] "s"(q[0][1]),
          [q1a] "s"(q[1][0]), [q1b] "s"(q[1][1]), [q2a] "s"(q[2][0]), [q2b] "s"(q[2][1]), [q3a] "s"(q[3][0]),
          [q3b] "s"(q[3][1]), [q4a] "s"(q[4][0]), [q4b] "s"(q[4][1]), [q5a] "s"(q[5][0]), [q5b] "s"(q[5][1]),
          [q6a] "s"(q[6][0]), [q6b] "s"(q[6][1]), [q7a] "s"(q[7][0]), [q7b] "s"(q[7][1]));
}
// four queries, 128-bit codes
__device__ __forceinline__ void hamming_test4(uint32_t &far, const uint32_t (&w)[4], uint32_t bias,
                                              const uint32_t (*q)[4])
{
    uint32_t t0, t1;
    asm(PSC_PAIR_W4("q0a", "q0b", "q0c", "q0d") PSC_PAIR_W4("q1a", "q1b", "q1c", "q1d")
            PSC_PAIR_W4("q2a", "q2b", "q2c", "q2d") PSC_PAIR_W4("q3a", "q3b", "q3c", "q3d")
        : [far] "+v"(far), [t0] "=&v"(t0), [t1] "=&v"(t1)
        : [w0] "v"(w[0]), [w1] "v"(w[1]), [w2] "v"(w[2]), [w3] "v"(w[3]), [b] "s"(bias), [q0a] "s"(q[0][0]),
          [q0b] "s"(q[0][1]), [q0c] "s"(q[0][2]), [q0d] "s"(q[0][3]), [q1a] "s"(q[1][0]), [q1b] "s"(q[1][1]),
          [q1c] "s"(q[1][2]), [q1d] "s"(q[1][3]), [q2a] "s"(q[2][0]), [q2b] "s"(q[2][1]), [q2c] "s"(q[2][2]),
          [q2d] "s"(q[2][3]), [q3a] "s"(q[3][0]), [q3b] "s"(q[3][1]), [q3c] "s"(q[3][2]), [q3d] "s"(q[3][3]));
}
// all TQ queries of a tile against one code
template <int TQ, int WPC>
__device__ __forceinline__ void hamming_test_tile(uint32_t &far, const uint32_t (&w)[WPC], uint32_t bias,
                                                  const uint32_t (&qw)[TQ][WPC])
{
    if constexpr (WPC == 2 && TQ % 8 == 0) {
#pragma unroll
        for (int q = 0; q < TQ; q += 8) hamming_test8(far, w, bias, &qw[q]);
    } else {
#pragma unroll
        for (int q = 0; q < TQ; q += 4) hamming_test4(far, w, bias, &qw[q]);
    }
}

// Smallest value of v over the wave, in every lane: four row-local steps on the data-parallel
// path, then the four row results through scalar registers.
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v)
{
    auto step = [](uint32_t x, uint32_t y) { return y < x ? y : x; };
    v = step(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xf, 0xf, false));   // lane ^ 1
    v = step(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xf, 0xf, false));   // lane ^ 2
    v = step(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xf, 0xf, false));  // mirror in 8
    v = step(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x140, 0xf, 0xf, false));  // mirror in 16
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 0);
    const uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
    const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)v, 32);
    const uint32_t r3 = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
    return step(step(r0, r1), step(r2, r3));
}

constexpr int kLocked = -1;

// The 64-bit value held by the lane below (lane 0 receives `first`): a whole-wave shift by one
// lane on the data-parallel path.
__device__ __forceinline__ uint64_t from_lane_below(uint64_t v, uint64_t first)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)first, (int)(uint32_t)v, 0x138, 0xf,
                                                              0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(first >> 32), (int)(uint32_t)(v >> 32),
                                                              0x138, 0xf, 0xf, false);
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t lane_value_u64(uint64_t v, int l)
{
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
}
// Whether a candidate comes before the k-th entry of slot q's list.  A place past the list's end holds
// kNoEntry, entries only ever get smaller, and a 64-bit LDS access is one access: whatever is read is a bound.
// The thresholds are distances alone and let every candidate through that ties with the k-th entry, though
// it loses by its id nearly always (ids rise during a scan); clustered vectors share codes by the thousand, and
// each such tie took the list's lock to be turned away.  Asked only when a batch has a tie.
// 10M x 10k at ht = 24, k = 100 24.6 -> 14.0 ms (of seeds with many codes at the k-th distance), 1M x 777 pure
// ADC 829 -> 744 us, 1M x 1M graph at ht = 20 80.4 -> 77.4 ms.  128-bit codes, 10M x 2000 at ht = 48: 10k distinct
// codes 3.33 -> 3.14 ms (by xor and popcount 5.66 -> 5.49), 1M x 2000, k = 10 0.331 -> 0.311; all distinct 3.12 / 3.08.
// Inverted lists do without: of 1M codes 1000 distinct 1.109 / 1.106 ms with it, of 10M of 128 bits 2.307 / 2.342, all
// distinct 2.195 / 2.219 (a job's list fills once, and few of its ties come after that).
template <int M, int TQ>
__device__ __forceinline__ bool before_kth(const Lds<M, TQ> &s, const ScanArgs &a, int q, float d, uint32_t id)
{
    return pack_entry(d, id) < s.top[q * a.kpad + a.k - 1];
}
// Lower a threshold in LDS, no answer awaited.
__device__ __forceinline__ void lower_threshold(lds_vf32 *p, float v)
{
    (void)__hip_atomic_fetch_min((lds_f32 *)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// An upper bound on the kth smallest (kth >= 1) of the keys held by the 64 lanes, the same in
// every lane: the key's upper 20 bits are found one by one, by counting the lanes at or below
// the value tried (sign, exponent and 11 bits of mantissa: within 0.05% of the exact value),
// the rest is filled with ones.  kKeyInf or above: fewer than kth lanes hold a finite key.
__device__ __forceinline__ uint32_t wave_kth_smallest_bound(uint32_t v, int kth)
{
    uint32_t prefix = 0u;
#pragma unroll 1
    for (int bit = 31; bit >= 12; --bit) {
        const uint32_t trial = prefix | ((1u << bit) - 1u);
        if (__builtin_popcountll(ballot64(v <= trial)) < kth) prefix |= 1u << bit;
    }
    return prefix | 0xfffu;
}

// Insert the candidates held by the lanes in `mine` (all for query slot q) into q's sorted list.
// Executed by the whole wave; mine is wave-uniform.  The slot's lock word doubles as the entry
// count, so taking the lock also fetches the count and releasing it stores the new one.
// Lists of up to 128 entries (two per lane) are read into registers once, every candidate is
// ranked by ballot and spliced in with a one-lane shift, and the list is written back once: two
// trips to LDS per call however many candidates it brings.
// SHARE: the list's k-th best is published to the other workgroups of the query.  EAGER: every
// call also reads what they have published (worth the wait at its end when a query is spread
// over hundreds of workgroups; with the few dozen lists of an inverted-file probe the reads made
// once per batch of candidates are enough).
template <int M, int TQ, bool SHARE, bool EAGER>
__device__ __forceinline__ void insert_candidates(const Lds<M, TQ> &s, const ScanArgs &a, int q, uint64_t mine,
                                                  float d, uint32_t id)
{
    const int lane = lane_id();
    // The other waves of the SIMD are busy filtering and would get three of every four issue
    // slots: whoever works on a list (and may hold its lock) goes first.
    __builtin_amdgcn_s_setprio(3);
    int cnt = kLocked;
    if (lane == 0) {
        int spins = 0;
        while (true) {
            cnt = __hip_atomic_exchange(&s.lock[q], kLocked, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (cnt != kLocked || ++spins > kSpinLimit) break;
            __builtin_amdgcn_s_sleep(2);
        }
    }
    cnt = __builtin_amdgcn_readfirstlane(cnt);
    if (cnt == kLocked) {  // never expected: flag the run instead of waiting for ever
        if (lane == 0) atomicExch(a.status, 1);
        __builtin_amdgcn_s_setprio(0);
        return;
    }
    // Everything the lock protects lives in LDS, which serves the accesses of a wave in the order
    // they were issued and those of different waves one after the other: a lock word taken by
    // an exchange and given back by a plain store after the data needs no hardware fence.  (A
    // workgroup-scope fence would also wait for every global load the wave has in flight, its
    // prefetched codes included, with the lock held.)  Only the compiler must keep the order.
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    // What the other workgroups of this query have reached by now: asked for here, used after
    // the lock is given back, so the trip to memory overlaps the work on the list.
    uint32_t seen = kKeyInf;
    int gi = -1;
    const bool many = SHARE && a.pub_slots > 1;  // (wave-uniform) the exchange over many slices
    uint32_t slots_seen = kKeyInf;               // many: lane l holds word l of the query
    int my_slot = 0;                             // many: the word this list publishes to
    if constexpr (SHARE) {
        if (many) {
            gi = __builtin_amdgcn_readfirstlane(s.gidx[q]);
            my_slot = __builtin_amdgcn_readfirstlane(s.pslot[q]);
            if (lane < a.pub_slots)
                slots_seen = __hip_atomic_load(&a.gthr[(int64_t)gi * a.pub_slots + lane], __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
        } else if (lane == 0) {
            gi = s.gidx[q];
            if constexpr (EAGER) seen = __hip_atomic_load(&a.gthr[gi], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    lds_vu64 *list = s.top + q * a.kpad;
    const int k = a.k;
    const int pr = a.pub_r;      // (1 <= pub_r <= k whenever `many`)
    uint32_t own_key = kKeyInf;  // the list's k-th best once it is full
    uint32_t pub_key = kKeyInf;  // many: the list's pub_r-th best once it has that many entries
    bool changed = false;
    float thr_old;
    if (k <= 128) {
        const int i0 = lane, i1 = 64 + lane;  // the two list places of the lane
        thr_old = s.thr[q];
        mine &= ballot64(d <= thr_old);  // the threshold may have dropped since the candidates were scored
        // Short lists (k <= 64, or a list that stays within 64 entries after this call: most lists
        // of inverted-file jobs) live in one register per lane.
        const bool one = k <= 64 || cnt + __builtin_popcountll(mine) <= 64;  // (wave-uniform)
        uint64_t e0 = ~0ull, e1 = ~0ull;  // places past the end hold the largest key
        if (i0 < cnt) e0 = list[i0];
        if (one) {
            while (mine) {
                const int src = __builtin_ctzll(mine);
                mine &= mine - 1;
                const uint64_t cand = pack_entry(bcast_f(d, src), bcast_u(id, src));
                const int pos = __builtin_popcountll(ballot64(e0 < cand));
                if (pos >= k) continue;
                const uint64_t up0 = from_lane_below(e0, e0);
                e0 = i0 > pos ? up0 : (i0 == pos ? cand : e0);
                if (i0 >= k) e0 = ~0ull;
                if (cnt < k) ++cnt;
                changed = true;
            }
            if (changed) {
                if (i0 < cnt) list[i0] = e0;
                if (cnt == k) own_key = (uint32_t)(lane_value_u64(e0, (k - 1) & 63) >> 32);  // (k <= 64 here)
                if (many && cnt >= pr) pub_key = (uint32_t)(lane_value_u64(e0, (pr - 1) & 63) >> 32);  // (pr <= cnt <= 64)
            }
        } else {
            if (i1 < cnt) e1 = list[i1];
            while (mine) {
                const int src = __builtin_ctzll(mine);
                mine &= mine - 1;
                const uint64_t cand = pack_entry(bcast_f(d, src), bcast_u(id, src));
                const int pos = __builtin_popcountll(ballot64(e0 < cand)) + __builtin_popcountll(ballot64(e1 < cand));
                if (pos >= k) continue;
                // places pos.. move one down the list; what falls off the end is forgotten
                const uint64_t up0 = from_lane_below(e0, e0);
                const uint64_t up1 = from_lane_below(e1, lane_value_u64(e0, 63));
                e0 = i0 > pos ? up0 : (i0 == pos ? cand : e0);
                e1 = i1 > pos ? up1 : (i1 == pos ? cand : e1);
                if (i0 >= k) e0 = ~0ull;
                if (i1 >= k) e1 = ~0ull;
                if (cnt < k) ++cnt;
                changed = true;
            }
            if (changed) {
                if (i0 < cnt) list[i0] = e0;
                if (i1 < cnt) list[i1] = e1;
                if (cnt == k) own_key = (uint32_t)(lane_value_u64(k <= 64 ? e0 : e1, (k - 1) & 63) >> 32);
                if (many && cnt >= pr) pub_key = (uint32_t)(lane_value_u64(pr <= 64 ? e0 : e1, (pr - 1) & 63) >> 32);
            }
        }
    } else {
        thr_old = s.thr[q];
        while (mine) {
            const int src = __builtin_ctzll(mine);
            mine &= mine - 1;
            const uint64_t cand = pack_entry(bcast_f(d, src), bcast_u(id, src));
            if (cnt == k && !(cand < list[k - 1])) continue;
            // entries pos..last-1 move one place down the list (the k-th falls off when full)
            const int last = cnt < k ? cnt : k - 1;
            int pos = 0;
            for (int base = 0; base < cnt; base += 64) {
                const int p = base + lane;
                const bool before = p < cnt && list[p] < cand;
                pos += __builtin_popcountll(ballot64(before));
            }
            if (last > pos) {
                for (int base = ((last - 1) >> 6) << 6; base >= ((pos >> 6) << 6); base -= 64) {
                    const int p = base + lane;
                    const bool mv = p >= pos && p < last;
                    uint64_t e = 0;
                    if (mv) e = list[p];
                    __builtin_amdgcn_wave_barrier();
                    if (mv) list[p + 1] = e;
                    __builtin_amdgcn_wave_barrier();
                }
            }
            if (lane == 0) list[pos] = cand;
            if (cnt < k) ++cnt;
            changed = true;
            __builtin_amdgcn_wave_barrier();
        }
        if (changed && cnt == k) own_key = (uint32_t)(list[k - 1] >> 32);
        if (changed && many && cnt >= pr) pub_key = (uint32_t)(list[pr - 1] >> 32);
    }
    const float own = key_dist(own_key);
    const bool lowered = own < thr_old;  // this list's k-th best is below everything known so far
    if (lowered && lane == 0) lower_threshold(&s.thr[q], own);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    if (lane == 0) {
        __hip_atomic_store(&s.lock[q], cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        // Outside the lock: adopt what the others had reached, and tell them (no answer awaited).
        if constexpr (SHARE) {
            if (!many) {
                if (seen != kKeyInf && key_dist(seen) < (lowered ? own : thr_old))
                    lower_threshold(&s.thr[q], key_dist(seen));
                if (lowered && own_key < seen)
                    (void)__hip_atomic_fetch_min(&a.gthr[gi], own_key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    if constexpr (SHARE) {
        if (many) {
            // the word of this list first (as read at the start, or what the list has just reached)
            if (lane == my_slot) {
                if (pub_key < slots_seen) {
                    slots_seen = pub_key;
                    (void)__hip_atomic_fetch_min(&a.gthr[(int64_t)gi * a.pub_slots + lane], pub_key, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            const uint32_t bound = wave_kth_smallest_bound(slots_seen, a.pub_kth);
            if (lane == 0 && bound < kKeyInf && key_dist(bound) < (lowered ? own : thr_old))
                lower_threshold(&s.thr[q], key_dist(bound));
        }
    }
    __builtin_amdgcn_s_setprio(0);
}

// What the other workgroups of the tile's queries have reached.  `ask`: lane q < TQ requests the
// shared threshold of slot q.  `adopt`: lowers the slots' own thresholds to the answers.  Callers
// ask where a batch of candidates starts, next to a memory access of their own that they wait
// for anyway, and adopt before the candidates are tested -- but only while lists are changing
// (the previous batch inserted something), so that a settled scan asks nothing.
template <int M, int TQ>
__device__ __forceinline__ uint32_t ask_shared_thresholds(const Lds<M, TQ> &s, const ScanArgs &a)
{
    const int lane = lane_id();
    uint32_t g = kKeyInf;
    if (a.pub_slots > 1) return g;  // (the exchange over many slices happens where lists change)
    if (lane < TQ) {
        const int gi = s.gidx[lane];
        if (gi >= 0) g = __hip_atomic_load(&a.gthr[gi], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return g;
}
template <int M, int TQ>
__device__ __forceinline__ void adopt_shared_thresholds(const Lds<M, TQ> &s, uint32_t g)
{
    const int lane = lane_id();
    if (lane < TQ && g != kKeyInf) lower_threshold(&s.thr[lane], key_dist(g));
}

// Inverted-file tiles start at different times: a job whose query has been served by other lists
// already starts from what those have published (ScanArgs::pub_slots) instead of +infinity.
// Wave w takes job slot w; called after the barrier that follows the per-slot state.
template <int M, int TQ>
__device__ __forceinline__ void start_from_published_bounds(const Lds<M, TQ> &s, const ScanArgs &a, int wave, int nvq)
{
    if (a.pub_slots <= 1 || wave >= nvq) return;
    const int lane = lane_id();
    const int gi = __builtin_amdgcn_readfirstlane(s.gidx[wave]);
    uint32_t v = kKeyInf;
    if (lane < a.pub_slots)
        v = __hip_atomic_load(&a.gthr[(int64_t)gi * a.pub_slots + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (ballot64(v != kKeyInf) == 0) return;  // (nothing published yet)
    const uint32_t bound = wave_kth_smallest_bound(v, a.pub_kth);
    if (lane == 0 && bound < kKeyInf) lower_threshold(&s.thr[wave], key_dist(bound));
}

// State a wave carries from one batch of candidates to the next for the exchange above.
struct SharedAsk {
    bool wanted = true;  // wave-uniform: the previous batch changed a list (or there was none yet)
};

// A batch of survivors, one per lane, whose codes have been asked for: scored when the next batch is
// taken, so that the trip to memory overlaps what the wave does in between.
template <int M>
struct Batch {
    uint32_t w[M / 4];  // the code
    uint32_t rel = 0;   // its position
    int q = 0;          // query slot
    int n = 0;          // lanes 0 .. n-1 have one (the same in every lane)
    __device__ __forceinline__ Batch()
    {
#pragma unroll
        for (int i = 0; i < M / 4; ++i) w[i] = 0u;
    }
};

// Take one survivor in each of the lanes 0 .. n-1: bit b of a mask that belongs to `rel0`.
// `slice_codes` = the codes of the tile's slice (position 0).
// MFMA_BITS: the mask comes from the matrix-core filter (see scan_mfma_kernel for its layout).
template <int M, int TQ, bool MFMA_BITS>
__device__ __forceinline__ void take_batch(Batch<M> &p, const int n, const uint32_t b, const uint32_t rel0,
                                           const uint8_t *slice_codes)
{
    p.n = n;
    if constexpr (MFMA_BITS) {  // b = 4 * (16-code group; 128 bits: 32) + row; rel0 = position | row group << kGroupShift
        p.q = (int)(4u * ((rel0 >> kGroupShift<M>) & kGroupMask<M>) + (b & 3u));
        p.rel = (rel0 & ~(kGroupMask<M> << kGroupShift<M>)) + (M == 8 ? 16u : 32u) * (b >> 2);
    } else {  // b = c * TQ + (TQ - 1 - q); rel0 = position of the lane's first code
        p.q = (int)((TQ - 1) - (b & (TQ - 1)));
        p.rel = rel0 + b / TQ;
    }
    if (n < 64 && lane_id() >= n) p.rel = 0u;  // (a position that exists)
    const uint32_t *cw = (const uint32_t *)(slice_codes + (uint64_t)p.rel * M);
    if constexpr (M == 8) {
        const uint2 v = *(const uint2 *)cw;
        p.w[0] = v.x;
        p.w[1] = v.y;
    } else {
        const uint4 v = *(const uint4 *)cw;
        p.w[0] = v.x;
        p.w[1] = v.y;
        p.w[2] = v.z;
        p.w[3] = v.w;
    }
}

// Sub-quantizers summed before a survivor may be rejected.
template <int M>
constexpr int kEarly = (M * 3) / 8;

// Score a batch and feed the survivors that beat the current threshold to the lists.  `self0 + q` =
// the position query slot q must not return (graph mode; a value no position can take otherwise).
template <int M, int TQ, bool IVF, bool SHARE>
__device__ __forceinline__ void score_batch(const Lds<M, TQ> &s, const ScanArgs &a, const Batch<M> &p,
                                            int64_t slice_begin, uint32_t self0, SharedAsk &ask)
{
    float d = __builtin_inff();
    const int q = p.q;
    const uint32_t rel = p.rel;
    const uint32_t(&w)[M / 4] = p.w;
    if constexpr (SHARE) {
        if (ask.wanted) adopt_shared_thresholds<M, TQ>(s, ask_shared_thresholds<M, TQ>(s, a));
    }
    const float thr = s.thr[q];
    {
        // The gathers are issued last sub-quantizer first and summed first sub-quantizer first:
        // LDS answers in order, so the first addition waits for all of them and the others for
        // nothing (one wait instruction instead of one per addition).
        const lds_f32 *t = s.lut + q * (M * 256);
        if constexpr (IVF) {
            float tv[M];
#pragma unroll
            for (int j = M - 1; j >= 0; --j) {
                const uint32_t byte = (w[j >> 2] >> (8 * (j & 3))) & 0xffu;
                tv[j] = t[j * 256 + byte];
            }
            float acc = tv[0];
#pragma unroll
            for (int j = 1; j < M; ++j) acc += tv[j];
            d = acc;
        } else {
            // Tables of squared distances have no negative entries, so the sum over the first
            // sub-quantizers already bounds the distance from below: once the lists are warm it
            // rejects nearly every survivor, and the other gathers are issued only if some lane
            // of the wave still needs them.  The additions keep their order (j ascending), so a
            // distance that is finished is the same float32 as without the shortcut.
            constexpr int M0 = kEarly<M>;
            float tv[M];
#pragma unroll
            for (int j = M0 - 1; j >= 0; --j) {
                const uint32_t byte = (w[j >> 2] >> (8 * (j & 3))) & 0xffu;
                tv[j] = t[j * 256 + byte];
            }
            float acc = tv[0];
#pragma unroll
            for (int j = 1; j < M0; ++j) acc += tv[j];
            if (acc <= thr) {
#pragma unroll
                for (int j = M - 1; j >= M0; --j) {
                    const uint32_t byte = (w[j >> 2] >> (8 * (j & 3))) & 0xffu;
                    tv[j] = t[j * 256 + byte];
                }
#pragma unroll
                for (int j = M0; j < M; ++j) acc += tv[j];
                d = acc;
            }
        }
    }
    bool pass = (d <= thr) & (lane_id() < p.n);
    uint32_t key = rel;    // what breaks distance ties: the position, or the stored id
    if constexpr (IVF) {
        if (pass) key = (uint32_t)a.ext_ids[slice_begin + rel];
    } else {
        pass = pass & (rel != self0 + (uint32_t)q);  // a vector is not its own neighbour
    }
    uint64_t pm = ballot64(pass);
    ask.wanted = pm != 0;
    if constexpr (!IVF) {
        if (pm) {
            if (ballot64(pass && d == thr)) {
                pass = pass && before_kth(s, a, q, d, key);
                pm = ballot64(pass);
            }
        }
    }
    while (pm) {
        const int leader = __builtin_ctzll(pm);
        const int qcur = __builtin_amdgcn_readlane(q, leader);
        const uint64_t mine = ballot64(pass && q == qcur);
        pm &= ~mine;
        insert_candidates<M, TQ, SHARE, SHARE && !IVF>(s, a, qcur, mine, d, key);
    }
}

// The survivors of one block -- `sv`, a bit per (code, query) pair in every lane -- scored a full
// wave at a time; what does not fill a wave yet waits in the wave's queue, places assigned with
// ballot + prefix popcount.  `fill`: entries waiting, < 64 between calls.
//
// Flat scans queue whole masks: lanes with bits left append (mask, position); once 64 masks wait,
// every lane takes one, scores its lowest bit and what is left of the masks is appended again.  Per
// block that is one append whatever the number of bits, where queueing bit by bit takes a turn of
// about 16 instructions per bit of the fullest lane (4 turns at 1 bit per lane).  What the queue
// cannot take of a block's masks waits in its lanes.  1M x 1M at ht = 20 106.3 -> 95.1 ms, 10M x 10k at ht
// = 24 24.6 -> 20.6 (batches scored when the next one is taken instead of waiting for their codes: 23.0 ->
// 20.6 of that).
//
// Inverted lists queue bits: a wave sees a block or two of a list, so nearly everything it queues is
// left over when its list ends (10k x 64 probes of 10M vectors 4.46 -> 4.64 ms with masks whose bits
// are spread over the lanes at the end), and a batch is scored as soon as it is taken.
template <int M, int TQ, bool IVF, bool SHARE, bool MFMA_BITS, int CAP>
__device__ __forceinline__ void score_survivors(const Lds<M, TQ> &s, const ScanArgs &a, lds_u64 *queue, int &fill,
                                                Batch<M> &batch, uint32_t sv, uint32_t rel0, const uint8_t *slice_codes,
                                                int64_t slice_begin, uint32_t self0, SharedAsk &ask)
{
    if constexpr (IVF) {
        static_assert(2 * CAP >= 127, "fewer than 64 entries wait, at most 64 come");
        lds_u32 *bits = (lds_u32 *)queue;
        while (true) {
            const uint64_t m = ballot64(sv != 0u);
            if (m == 0) return;
            if (sv != 0u) bits[fill + prefix_count(m)] = ((uint32_t)__builtin_ctz(sv) << 27) | rel0;
            sv &= sv - 1u;
            fill += __builtin_popcountll(m);
            if (fill < 64) continue;
            __builtin_amdgcn_wave_barrier();
            fill -= 64;
            const uint32_t e = bits[fill + lane_id()];
            __builtin_amdgcn_wave_barrier();
            take_batch<M, TQ, MFMA_BITS>(batch, 64, e >> 27, e & ((1u << 27) - 1u), slice_codes);
            score_batch<M, TQ, IVF, SHARE>(s, a, batch, slice_begin, self0, ask);
        }
    } else {
        uint64_t m = ballot64(sv != 0u);
        int total = fill + __builtin_popcountll(m);
        uint32_t at = (uint32_t)(fill + prefix_count(m));
        if (sv != 0u) queue[at < (uint32_t)CAP ? at : (uint32_t)CAP] = ((uint64_t)rel0 << 32) | sv;  // (CAP: nobody's place)
        fill = total;
        if (total < 64) return;
        uint32_t rest = 0u;  // the block's masks the queue had no place for
        if (__builtin_expect(total > CAP, 0)) {
            rest = at >= (uint32_t)CAP ? sv : 0u;
            fill = CAP;
        }
        auto round = [&]() {
            __builtin_amdgcn_wave_barrier();
            fill -= 64;  // the newest 64 masks go, the others stay where they are
            const uint64_t e = queue[fill + lane_id()];
            __builtin_amdgcn_wave_barrier();
            score_batch<M, TQ, IVF, SHARE>(s, a, batch, slice_begin, self0, ask);
            sv = (uint32_t)e;
            take_batch<M, TQ, MFMA_BITS>(batch, 64, (uint32_t)__builtin_ctz(sv), (uint32_t)(e >> 32), slice_codes);
            sv &= sv - 1u;
            m = ballot64(sv != 0u);
            if (sv != 0u) queue[fill + prefix_count(m)] = (e >> 32 << 32) | sv;
            fill += __builtin_popcountll(m);
            if (__builtin_expect(total > CAP, 0)) {
                m = ballot64(rest != 0u);
                total = fill + __builtin_popcountll(m);
                at = rest != 0u ? (uint32_t)(fill + prefix_count(m)) : (uint32_t)CAP;
                queue[at < (uint32_t)CAP ? at : (uint32_t)CAP] = ((uint64_t)rel0 << 32) | rest;
                rest = at >= (uint32_t)CAP ? rest : 0u;
                fill = total < CAP ? total : CAP;
            }
        };
        // The first round stands by itself: the batch it scores was asked for before the block's last
        // loads, so it waits for that batch and not for them; in a round right after another one it
        // is the youngest load, and the wait is for everything.
        round();
        while (fill >= 64) round();
    }
}
// What waits when the wave has seen its last block: the batch taken last and fewer than 64 entries
// (of masks, the bits are spread over the lanes first).
template <int M, int TQ, bool IVF, bool SHARE, bool MFMA_BITS, int CAP>
__device__ __forceinline__ void score_remaining(const Lds<M, TQ> &s, const ScanArgs &a, lds_u64 *queue, int fill,
                                                Batch<M> &batch, const uint8_t *slice_codes, int64_t slice_begin,
                                                uint32_t self0, SharedAsk &ask)
{
    __builtin_amdgcn_wave_barrier();
    const int lane = lane_id();
    lds_u32 *bits = (lds_u32 *)queue;  // entries of one bit each: (bit number, position)
    if constexpr (IVF) {
        if (fill == 0) return;
        const uint32_t e = lane < fill ? bits[lane] : 0u;
        take_batch<M, TQ, MFMA_BITS>(batch, fill, e >> 27, e & ((1u << 27) - 1u), slice_codes);
        score_batch<M, TQ, IVF, SHARE>(s, a, batch, slice_begin, self0, ask);
        return;
    }
    uint32_t sv = 0u, rel0 = 0u;
    if (lane < fill) {
        const uint64_t e = queue[lane];
        sv = (uint32_t)e;
        rel0 = (uint32_t)(e >> 32);
    }
    fill = 0;
    __builtin_amdgcn_wave_barrier();
    while (true) {
        score_batch<M, TQ, IVF, SHARE>(s, a, batch, slice_begin, self0, ask);
        while (fill < 64) {
            const uint64_t m = ballot64(sv != 0u);
            if (m == 0) break;
            if (sv != 0u) bits[fill + prefix_count(m)] = ((uint32_t)__builtin_ctz(sv) << 27) | rel0;
            sv &= sv - 1u;
            fill += __builtin_popcountll(m);
        }
        if (fill == 0) return;
        __builtin_amdgcn_wave_barrier();
        const int n = fill < 64 ? fill : 64;
        fill -= n;
        const uint32_t e = lane < n ? bits[fill + lane] : 0u;
        __builtin_amdgcn_wave_barrier();
        take_batch<M, TQ, MFMA_BITS>(batch, n, e >> 27, e & ((1u << 27) - 1u), slice_codes);
    }
}

// Inverted-file tile set-up, shared by the fused kernels: the residual tables of the tile's jobs
// put together in LDS (see ScanArgs::list_tab) and the jobs' query codes taken from them (s.qcw).
// Called by the whole workgroup (NW waves) after the per-slot state (s.gidx) is written; ends with
// a barrier.  With short lists this is 40 % of the scan, bound by instruction issue and the waits between
// barriers: whole rows per wave need no division to find their place and give their minimum from registers,
// the first rows' shares come while the vectors are staged, four coordinates a read spare sterm the bank conflicts
// of its stride.  10k queries x 64 of 4096 lists over 10M codes, ht = 24, k = 100: 7200 vector instructions a tile
// before, 6200 now; the search 4.43 -> 4.09 ms with what short lists save in scan_kernel's last turn.
template <int M, int TQ, int NW>
__device__ __forceinline__ void stage_list_tables(const Lds<M, TQ> &s, const ScanArgs &a, int tile_list, int64_t q0,
                                                  int nvq)
{
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int dsub = a.dim / M;
    // direct: the jobs' tables were built one by one by direct differences (a.lut holds them in job
    // order); nothing to put together
    const bool direct = a.list_tab == nullptr;
    // A wave takes whole rows, four entries a lane: rows wave, wave + NW, ...; up to four rows' shares are asked for
    // at once, the first ahead of everything else here.
    constexpr int kRows = TQ * M / NW, kChunk = kRows < 4 ? kRows : 4;
    static_assert(kRows * NW == TQ * M && kRows % kChunk == 0, "rows of a wave");
    f32x4 xv[kChunk], tv[kChunk];
    auto ask = [&](int u0) {
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
            const int row = wave + (u0 + u) * NW, q = row / M, j = row % M;
            xv[u] = f32x4{0.f, 0.f, 0.f, 0.f};
            tv[u] = xv[u];
            if (q < nvq) {
                const int64_t from = direct ? q0 + q : (int64_t)a.job_q[q0 + q];
                xv[u] = ((const f32x4 *)(a.lut + (from * M + j) * 256))[lane];
                if (!direct) tv[u] = ((const f32x4 *)(a.list_tab + ((int64_t)tile_list * M + j) * 256))[lane];
            }
        }
    };
    ask(0);
    if (!direct) {
        // the list's centroid and the jobs' queries staged where the tables will go (all loads of the
        // workgroup in flight together; (TQ + 1) * dim floats fit: dim <= 1024 = a quarter of one
        // job's tables at M = 8)
        PSC_LDS float *gs = (PSC_LDS float *)s.lut, *xs = gs + a.dim;
        for (int r = wave; r <= nvq; r += NW) {
            const float *from = r == 0 ? a.coarse + (int64_t)tile_list * a.dim
                                       : a.queries + (int64_t)a.job_q[q0 + r - 1] * a.dim;
            for (int t = lane; t < a.dim; t += 64) gs[r * a.dim + t] = from[t];
        }
        __syncthreads();
        if (tid < TQ * M) {  // the per-job constant || (q - g)_j ||^2, from the raw vectors
            const int q = tid / M, j = tid - q * M;
            float sterm = 0.f;
            if (q < nvq) {
                int t = j * dsub;
                if (dsub % 4 == 0) {  // (the same sums in the same order, four coordinates a read)
                    for (; t < (j + 1) * dsub; t += 4) {
                        const f32x4 d4 = *(const PSC_LDS f32x4 *)(xs + q * a.dim + t) - *(const PSC_LDS f32x4 *)(gs + t);
                        sterm = fmaf(d4.x, d4.x, sterm);
                        sterm = fmaf(d4.y, d4.y, sterm);
                        sterm = fmaf(d4.z, d4.z, sterm);
                        sterm = fmaf(d4.w, d4.w, sterm);
                    }
                }
                for (; t < (j + 1) * dsub; ++t) {
                    const float df = xs[q * a.dim + t] - gs[t];
                    sterm = fmaf(df, df, sterm);
                }
            }
            s.sterm[tid] = sterm;
        }
        __syncthreads();  // (the staged vectors are read; their place is the tables' from here on)
    }
    PSC_LDS f32x4 *dst = (PSC_LDS f32x4 *)s.lut;
#pragma unroll 1
    for (int u0 = 0; u0 < kRows; u0 += kChunk) {
        if (u0 > 0) ask(u0);
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
            const int row = wave + (u0 + u) * NW;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (row / M < nvq) v = direct ? xv[u] : (xv[u] + tv[u]) + s.sterm[row];
            dst[row * 64 + lane] = v;
            // arg-min of the row (lowest index on ties)
            float best = v.x;
            int bi = 4 * lane;
            if (v.y < best) { best = v.y; bi = 4 * lane + 1; }
            if (v.z < best) { best = v.z; bi = 4 * lane + 2; }
            if (v.w < best) { best = v.w; bi = 4 * lane + 3; }
            const uint32_t key = dist_key(best);
            const uint32_t wk = wave_min_u32(key);
            const int win = __builtin_ctzll(ballot64(key == wk));  // lower lanes hold lower indices
            const int code = __builtin_amdgcn_readlane(bi, win);
            if (lane == 0) ((PSC_LDS volatile uint8_t *)s.qcw)[row] = (uint8_t)code;
        }
    }
    __syncthreads();
}

// IVF: tiles are (inverted list, up to TQ of its jobs) instead of (query tile, slice).
// SHARE: the workgroups of one query exchange their k-th-best distance through `gthr`; worth
// it when a query is served by many workgroups (inverted lists, four slices or more).
template <int M, int TQ, int NW, bool IVF, bool SHARE>
__global__ void __launch_bounds__(NW * 64)
scan_kernel(ScanArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const Lds<M, TQ> s((PSC_LDS unsigned char *)smem, a.kpad);
    constexpr int WPC = M / 4;       // 32-bit words per code
    constexpr int CB = 32 / TQ;      // codes per lane and block: one survivor bit per (code, query)
    constexpr int NLD = CB * M / 16; // 16-byte loads per lane and block
    constexpr int CPL = 16 / M;      // codes per 16-byte load
    static_assert(CB * TQ == 32 && NLD >= 1, "tile shape");
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // flat mode: tile -> (query tile, database slice); inverted-file mode: tile -> descriptor.
    // [valid_begin, slice_end) is scanned; slice_begin (<= valid_begin) is where positions count
    // from and is a whole number of 16-byte loads into `codes`.
    int slice = 0, tile_list = 0;
    bool whole_db = false;
    int64_t q0, slice_begin, valid_begin, slice_end;
    int nvq;
    if constexpr (IVF) {
        if ((int)blockIdx.x >= *a.ntiles) return;  // the grid is an upper bound on the tile count
        const IvfTile t = a.tiles[blockIdx.x];
        tile_list = t.list;
        q0 = t.job_begin;
        nvq = t.njobs;
        valid_begin = a.list_off[t.list];
        slice_end = a.list_off[t.list + 1];
        slice_begin = valid_begin - valid_begin % CPL;
    } else {
        const FlatTile t = flat_tile(a, blockIdx.x, TQ);
        slice = t.slice;
        whole_db = t.whole;
        q0 = t.q0;
        nvq = (int)((a.nq - q0) < TQ ? (a.nq - q0) : TQ);
        if (!tile_wanted(a, q0, nvq)) return;
        slice_begin = t.slice_begin;
        valid_begin = slice_begin;
        slice_end = t.slice_end;
    }

    const bool spread = a.spread_lists != 0 && nvq == 1;  // (workgroup-uniform)
    // ---- per-slot state
    if (tid < TQ) {
        const int job = spread ? 0 : tid;
        const int gi = job < nvq ? (int)(IVF ? (int64_t)a.job_q[q0 + job] : q0 + job) : -1;
        float t0 = __builtin_inff();
        if constexpr (SHARE) {
            if (gi >= 0 && a.pub_slots == 1)
                t0 = key_dist(__hip_atomic_load(&a.gthr[gi], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        }
        s.thr[tid] = t0;
        s.lock[tid] = 0;
        s.top[tid * a.kpad + a.k - 1] = kNoEntry;
        s.gidx[tid] = gi;
        s.pslot[tid] = (IVF ? (gi >= 0 ? a.job_slot[q0 + job] : 0) : slice) % a.pub_slots;
    }
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    uint32_t qw[TQ][WPC];  // the tile's query codes, in scalar registers
    if constexpr (IVF) {
        stage_list_tables<M, TQ, NW>(s, a, tile_list, q0, nvq);
        if (tid < nvq * WPC) ((uint32_t *)a.job_qcodes)[q0 * WPC + tid] = s.qcw[tid];
        start_from_published_bounds<M, TQ>(s, a, wave, spread ? TQ : nvq);
        if (spread) {  // every slot gets the job's tables and query code
            PSC_LDS f32x4 *tab = (PSC_LDS f32x4 *)s.lut;
            for (int e = tid; e < (TQ - 1) * (M * 64); e += NW * 64) tab[M * 64 + e] = tab[e % (M * 64)];
            if (tid >= WPC && tid < TQ * WPC) s.qcw[tid] = s.qcw[tid % WPC];
            __syncthreads();
        }
#pragma unroll
        for (int q = 0; q < TQ; ++q) {
#pragma unroll
            for (int w = 0; w < WPC; ++w) qw[q][w] = __builtin_amdgcn_readfirstlane(s.qcw[q * WPC + w]);
        }
    } else {
        // ---- stage the tables
        const f32x4 *src = (const f32x4 *)(a.lut + q0 * (M * 256));
        PSC_LDS f32x4 *dst = (PSC_LDS f32x4 *)s.lut;
        const int nvec = nvq * (M * 256 / 4);
        for (int e = tid; e < TQ * (M * 256 / 4); e += NW * 64) {
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (e < nvec) v = src[e];
            else if (spread) v = src[e % (M * 256 / 4)];  // a single query: every slot gets its tables
            dst[e] = v;
        }
        // ---- query codes -> scalar registers
        const uint32_t *qc = (const uint32_t *)a.qcodes;
#pragma unroll
        for (int q = 0; q < TQ; ++q) {
            const int64_t qq = (q < nvq) ? (q0 + q) : q0;
#pragma unroll
            for (int w = 0; w < WPC; ++w)
                qw[q][w] = __builtin_amdgcn_readfirstlane(qc[qq * WPC + w]);
        }
        __syncthreads();
    }

    // bit TQ-1-q of a code's TQ-bit field <-> query slot q; only the first nvq slots are real
    uint32_t qmask = ((1u << TQ) - 1u) & ~((1u << (TQ - nvq)) - 1u);
    if (spread) qmask = 1u << (TQ - 1 - wave % TQ);  // the wave's own slot
    uint32_t qmask_all = 0u;
#pragma unroll
    for (int c = 0; c < CB; ++c) qmask_all |= qmask << (c * TQ);
    lds_u64 *queue = s.queue + wave * (kQueueCap + 1);
    Batch<M> batch;
    int fill = 0;  // wave-uniform: masks waiting in the queue
    SharedAsk ask;
    const uint8_t *slice_codes = a.codes + slice_begin * M;
    // graph mode: slot q's own vector sits at position self0 + q of the slice (if it is in there)
    uint32_t self0 = 0x80000000u;
    if (!IVF && a.skip_first >= 0) {
        const int64_t at = a.skip_first + q0 - slice_begin;
        if (at > -64 && at < kMaxSliceLen) self0 = (uint32_t)at;
    }

    const uint32_t bias = a.bias;
    const int64_t stride = (int64_t)NW * 64 * CB;
    const int64_t wave_first = slice_begin + (int64_t)wave * 64 * CB;
    const uint8_t *lane_ptr = a.codes + (wave_first + (int64_t)lane * CB) * M;  // lane's first code

    // The lane's CB consecutive codes as NLD 16-byte loads.  `whole` (wave-uniform) says the
    // wave's block lies entirely inside the slice; otherwise codes past the end read as zero
    // (their survivor bits are masked off below).
    auto load_block = [&](const uint8_t *ptr, int64_t first, bool whole, uint32_t (&w)[CB * WPC]) {
        if (whole) {
#pragma unroll
            for (int l = 0; l < NLD; ++l) {
                const uint4 v = *(const uint4 *)(ptr + l * 16);
                w[l * 4 + 0] = v.x;
                w[l * 4 + 1] = v.y;
                w[l * 4 + 2] = v.z;
                w[l * 4 + 3] = v.w;
            }
        } else {
            const int64_t p = first + (int64_t)lane * CB;
#pragma unroll
            for (int l = 0; l < NLD; ++l) {
                const int64_t pl = p + l * CPL;
                uint32_t *o = &w[l * 4];
                o[0] = o[1] = o[2] = o[3] = 0u;
                if (pl + CPL <= slice_end) {
                    const uint4 v = *(const uint4 *)(ptr + l * 16);
                    o[0] = v.x;
                    o[1] = v.y;
                    o[2] = v.z;
                    o[3] = v.w;
                } else if (CPL == 2 && pl < slice_end) {  // the last, odd 64-bit code
                    const uint2 v = *(const uint2 *)(ptr + l * 16);
                    o[0] = v.x;
                    o[1] = v.y;
                }
            }
        }
    };

    // A wave works on U of its blocks per turn of the main loop ("super-block"): all U filters run
    // back to back (pure VALU) with the U next blocks already asked for, and only then are the U
    // survivor masks queued one after the other -- so a wave waits for memory once per U blocks.
    // (Codes between slice_begin and valid_begin are readable -- they belong to the previous list
    //  -- and are masked off.)
    constexpr int U = (CB * WPC <= 4) ? 4 : (CB * WPC <= 16 ? 2 : 1);
    const int64_t sstride = stride * U;
    uint32_t cur[U][CB * WPC];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t b = wave_first + u * stride;
        if (b < slice_end) load_block(lane_ptr + u * stride * M, b, b + 64 * CB <= slice_end, cur[u]);
    }
    // One super-block of the wave, starting at code `sb` of the database.  INSIDE: this
    // super-block and the next one lie entirely inside the scanned range, so no code needs masking
    // and the next loads need no bounds -- the form all but the first and last turns take.
    auto superblock = [&](auto inside, const int64_t sb) {
        constexpr bool INSIDE = decltype(inside)::value;
        // ---- Hamming filter: bit c*TQ + (TQ-1-q) of a mask <=> code c is within ht of query q
        uint32_t svs[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t blk = sb + u * stride;
            if constexpr (!INSIDE) {
                if (blk >= slice_end) {  // (short lists: most blocks of their only turn)
                    svs[u] = 0u;
                    continue;
                }
            }
            uint32_t far = 0u;
#pragma unroll
            for (int c = CB - 1; c >= 0; --c) {
                uint32_t wc[WPC];
#pragma unroll
                for (int w = 0; w < WPC; ++w) wc[w] = cur[u][c * WPC + w];
                hamming_test_tile<TQ, WPC>(far, wc, bias, qw);
            }
            uint32_t valid = qmask_all;
            if constexpr (!INSIDE) {
                if (!(blk + 64 * CB <= slice_end && blk >= valid_begin)) {  // ragged: the lane's codes [skip, left)
                    const int left = (int)(slice_end - blk < 64 * CB ? slice_end - blk : 64 * CB) - lane * CB;
                    const int skip = (int)(valid_begin > blk ? valid_begin - blk : 0) - lane * CB;
                    if (left < CB) valid &= left > 0 ? (1u << (left * TQ)) - 1u : 0u;
                    if (skip > 0) valid &= skip < CB ? ~0u << (skip * TQ) : 0u;
                }
            }
            svs[u] = ~far & valid;
        }
        // ---- ask for the next super-block
        lane_ptr += sstride * M;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (INSIDE) {
                load_block(lane_ptr + u * stride * M, 0, true, cur[u]);
            } else {
                const int64_t b = sb + sstride + u * stride;
                if (b < slice_end) load_block(lane_ptr + u * stride * M, b, b + 64 * CB <= slice_end, cur[u]);
            }
        }
        // ---- survivors -> queue, full wavefronts -> ADC
        uint32_t rel0 = (uint32_t)(sb - slice_begin) + (uint32_t)lane * CB;
        auto queue_block = [&](uint32_t sv) {
            score_survivors<M, TQ, IVF, SHARE, false, kQueueCap>(s, a, queue, fill, batch, sv, rel0, slice_codes,
                                                                 slice_begin, self0, ask);
        };
        if constexpr (INSIDE) {  // the hot form: one copy of the queueing code per block, no loop around them
#pragma unroll
            for (int u = 0; u < U; ++u) {
                queue_block(svs[u]);
                rel0 += (uint32_t)stride;
            }
        } else {
#pragma nounroll
            for (int u = 0; u < U; ++u) {
                queue_block(svs[0]);
#pragma unroll
                for (int v = 0; v + 1 < U; ++v) svs[v] = svs[v + 1];  // the next mask moves into place
                rel0 += (uint32_t)stride;
            }
        }
    };
    int64_t sb = wave_first;
    if (sb < slice_end && valid_begin != slice_begin) {  // a list that starts inside a 16-byte load
        superblock(std::false_type{}, sb);
        sb += sstride;
    }
    // turns with two whole super-blocks ahead of sb (computed once, counted in 32 bits)
    const int64_t room = slice_end - sb - (2 * sstride - stride + 64 * CB);
    const int ninside = room >= 0 ? (int)(room / sstride) + 1 : 0;
    for (int i = 0; i < ninside; ++i, sb += sstride) superblock(std::true_type{}, sb);
    for (; sb < slice_end; sb += sstride) superblock(std::false_type{}, sb);
    score_remaining<M, TQ, IVF, SHARE, false, kQueueCap>(s, a, queue, fill, batch, slice_codes, slice_begin, self0, ask);
    __syncthreads();

    if (spread) {
        // ---- one job, TQ lists: every entry goes to its rank in their union (its place in its
        // own list plus the entries of the other lists below it), the first k ranks are the job's
        int cnt[TQ], total = 0;
#pragma unroll
        for (int t = 0; t < TQ; ++t) {
            cnt[t] = s.lock[t];
            total += cnt[t];
        }
        const int64_t o = IVF ? (int64_t)a.job_slot[q0] * a.k : (q0 * a.nslice + slice) * a.k;
        for (int e = tid; e < TQ * a.k; e += NW * 64) {
            const int t = e / a.k, p = e - t * a.k;
            int mine = 0;
#pragma unroll
            for (int u = 0; u < TQ; ++u) mine = u == t ? cnt[u] : mine;
            if (p >= mine) continue;
            const uint64_t ent = s.top[t * a.kpad + p];
            int rank = p;
#pragma unroll
            for (int u = 0; u < TQ; ++u) {
                if (u == t) continue;
                int lo = 0, hi = cnt[u];  // number of entries of list u below ent
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (s.top[u * a.kpad + mid] < ent) lo = mid + 1; else hi = mid;
                }
                rank += lo;
            }
            if (rank < a.k) {
                a.part_d[o + rank] = entry_dist(ent);
                a.part_i[o + rank] = IVF ? (int64_t)entry_id(ent) : slice_begin + (int64_t)entry_id(ent);
            }
        }
        for (int r = tid; r < a.k; r += NW * 64)
            if (r >= total) {
                a.part_d[o + r] = __builtin_inff();
                a.part_i[o + r] = (int64_t)-1;
            }
        return;
    }
    // ---- write the tile's lists (padded) to the workspace
    for (int e = tid; e < nvq * a.k; e += NW * 64) {
        const int q = e / a.k, r = e - q * a.k;
        const bool have = r < s.lock[q];
        const uint64_t ent = s.top[q * a.kpad + r];
        int64_t o, id;
        if constexpr (IVF) {
            o = (int64_t)a.job_slot[q0 + q] * a.k + r;
            id = (int64_t)entry_id(ent);
        } else {
            o = ((q0 + q) * a.nslice + slice) * a.k + r;
            id = slice_begin + (int64_t)entry_id(ent);
        }
        a.part_d[o] = have ? entry_dist(ent) : __builtin_inff();
        a.part_i[o] = have ? id : (int64_t)-1;
    }
    if constexpr (!IVF) {
        if (whole_db && a.nslice > 1) pad_unused_slices(a, q0, nvq, tid, NW * 64);
    }
}

// ---------------------------------------------------------------------------------------------
// The fused scan with the Hamming test of Section 3.3 ("dual" in Section 4.2) on the matrix cores (tiles
// of 16 queries at 64 bits, of 8 at 128; the description is for 64 bits up to the last paragraph).  With
// the code's bits c_i in {0, 1}, the query's bits turned into s_i = +1 (bit 0) or -1 (bit 1) and p the
// number of ones of the query,
//     distance = p + sum_i s_i c_i,   so   f = (ht + 64 - p) - sum_i s_i c_i = ht + 64 - distance
// lies in 0 .. 127 (ht <= 63) and its bit 6 says "within ht": a contraction whose small-integer
// operands 4-bit floating point (E2M1) holds exactly, v_mfma_scale_f32_16x16x128_f8f6f4.
//
// Bits to operands costs one vector instruction per 8 bits and no table: E2M1 reads the nibbles
// 0001, 0010, 0100 as 0.5, 1, 2, so `word & 0x11111111`, `& 0x22222222` and `& 0x44444444` are operands
// already; the query side carries 2, 1, 0.5 in the same places, every product is 0 or +-1.  The top
// bit of a nibble is the sign: `(word & 0x88888888) | 0x22222222` is 1 - 2 c, and with
// s c = s / 2 - s (1 - 2 c) / 2 it meets +-0.5 on the query side and a constant.
//
// Two pairs to a result: the instruction's K = 128 positions hold the 64 bits of two codes (lanes
// 0 .. 31 the halves of one, lanes 32 .. 63 of the other), and the per-lane block scales weigh
// their sums 2^(s+1) and 2^(s+9), s = 0 .. 7.  With 2^23 added (through the accumulator, like the
// constants) the result is a float32 in [2^23, 2^24) whose mantissa is the two fields side by side,
// exact, bits 7 + s and 15 + s being the two verdicts.  s differs between the four result registers of
// a product and between the two products of a pair, so one `(result & mask) | near` per register
// puts sixteen verdicts into bits 7 .. 22 of one word: half a vector instruction per pair and lane.
//
// Operand layout (wave64, lane l, col = l % 16, grp = l / 16): A = query slot col, B = a code of
// column col, K positions 32 grp .. 32 grp + 31; the lane receives (query slots 4 grp + r, column
// col), r = 0 .. 3.  A wave reads 64 codes with one 8-byte load per lane (lane l: code l); one
// v_permlane16_swap of the two words leaves in one register the halves of the codes of lanes 0 .. 15
// and 32 .. 47, in the other those of lanes 16 .. 31 and 48 .. 63, each half in its row of lanes.
//
// Survivor masks: bit 4 * t + r of a lane's mask <=> (code 16 * t + col of the 128-code block,
// query slot 4 * grp + r), t = 0..7.  Queue entries carry the mask, grp and the position of the
// block's code `col`.
//
// 128 bits: one product takes words 0 and 2 of its two codes (lanes read 8 bytes: row 0 of lanes the
// first half of a code, row 1 the second, rows 2 and 3 those of the code 64 on), the next, into the
// same result, words 1 and 3; no word changes lanes.  8 queries fill half of the rows, so two such
// pairs serve one result, the first with the queries in rows 0 .. 7 (the others zero), the second,
// with the next 16 codes, in rows 8 .. 15.  The fields are ht + 128 - distance, 8 bits, their bit 7 at
// 7 + s and 15 + s.  Their lowest bit is the accumulator's (2^23's) last one at s = 0, so the +-0.5 of
// the nibbles' top bits have to be added up before they meet it: a word has eight of them, whose sum is
// whole, and the hardware adds a block's products first (tested at every threshold, on pairs at the
// threshold and one beyond; 64 bits leave a bit to spare and do not depend on it).  Bit 4 * t + r of a
// mask is code 32 * t + 16 * (grp / 2) + col of a 256-code block and query slot 4 * (grp % 2) + r.
//
// What bounds it: vector instruction issue (10M x 10k, 64 bits, ht = 24: 73 % of the slots, matrix cores 10
// %, LDS 38 %), about 45 per 2048 pairs for the test (22 to make operands, the rest to collect verdicts)
// beside 4 products of 16 cycles; at 128 bits what crosses the fabric (162 GB in 25.9 ms; vector issue 50
// %, matrix cores 22 %).  Bytes of +-1 from a table in LDS and one int8 product per 16 codes (16
// look-ups, 80 vector instructions) took 134.8 ms for 1M x 1M at ht = 20 where this takes 80.3, queues
// that hold survivors bit by bit 106.3; 10M x 10k at ht = 24, k = 100 13.9 ms with the workload's data.
// ---------------------------------------------------------------------------------------------
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float mfma_f32x4 __attribute__((ext_vector_type(4)));

// (One 16-wave workgroup per compute unit = 4 waves per SIMD: telling the compiler so lets it
//  spend registers on keeping the products of a block in flight together.)
// IVF: tiles are (inverted list, up to 16 of its jobs), as in scan_kernel.
template <int M, int NW, bool SHARE, bool IVF = false>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(4, 4)))
scan_mfma_kernel(ScanArgs a)
{
    static_assert(M == 8 || !IVF, "inverted lists of 128-bit codes take scan_kernel");
    constexpr int TQ = M == 8 ? 16 : 8;
    constexpr int WPC = M / 4;                  // 32-bit words per code
    constexpr int kBlock = M == 8 ? 128 : 256;  // codes per wave and turn
    constexpr int NLD = kBlock * M / 512;       // 8-byte loads per lane and turn
    extern __shared__ __align__(16) unsigned char smem[];
    const Lds<M, TQ> s((PSC_LDS unsigned char *)smem, a.kpad);
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;

    FlatTile ft{};
    int slice = 0, tile_list = 0;
    int64_t q0, slice_begin, slice_end;
    int nvq;
    if constexpr (IVF) {
        if ((int)blockIdx.x >= *a.ntiles) return;  // the grid is an upper bound on the tile count
        const IvfTile t = a.tiles[blockIdx.x];
        tile_list = t.list;
        q0 = t.job_begin;
        nvq = t.njobs;
        slice_begin = a.list_off[t.list];  // (8-byte loads, one code each: a list may start anywhere)
        slice_end = a.list_off[t.list + 1];
    } else {
        ft = flat_tile(a, blockIdx.x, TQ);
        slice = ft.slice;
        q0 = ft.q0;
        nvq = (int)((a.nq - q0) < TQ ? (a.nq - q0) : TQ);
        if (!tile_wanted(a, q0, nvq)) return;
        slice_begin = ft.slice_begin;
        slice_end = ft.slice_end;
    }
    // the queue entries take a position in 27 bits: flag the run instead of returning something wrong
    if (slice_end - slice_begin > kMaxSliceLen) {
        if (tid == 0) atomicExch(a.status, 1);
        return;
    }

    if (tid < TQ) {
        const int gi = tid < nvq ? (int)(IVF ? (int64_t)a.job_q[q0 + tid] : q0 + tid) : -1;
        float t0 = __builtin_inff();
        if constexpr (SHARE) {
            if (gi >= 0 && a.pub_slots == 1)
                t0 = key_dist(__hip_atomic_load(&a.gthr[gi], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        }
        s.thr[tid] = t0;
        s.lock[tid] = 0;
        s.top[tid * a.kpad + a.k - 1] = kNoEntry;
        s.gidx[tid] = gi;
        s.pslot[tid] = (IVF ? (gi >= 0 ? a.job_slot[q0 + tid] : 0) : slice) % a.pub_slots;
    }
    if constexpr (IVF) {
        stage_list_tables<M, TQ, NW>(s, a, tile_list, q0, nvq);
        if (tid < nvq * 2) ((uint32_t *)a.job_qcodes)[q0 * 2 + tid] = s.qcw[tid];
        start_from_published_bounds<M, TQ>(s, a, wave, nvq);
    } else {
        typedef float f32x4 __attribute__((ext_vector_type(4)));
        const f32x4 *src = (const f32x4 *)(a.lut + q0 * (M * 256));
        PSC_LDS f32x4 *dst = (PSC_LDS f32x4 *)s.lut;
        const int nvec = nvq * (M * 256 / 4);
        for (int e = tid; e < TQ * (M * 256 / 4); e += NW * 64) {
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (e < nvec) v = src[e];
            dst[e] = v;
        }
        __syncthreads();
    }

    // A operand: one word of query slot col % TQ as signs on the magnitudes 2, 1, 0.5 (minus for a 0)
    // and 0.5 (minus for a 1: the database's fourth bits are signs, see above); slots past nvq are all
    // zero.  64 bits: word grp % 2.  128 bits: qa[h][i] holds word 2 * (grp % 2) + i, in rows
    // 8 h .. 8 h + 7, the other rows being zero.
    auto query_word = [&](int slot, int w) {
        if constexpr (IVF) return (uint32_t)s.qcw[slot * WPC + w];
        else return ((const uint32_t *)a.qcodes)[(q0 + slot) * WPC + w];
    };
    const int ht = (int)(0x7fffffffu - a.bias);
    i32x8 qa[16 / TQ][WPC / 2];
#pragma unroll
    for (int i = 0; i < WPC / 2; ++i) {
        const bool real = col % TQ < nvq;
        const uint32_t w = real ? query_word(col % TQ, (WPC / 2) * (grp & 1) + i) : 0u;
        const int v[4] = {(int)(((~w & 0x11111111u) << 3) | 0x44444444u), (int)(((~w & 0x22222222u) << 2) | 0x22222222u),
                          (int)(((~w & 0x44444444u) << 1) | 0x11111111u), (int)((w & 0x88888888u) | 0x11111111u)};
#pragma unroll
        for (int h = 0; h < 16 / TQ; ++h) {
            qa[h][i] = i32x8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < 4; ++j) qa[h][i][j] = real && col / TQ == h ? v[j] : 0;
        }
    }
    // block scales (biased exponents): the row's place s = row % 4 (+ 4 for the second product of a
    // pair, on the other operand), eight bits higher for the second code
    constexpr int kLow = M == 8 ? 1 : 0;  // place of a field's lowest bit at s = 0
    const int scale_q = 127 + kLow + (col & 3) + (grp >= 2 ? 8 : 0);
    mfma_f32x4 cinit[2];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int slot = (4 * grp + r) % TQ;
        float f = 0.f;  // (an empty slot's fields stay 0: never within ht)
        if (slot < nvq) {
            int ones = M;  // ones of the query, the sign bits' constant (M - ones among the fourth bits) with them
#pragma unroll
            for (int w = 0; w < WPC; ++w) ones += __popc(query_word(slot, w) & 0x77777777u);
            f = (float)(ht + 8 * M - ones);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int low = kLow + r + 4 * t;
            cinit[t][r] = 8388608.f + f * (float)((1 << low) + (1 << (low + 8)));
        }
    }

    lds_u64 *queue = s.queue + wave * (kMfmaQueueCap + 1);
    Batch<M> batch;
    int fill = 0;
    SharedAsk ask;
    const uint8_t *slice_codes = a.codes + slice_begin * M;
    uint32_t self0 = 0x80000000u;
    if (!IVF && a.skip_first >= 0) {
        const int64_t at = a.skip_first + q0 - slice_begin;
        if (at > -64 && at < kMaxSliceLen) self0 = (uint32_t)at;
    }
    // what a queue entry adds to the block's position: the place of the mask's first code in the block
    // and, in the bits that both leave free, the lane's group of query slots
    const uint32_t lane_code = (uint32_t)(M == 8 ? col : col + 16 * (grp >> 1));
    const uint32_t lane_bits = lane_code | (((uint32_t)grp & kGroupMask<M>) << kGroupShift<M>);
    constexpr int kStep = M == 8 ? 16 : 32;  // codes from one group of four mask bits to the next
    uint32_t m1 = 0x11111111u, m2 = 0x22222222u, m4 = 0x44444444u, m8 = 0x88888888u, ones = 0x22222222u;
    asm("" : "+s"(m1), "+s"(m2), "+s"(m4), "+s"(m8), "+v"(ones));  // (in registers: half the code size of literals)

    // The wave's blocks: wave, wave + NW, ... of the slice's 128-code blocks, positions counted from
    // the slice's start (at most 2^27).  Two register sets in turn: a block's next-but-one is asked
    // for as soon as its codes have become operands.  Past the slice's end the buffer's range check
    // answers zero (and the bits are masked below).
    const int len = (int)(slice_end - slice_begin);
    constexpr int stride = NW * kBlock;
    // (128 bits: rows 0, 1 of lanes read the halves of 16 codes, rows 2, 3 those of the 16 codes 64 on)
    const uint32_t lane_off = M == 8 ? (uint32_t)lane * 8u : (uint32_t)(64 * (grp >> 1) + col) * 16u + 8u * (grp & 1);
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void *)slice_codes, 0, (int)((uint32_t)len * (uint32_t)M), 0x00020000);
    auto load_block = [&](int blk, u32x2 (&c)[NLD]) {
        const uint32_t at = (uint32_t)blk * (uint32_t)M + lane_off;  // (below 2^31 + 2^18: blk < len + 3 * stride)
#pragma unroll
        for (int l = 0; l < NLD; ++l) {
            // 64 bits: 64 codes in a row; 128 bits: two runs of 16, l = 4 p + 2 t + h as used below
            const uint32_t first = M == 8 ? 64 * l : 128 * (l >> 2) + 16 * (l & 3);
            c[l] = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)(at + first * M), 0, 0);
        }
    };
    auto scan_block = [&](int blk, u32x2 (&c)[NLD]) {
        // (the pairs stay pairs up to here: split earlier, their halves are copied at the loop's end,
        //  which waits for the loads just issued)
#pragma unroll
        for (int l = 0; l < NLD; ++l) asm volatile("" : "+v"(c[l]));
        auto operand = [&](uint32_t w) {
            return i32x8{(int)(w & m1), (int)(w & m2), (int)(w & m4), (int)((w & m8) | ones), 0, 0, 0, 0};
        };
        i32x8 cb[2 * NLD];
#pragma unroll
        for (int l = 0; l < NLD; ++l) {
            uint32_t w0 = c[l][0], w1 = c[l][1];
            if constexpr (M == 8) {
                const auto w = __builtin_amdgcn_permlane16_swap(w0, w1, false, false);
                w0 = w[0];
                w1 = w[1];
            }
            cb[2 * l] = operand(w0);
            cb[2 * l + 1] = operand(w1);
        }
        load_block(blk + 2 * stride, c);
        mfma_f32x4 acc[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int t = i & 1, scale_t = 127 + 4 * t;
            acc[i] = cinit[t];
            if constexpr (M == 8) {
                acc[i] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(qa[0][0], cb[i], acc[i], 4, 4, 0, scale_q, 0, scale_t);
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int w = 0; w < 2; ++w)
                        acc[i] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                            qa[16 / TQ - 1 < h ? 0 : h][WPC / 2 - 1 < w ? 0 : w], cb[NLD < 8 ? 0 : 4 * i + 2 * h + w], acc[i],
                            4, 4, 0, scale_q, 0, scale_t);
                }
            }
        }
        uint32_t near[2] = {0u, 0u};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    near[h] |= __float_as_uint(acc[2 * h + t][r]) & (0x8080u << (r + 4 * t));
                    asm("" : "+v"(near[h]));  // (one and-or per register: left alone the compiler takes 1.5)
                }
            }
        }
        uint32_t sv = (near[0] >> 7) | (near[1] << 9);
        if (blk + kBlock > len) {  // ragged block: codes past the end do not count
            uint32_t in = 0u;
#pragma unroll
            for (int t = 0; t < 8; ++t)
                if (blk + kStep * t + (int)lane_code < len) in |= 0xfu << (4 * t);
            sv &= in;
        }
        score_survivors<M, TQ, IVF, SHARE, true, kMfmaQueueCap>(s, a, queue, fill, batch, sv, (uint32_t)blk + lane_bits,
                                                                slice_codes, slice_begin, self0, ask);
    };
    u32x2 even[NLD], odd[NLD];
    int blk = wave * kBlock;
    load_block(blk, even);
    __builtin_amdgcn_sched_barrier(0);  // (waits are counted: the order of the loads matters)
    load_block(blk + stride, odd);
    while (blk < len) {  // (an odd block past the end is all masked; a way out between the two would cost
                         //  the waits their exact counts)
        scan_block(blk, even);
        scan_block(blk + stride, odd);
        blk += 2 * stride;
    }
    score_remaining<M, TQ, IVF, SHARE, true, kMfmaQueueCap>(s, a, queue, fill, batch, slice_codes, slice_begin, self0, ask);
    __syncthreads();

    for (int e = tid; e < nvq * a.k; e += NW * 64) {
        const int q = e / a.k, r = e - q * a.k;
        const bool have = r < s.lock[q];
        const uint64_t ent = s.top[q * a.kpad + r];
        int64_t o, id;
        if constexpr (IVF) {
            o = (int64_t)a.job_slot[q0 + q] * a.k + r;
            id = (int64_t)entry_id(ent);
        } else {
            o = ((q0 + q) * a.nslice + slice) * a.k + r;
            id = slice_begin + (int64_t)entry_id(ent);
        }
        a.part_d[o] = have ? entry_dist(ent) : __builtin_inff();
        a.part_i[o] = have ? id : (int64_t)-1;
    }
    if constexpr (!IVF) {
        if (ft.whole && a.nslice > 1) pad_unused_slices(a, q0, nvq, tid, NW * 64);
    }
}

// ---------------------------------------------------------------------------------------------
// Pure ADC scan: ht >= 8m keeps every code (Section 4.2 "ADC", the PQ baseline of the paper), so
// there is nothing to filter or to queue: every (query, code) pair is scored.  The bound is the
// LDS gather rate, so the TQ tables are interleaved in LDS four queries to an entry,
// lut4[g][j][c] = (T_{4g}[j][c], .., T_{4g+3}[j][c]): one 16-byte read serves four queries of
// the tile, and a code's m byte offsets are computed once for all TQ queries.
// Same tiling (query tile x database slice), lists, ordering and outputs as scan_kernel.
// FILTER: the Hamming test of Section 3.3 is still applied -- to the pairs whose distance beats the
// current k-th best, which are few; since that k-th best is taken among pairs that pass the test,
// the outcome is the one of testing every pair first.  This is the cheaper route when the
// threshold lets a large share of the codes through: scoring everything from the interleaved
// tables then costs less than queueing the survivors one by one.
// ---------------------------------------------------------------------------------------------
template <int M, int TQ, int NW, bool SHARE, bool FILTER>
__global__ void __launch_bounds__(NW * 64)
adc_kernel(ScanArgs a)
{
    static_assert(TQ % 4 == 0, "four queries per table entry");
    extern __shared__ __align__(16) unsigned char smem[];
    const Lds<M, TQ> s((PSC_LDS unsigned char *)smem, a.kpad);
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int G = TQ / 4;
    constexpr int WPC = M / 4;
    constexpr int CPL = 16 / M;  // codes per 16-byte load
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    const FlatTile ft = flat_tile(a, blockIdx.x, TQ);
    const int slice = ft.slice;
    const int64_t q0 = ft.q0;
    const int nvq = (int)((a.nq - q0) < TQ ? (a.nq - q0) : TQ);
    if (!tile_wanted(a, q0, nvq)) return;
    const int64_t slice_begin = ft.slice_begin;
    const int64_t slice_end = ft.slice_end;

    // ---- stage the tables interleaved, reset the lists
    {
        const float *src = a.lut + q0 * (M * 256);
        PSC_LDS float *dst = (PSC_LDS float *)s.lut;
        for (int e = tid; e < TQ * M * 256; e += NW * 64) {
            const int q = e / (M * 256), r = e - q * (M * 256);
            dst[(((q >> 2) * (M * 256) + r) << 2) + (q & 3)] = q < nvq ? src[e] : 0.f;
        }
        if (tid < TQ) {
            float t0 = __builtin_inff();
            if constexpr (SHARE) {
                if (tid < nvq && a.pub_slots == 1)
                    t0 = key_dist(__hip_atomic_load(&a.gthr[q0 + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            }
            s.thr[tid] = t0;
            s.lock[tid] = 0;
            s.top[tid * a.kpad + a.k - 1] = kNoEntry;
            s.gidx[tid] = tid < nvq ? (int)(q0 + tid) : -1;
            s.pslot[tid] = slice % a.pub_slots;
        }
    }
    // ---- query codes -> scalar registers (only the filtering variant reads them)
    uint32_t qw[TQ][WPC];
    if constexpr (FILTER) {
        const uint32_t *qc = (const uint32_t *)a.qcodes;
#pragma unroll
        for (int q = 0; q < TQ; ++q) {
            const int64_t qq = (q < nvq) ? (q0 + q) : q0;
#pragma unroll
            for (int w = 0; w < WPC; ++w) qw[q][w] = __builtin_amdgcn_readfirstlane(qc[qq * WPC + w]);
        }
    }
    __syncthreads();

    const PSC_LDS f32x4 *lut4 = (const PSC_LDS f32x4 *)s.lut;
    SharedAsk ask;
    const int64_t stride = (int64_t)NW * 64 * CPL;
    const int64_t skip_rel = a.skip_first + q0 - slice_begin;
    const bool skipping = a.skip_first >= 0 && skip_rel > -(int64_t)TQ && skip_rel < kMaxSliceLen;
    for (int64_t blk = slice_begin + (int64_t)wave * 64 * CPL; blk < slice_end; blk += stride) {
        const int64_t p0 = blk + (int64_t)lane * CPL;
        uint32_t shared = kKeyInf;
        const bool asking = SHARE && ask.wanted;
        if (asking) shared = ask_shared_thresholds<M, TQ>(s, a);
        ask.wanted = false;
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        if (p0 + CPL <= slice_end) {
            const uint4 v = *(const uint4 *)(a.codes + p0 * M);
            w[0] = v.x;
            w[1] = v.y;
            w[2] = v.z;
            w[3] = v.w;
        } else if (CPL == 2 && p0 < slice_end) {
            const uint2 v = *(const uint2 *)(a.codes + p0 * M);
            w[0] = v.x;
            w[1] = v.y;
        }
        if (asking) adopt_shared_thresholds<M, TQ>(s, shared);
        // thresholds of the tile, refreshed once per block: lane q holds thr[q]
        const float thr_v = s.thr[lane & (TQ - 1)];
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const bool live = p0 + c < slice_end;
            const uint32_t rel = (uint32_t)(p0 + c - slice_begin);
            uint32_t off[M];  // the code's byte for sub-quantizer j = its entry in sub-table j
#pragma unroll
            for (int j = 0; j < M; ++j) off[j] = ((w[c * WPC + (j >> 2)] >> (8 * (j & 3))) & 0xffu);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                f32x4 acc = lut4[(g * M + 0) * 256 + off[0]];
#pragma unroll
                for (int j = 1; j < M; ++j) acc += lut4[(g * M + j) * 256 + off[j]];
                float d[4] = {acc.x, acc.y, acc.z, acc.w};
                uint64_t any = 0;
                bool pass[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int q = g * 4 + i;
                    const float thr = bcast_f(thr_v, q);
                    pass[i] = live && q < nvq && d[i] <= thr;
                    if (skipping) pass[i] = pass[i] && rel != (uint32_t)((int32_t)skip_rel + q);
                    any |= ballot64(pass[i]);
                }
                if (any) {
                    // FILTER: the Hamming test is taken only here, on the few pairs whose distance
                    // beats the threshold (which is the k-th best among the pairs that pass the test:
                    // the result is that of testing every pair), not on every pair of the stream.
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if constexpr (FILTER) {  // bias + h overflows into the sign bit iff h > ht
                            const int q = g * 4 + i;
                            uint32_t acc = a.bias;
#pragma unroll
                            for (int ww = 0; ww < WPC; ++ww) acc += (uint32_t)__popc(w[c * WPC + ww] ^ qw[q][ww]);
                            pass[i] = pass[i] && (int32_t)acc >= 0;
                        }
                        uint64_t mine = ballot64(pass[i]);
                        if (mine) {
                            ask.wanted = true;
                            if (ballot64(pass[i] && d[i] == bcast_f(thr_v, g * 4 + i)))
                                mine = ballot64(pass[i] && before_kth(s, a, g * 4 + i, d[i], rel));
                        }
                        if (mine) {
                            insert_candidates<M, TQ, SHARE, SHARE>(s, a, g * 4 + i, mine, d[i], rel);
                        }
                    }
                }
            }
        }
    }
    __syncthreads();

    for (int e = tid; e < nvq * a.k; e += NW * 64) {
        const int q = e / a.k, r = e - q * a.k;
        const bool have = r < s.lock[q];
        const uint64_t ent = s.top[q * a.kpad + r];
        const int64_t o = ((q0 + q) * a.nslice + slice) * a.k + r;
        a.part_d[o] = have ? entry_dist(ent) : __builtin_inff();
        a.part_i[o] = have ? (slice_begin + (int64_t)entry_id(ent)) : (int64_t)-1;
    }
    if (ft.whole && a.nslice > 1) pad_unused_slices(a, q0, nvq, tid, NW * 64);
}

// ---------------------------------------------------------------------------------------------
// Small scans: one workgroup of 16 waves per (query, database slice).  What such a scan waits for in
// the tiled kernels above is not the filter but the lists: with every threshold still at infinity
// each survivor is an insertion under a lock, one after the other (100 queries x 100k codes, k = 10:
// 74 us in scan_mfma_kernel for 6 us of filtering), besides 8 to 16 tables to stage per workgroup.
// Here the survivors' (distance, id) keys are appended to a pool in LDS as they come; only when it
// is full, and once at the end, are the k smallest selected, by a radix search over the bits in
// which the keys differ (keys are distinct, ids being so).  One slice per query needs no merge and nothing set
// up; the slices of a query (`arrived`: a word per query, kPresetWord before) are put together by the one of its
// workgroups that ends last: 1 query x 100k codes 31 -> 22 us, 100 x 100k 49 -> 35 (with the tables' arg-min
// taken where the tables are built), where the merge was a launch of its own.
// A wave whose keys find no place waits in `meet`; every wave comes there sooner or later, full
// pool or no codes left, and the selection makes room and lowers the bound.
// DENSE: every code is scored and the Hamming test is taken on those below the bound (pure ADC and
// permissive thresholds), instead of queueing the codes that pass the test.
// `open`: the largest distance that is listed while there are fewer than k.
// MARKED: the queries are those that a search by bounds has marked, if they are few, each by itself and in slices; they
// are marked no more then.  The words and the status of the scan that answers more of them are set on the way.  (Marks are
// scattered: a tile of up to 16 queries that has one takes the whole database for it.  10k queries x 10M codes with some
// 220 marks 16.0 ms so, 12.3 with their tables gathered for tiles of marked queries only, 11.4 this way.)
// ---------------------------------------------------------------------------------------------
constexpr int kSmallPool = 4096;   // keys
constexpr int kRankedKeys = 512;   // of that many every key's rank is taken sooner than a search among them ends
constexpr int kSmallCodes = 8;     // codes per lane and turn
constexpr int kSmallQueue = 128;   // (mask, position) entries per wave: fewer than 64 wait, 64 come at a time

template <int M>
struct SmallLds {
    float lut[M * 256];
    uint64_t pool[kSmallPool];
    uint64_t queue[16][kSmallQueue];
    uint64_t lo[16], hi[16];
    uint32_t hist[256];
    uint32_t count, stuck, kept, bin, below;
    float bound;
};

template <int M, bool DENSE, bool MARKED>
__global__ void __launch_bounds__(1024)
scan_pool_kernel(ScanArgs a, float open, int *status, uint32_t *arrived, int64_t *__restrict__ ids,
                 float *__restrict__ dists, MarkedQueries marked, int64_t nwords)
{
    extern __shared__ __align__(16) unsigned char smem[];
    PSC_LDS SmallLds<M> &s = *(PSC_LDS SmallLds<M> *)smem;
    constexpr int WPC = M / 4;
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t words __attribute__((ext_vector_type(WPC)));
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t item = blockIdx.x / a.nslice;  // the query, or its place among the marked ones
    const int slice = (int)(blockIdx.x % a.nslice);
    const int64_t begin = (int64_t)slice * a.slice_len;
    const int64_t end = begin + a.slice_len < a.n ? begin + a.slice_len : a.n;
    const int len = (int)(end - begin);
    const uint8_t *codes = a.codes + begin * M;
    const int k = a.k;
    if (blockIdx.x == 0 && tid == 0 && status) *status = 0;
    int64_t q = item;
    if constexpr (MARKED) {
        for (int64_t e = (int64_t)blockIdx.x * 1024 + tid; e < nwords; e += (int64_t)gridDim.x * 1024) a.gthr[e] = kKeyInf;
        const uint32_t count = *marked.count;
        if (count > (uint32_t)marked.few || item >= (int64_t)count) return;  // (uniform)
        q = __builtin_amdgcn_readfirstlane(marked.which[item]);
        if (slice == 0 && tid == 0) marked.redo[q] = 0u;
    } else {
        if (a.redo != nullptr && a.redo[q] == 0u) return;  // (uniform)
    }

    // codes of the wave's turn `blk`: code blk + 64 l + lane in c[l]; past the end the range check
    // answers zero
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)codes, 0, len * M, 0x00020000);
    constexpr int kStride = 16 * 64 * kSmallCodes;
    auto load = [&](int blk, words (&c)[kSmallCodes]) {
        const uint32_t at = (uint32_t)(blk + lane) * (uint32_t)M;  // (below 2^31: the planner's slices hold at most 2^24 codes)
#pragma unroll
        for (int l = 0; l < kSmallCodes; ++l) {
            if constexpr (M == 8) c[l] = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)(at + 64u * M * l), 0, 0);
            else c[l] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(at + 64u * M * l), 0, 0);
        }
    };
    words cur[kSmallCodes];
    int blk = wave * 64 * kSmallCodes;
    load(blk, cur);
    for (int e = tid; e < M * 64; e += 1024) ((PSC_LDS f32x4 *)s.lut)[e] = ((const f32x4 *)(a.lut + q * (M * 256)))[e];
    uint32_t qw[WPC];
#pragma unroll
    for (int w = 0; w < WPC; ++w) qw[w] = __builtin_amdgcn_readfirstlane(((const uint32_t *)a.qcodes)[q * WPC + w]);
    if (tid == 0) {
        s.count = 0u;
        s.stuck = 0u;
    }
    __syncthreads();
    float bound = open;  // (the same in every lane of the workgroup)

    // The k smallest of the pool's n keys to its front, in any order; n > k.  By the whole workgroup.
    auto select = [&](int n) {
        uint64_t e[kSmallPool / 1024], lo = ~0ull, hi = 0ull;
#pragma unroll
        for (int i = 0; i < kSmallPool / 1024; ++i) {
            const int p = tid + 1024 * i;
            e[i] = p < n ? s.pool[p] : ~0ull;
            if (p < n) {
                lo = e[i] < lo ? e[i] : lo;
                hi = e[i] > hi ? e[i] : hi;
            }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const uint64_t l2 = __shfl_xor(lo, off, 64), h2 = __shfl_xor(hi, off, 64);
            lo = l2 < lo ? l2 : lo;
            hi = h2 > hi ? h2 : hi;
        }
        if (lane == 0) {
            s.lo[wave] = lo;
            s.hi[wave] = hi;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            lo = s.lo[w] < lo ? s.lo[w] : lo;
            hi = s.hi[w] > hi ? s.hi[w] : hi;
        }
        // (n > k >= 1 distinct keys: lo != hi) the bits from `shift` on are searched next, those from
        // shift + width on are `prefix`
        const int top = 64 - __builtin_clzll(lo ^ hi);
        int width = top < 8 ? top : 8, shift = top - width;
        uint64_t prefix = top == 64 ? 0ull : lo >> top;
        uint32_t need = (uint32_t)k;
        uint64_t last;
        while (true) {
            if (tid < 256) s.hist[tid] = 0u;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kSmallPool / 1024; ++i) {
                const uint64_t d = e[i] >> shift;
                const bool in = tid + 1024 * i < n && (shift + width == 64 ? 0ull : d >> width) == prefix;
                if (in) __hip_atomic_fetch_add(&s.hist[(uint32_t)d & ((1u << width) - 1u)], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
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
                            s.bin = 4u * lane + i;
                            s.below = cum;
                        }
                        cum += h[i];
                    }
                }
            }
            __syncthreads();
            const uint32_t bin = s.bin, inside = s.hist[bin];
            need -= s.below;
            prefix = (prefix << width) | bin;
            if (inside == need || shift == 0) {
                last = ((prefix + 1) << shift) - 1;  // (prefix + 1 wraps to 0 only with every bit set: last = ~0)
                break;
            }
            width = shift < 8 ? shift : 8;
            shift -= width;
            __syncthreads();  // (the histogram is read)
        }
        if (tid == 0) s.kept = 0u;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kSmallPool / 1024; ++i) {
            const bool keep = tid + 1024 * i < n && e[i] <= last;
            const uint64_t m = ballot64(keep);
            uint32_t base = 0u;
            if (lane == 0 && m) base = __hip_atomic_fetch_add(&s.kept, (uint32_t)__builtin_popcountll(m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
            if (keep) s.pool[base + prefix_count(m)] = e[i];
        }
        // the k-th best distance: (the largest key kept has the bits of `last` above the ones not searched)
        uint64_t mx = 0ull;
#pragma unroll
        for (int i = 0; i < kSmallPool / 1024; ++i)
            if (tid + 1024 * i < n && e[i] <= last) mx = e[i] > mx ? e[i] : mx;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const uint64_t o = __shfl_xor(mx, off, 64);
            mx = o > mx ? o : mx;
        }
        if (lane == 0) s.hi[wave] = mx;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < 16; ++w) mx = s.hi[w] > mx ? s.hi[w] : mx;
        bound = entry_dist(mx);
    };
    // Where waves wait for one another: with keys that found no place (stuck) or without codes left.
    // True when no wave is stuck (then all are done); otherwise there is room again.
    auto meet = [&](bool stuck) {
        if (stuck && lane == 0) __hip_atomic_fetch_add(&s.stuck, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __syncthreads();
        const bool done = s.stuck == 0u;
        if (!done) {
            select(kSmallPool);  // (a wave is stuck: the pool is full; k <= 1024 < kSmallPool)
            if (tid == 0) {
                s.count = (uint32_t)k;
                s.stuck = 0u;
            }
            __syncthreads();
        }
        return done;
    };
    // Append the lanes' keys that are still below the bound.
    auto append = [&](bool pass, float d, uint32_t pos) {
        const uint64_t key = pack_entry(d, pos);
        while (true) {
            pass = pass & (d <= bound);
            const uint64_t m = ballot64(pass);
            if (m == 0) return;
            const int n = __builtin_popcountll(m);
            uint32_t base = 0u;
            if (lane == 0) base = __hip_atomic_fetch_add(&s.count, (uint32_t)n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
            const uint32_t at = base + (uint32_t)prefix_count(m);
            if (pass && at < (uint32_t)kSmallPool) {
                s.pool[at] = key;
                pass = false;
            }
            if (base + (uint32_t)n <= (uint32_t)kSmallPool) return;
            meet(true);
        }
    };
    // (a sum that is not a number after kEarly sub-quantizers: at infinity in the fused form, as
    //  score_batch has it; one that comes to be so later, and any in the dense form, passes nowhere)
    auto score = [&](const words &c) {
        float d = s.lut[c[0] & 0xffu];
        bool number = true;
#pragma unroll
        for (int j = 1; j < M; ++j) {
            d += s.lut[j * 256 + ((c[j >> 2] >> (8 * (j & 3))) & 0xffu)];
            if (j == kEarly<M> - 1) number = d == d;
        }
        return DENSE || number ? d : __builtin_inff();
    };

    PSC_LDS uint64_t *queue = s.queue[wave];
    int fill = 0;
    auto score_queued = [&](int n) {  // the newest n entries, one survivor of each; what is left of them goes back
        __builtin_amdgcn_wave_barrier();
        fill -= n;
        const uint64_t e = lane < n ? queue[fill + lane] : 0ull;
        __builtin_amdgcn_wave_barrier();
        uint32_t sv = (uint32_t)e;
        const uint32_t pos = lane < n ? (uint32_t)(e >> 32) + 64u * (uint32_t)__builtin_ctz(sv | 0x80000000u) : 0u;
        const words c = *(const words *)(codes + (uint64_t)pos * M);
        sv &= sv - 1u;
        const uint64_t m = ballot64(sv != 0u);
        if (sv != 0u) queue[fill + prefix_count(m)] = (e >> 32 << 32) | sv;
        fill += __builtin_popcountll(m);
        append(lane < n, score(c), pos);
    };
    while (blk < len) {
        words c[kSmallCodes];
#pragma unroll
        for (int l = 0; l < kSmallCodes; ++l) c[l] = cur[l];
        load(blk + kStride, cur);
        if constexpr (DENSE) {
#pragma unroll
            for (int l = 0; l < kSmallCodes; ++l) {
                const int pos = blk + 64 * l + lane;
                const float d = score(c[l]);
                bool pass = (pos < len) & (d <= bound);
                if (ballot64(pass)) {
                    uint32_t h = a.bias;
#pragma unroll
                    for (int w = 0; w < WPC; ++w) h += (uint32_t)__popc(c[l][w] ^ qw[w]);
                    append(pass & ((int32_t)h >= 0), d, (uint32_t)pos);
                }
            }
        } else {
            uint32_t sv = 0u;
#pragma unroll
            for (int l = 0; l < kSmallCodes; ++l) {
                uint32_t h = a.bias;
#pragma unroll
                for (int w = 0; w < WPC; ++w) h += (uint32_t)__popc(c[l][w] ^ qw[w]);
                sv |= ((int32_t)h >= 0 && blk + 64 * l + lane < len) ? 1u << l : 0u;
            }
            const uint64_t m = ballot64(sv != 0u);
            if (sv != 0u) queue[fill + prefix_count(m)] = ((uint64_t)(uint32_t)(blk + lane) << 32) | sv;
            fill += __builtin_popcountll(m);
            while (fill >= 64) score_queued(64);
        }
        blk += kStride;
    }
    if constexpr (!DENSE) {
        while (fill > 0) score_queued(fill < 64 ? fill : 64);
    }
    while (!meet(false)) {}
    int n = (int)s.count;
    if (n > k) {
        __syncthreads();
        select(n);
        n = k;
    }
    __syncthreads();
    if (arrived != nullptr) {
        // several slices, put together by the workgroup of the query that comes last: each leaves its keys where
        // every XCD sees them, counts itself, and all but the last are done
        const int total = a.nslice * k;  // (<= kSmallPool, the launcher sees to it)
        float *pd = a.part_d + item * total;
        int64_t *pi = a.part_i + item * total;
        if (tid < k) {
            const uint64_t key = tid < n ? s.pool[tid] : 0ull;
            __hip_atomic_store(pd + slice * k + tid, tid < n ? entry_dist(key) : 0.f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(pi + slice * k + tid, tid < n ? begin + (int64_t)entry_id(key) : (int64_t)-1, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
        // (Each wave waits until its stores are acknowledged, the barrier orders them before thread 0's count, and
        //  that releases them; the last workgroup acquires the others'.  One release per workgroup and one acquire
        //  per query (up to 512 keys still searched): 1 query x 100k codes 27.4 us and 27.1 with a relaxed count alone,
        //  100 x 100k 42.2 and 42.2;
        //  fences from each of the 16 waves 82 us, an acquire by every workgroup up to 2 us more than this.)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) {
            const uint32_t before = __hip_atomic_fetch_add(arrived + item, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            if (before == kPresetWord + (uint32_t)a.nslice - 1u) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            s.stuck = before;
            s.count = 0u;
        }
        __syncthreads();
        if (s.stuck != kPresetWord + (uint32_t)a.nslice - 1u) return;
        for (int e0 = 0; e0 < total; e0 += 1024) {
            const int e = e0 + tid;
            const int64_t id = e < total ? __hip_atomic_load(pi + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : (int64_t)-1;
            const float d = e < total ? __hip_atomic_load(pd + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.f;
            const uint64_t m = ballot64(id >= 0);
            uint32_t base = 0u;
            if (lane == 0 && m) base = __hip_atomic_fetch_add(&s.count, (uint32_t)__builtin_popcountll(m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
            if (id >= 0) s.pool[base + prefix_count(m)] = pack_entry(d, (uint32_t)id);
        }
        __syncthreads();
        n = (int)s.count;
        if (n > kRankedKeys && n > k) {  // (otherwise the ranks below decide)
            select(n);
            n = k;
        }
        __syncthreads();
    }
    // every key to its rank among the n kept (at most 1024: a key per thread)
    const bool final = arrived != nullptr || a.nslice == 1;
    const int64_t o = (final ? q : q * a.nslice + slice) * k, first = arrived != nullptr ? 0 : begin;
    float *od = final ? dists : a.part_d;
    int64_t *oi = final ? ids : a.part_i;
    if (tid < n) {
        const uint64_t key = s.pool[tid];
        int rank = 0;
        for (int j = 0; j < n; ++j) rank += s.pool[j] < key ? 1 : 0;
        if (rank < k) {
            od[o + rank] = entry_dist(key);
            oi[o + rank] = first + (int64_t)entry_id(key);
        }
    } else if (tid < k) {
        od[o + tid] = __builtin_inff();
        oi[o + tid] = (int64_t)-1;
    }
}

// Merge the nslice sorted partial lists of each query into the final k (one wave per query).
// Lane l owns lists l, l + 64, ...: it keeps the head of each in registers together with the
// entry after it, so that a step of the merge (pick the smallest head of the wave, advance that
// list) waits for memory only when one list wins several times in a row.  Padding entries
// (id < 0) end a list.
template <int OWN>
__global__ void __launch_bounds__(64)
merge_kernel(const float *__restrict__ part_d, const int64_t *__restrict__ part_i, int nslice, int k,
             int64_t id_base, const int *__restrict__ status, const uint32_t *__restrict__ redo,
             int64_t *__restrict__ ids, float *__restrict__ dists)
{
    const int64_t q = blockIdx.x;
    if (redo != nullptr && redo[q] == 0u) return;  // (ScanArgs::redo)
    const int lane = lane_id();
    const float *pd = part_d + q * nslice * k;
    const int64_t *pi = part_i + q * nslice * k;
    const bool poisoned = *status != 0;
    uint32_t hk[OWN], nk[OWN];  // distance keys of the head and of the entry after it (kKeyNone: none)
    int64_t hi[OWN], ni[OWN];   // their ids
    int pos[OWN];               // index of the head in its list
    constexpr uint32_t kKeyNone = 0xffffffffu;  // above every real key, +infinity included
    auto fetch = [&](int l, int at, uint32_t &key, int64_t &id) {
        key = kKeyNone;
        id = -1;
        if (l < nslice && at < k) {
            const int64_t i = pi[(int64_t)l * k + at];
            if (i >= 0) {
                id = i;
                key = dist_key(pd[(int64_t)l * k + at]);
            }
        }
    };
#pragma unroll
    for (int t = 0; t < OWN; ++t) {
        pos[t] = 0;
        fetch(lane + 64 * t, 0, hk[t], hi[t]);
        fetch(lane + 64 * t, 1, nk[t], ni[t]);
    }
    for (int r = 0; r < k; ++r) {
        // the lane's best head
        uint32_t bk = hk[0];
        int64_t bi = hi[0];
        int bt = 0;
#pragma unroll
        for (int t = 1; t < OWN; ++t) {
            if (hk[t] < bk || (hk[t] == bk && hk[t] != kKeyNone && hi[t] < bi)) {
                bk = hk[t];
                bi = hi[t];
                bt = t;
            }
        }
        // the wave's: smallest key, and the lowest id among the lanes that hold it
        const uint32_t wk = wave_min_u32(bk);
        uint64_t tied = ballot64(bk == wk);
        int win = __builtin_ctzll(tied);
        if (wk != kKeyNone && (tied & (tied - 1))) {
            int64_t best = INT64_MAX;
            while (tied) {
                const int l = __builtin_ctzll(tied);
                tied &= tied - 1;
                const int64_t cand = ((int64_t)__builtin_amdgcn_readlane((int)(bi >> 32), l) << 32) |
                                     (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)bi, l);
                if (cand < best) {
                    best = cand;
                    win = l;
                }
            }
        }
        const bool have = wk != kKeyNone;
        const int64_t wi = ((int64_t)__builtin_amdgcn_readlane((int)(bi >> 32), win) << 32) |
                           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)bi, win);
        if (lane == 0) {
            ids[q * k + r] = poisoned ? (int64_t)-2 : (have ? wi + id_base : (int64_t)-1);
            dists[q * k + r] = have ? key_dist(wk) : __builtin_inff();
        }
        if (have && lane == win) {  // advance the winning list
#pragma unroll
            for (int t = 0; t < OWN; ++t) {
                if (t == bt) {
                    hk[t] = nk[t];
                    hi[t] = ni[t];
                    ++pos[t];
                    fetch(lane + 64 * t, pos[t] + 1, nk[t], ni[t]);
                }
            }
        }
    }
}

// The same merge for a handful of queries, where the hundred dependent steps of the wave above are
// all there is to wait for: a workgroup of 16 waves per query selects the k smallest
// (distance, id) pairs of all partial lists at once.  Thread t holds the distance keys of
// entries t, t + 1024, ... of the query's lists; the k-th smallest key is found bit by bit with
// one workgroup-wide count per bit (per-wave sums through LDS, two buffers in turn so that one
// barrier per bit is enough); if more entries than needed share it, the same search over the bits
// of the id finds the last id that belongs.  The selected entries go to LDS in any order and each
// is written to its rank.
constexpr int64_t kMergeSelectQueries = 32;      // up to this many queries,
constexpr int64_t kMergeSelectManyQueries = 512; // or this many if each has 32 lists or more (probed lists:
                                                 // 10k queries x 64 probes of 100M vectors, whole search, with the
                                                 // wave above / with this kernel: 64 queries 0.45 / 0.34 ms,
                                                 // 256: 0.61 / 0.57, 512: 0.84 / 0.81, 1024: 1.31 / 1.32)
constexpr int64_t kMergeSelectEntries = 32768;   // and this many entries per query
// (its forty-odd counting steps take about 20 us whatever k is; the wave above takes 0.4 us per
//  result: measured 32 against 42 us at k = 100, 20 against 5 us at k = 10)
constexpr int kMergeSelectMinK = 64;

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

template <int KPL>
__global__ void __launch_bounds__(1024)
merge_select_kernel(const float *__restrict__ part_d, const int64_t *__restrict__ part_i, int nslice, int k,
                    bool infinite, const int *__restrict__ status, const uint32_t *__restrict__ redo,
                    int64_t *__restrict__ ids, float *__restrict__ dists)
{
    if (redo != nullptr && redo[blockIdx.x] == 0u) return;  // (ScanArgs::redo)
    __shared__ uint32_t part[2][16];
    __shared__ __align__(16) uint32_t selk[1024];
    __shared__ int64_t seli[1024];
    __shared__ uint32_t nsel;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t q = blockIdx.x;
    // Rank of (key, id) among the n selected entries in LDS: keys are compared four to a read; the
    // ids are looked at only by a thread whose key occurs more than once.
    auto rank_among = [&](uint32_t key, int64_t id, int n) {
        int lt = 0, eq = 0;
        const int n4 = n & ~3;
        for (int j = 0; j < n4; j += 4) {
            const uint4 v = *(const uint4 *)&selk[j];
            lt += (v.x < key ? 1 : 0) + (v.y < key ? 1 : 0) + (v.z < key ? 1 : 0) + (v.w < key ? 1 : 0);
            eq += (v.x == key ? 1 : 0) + (v.y == key ? 1 : 0) + (v.z == key ? 1 : 0) + (v.w == key ? 1 : 0);
        }
        for (int j = n4; j < n; ++j) {
            lt += selk[j] < key ? 1 : 0;
            eq += selk[j] == key ? 1 : 0;
        }
        if (eq > 1)
            for (int j = 0; j < n; ++j) lt += (selk[j] == key && seli[j] < id) ? 1 : 0;
        return lt;
    };
    const int total = nslice * k;
    const float *pd = part_d + q * total;
    const int64_t *pi = part_i + q * total;
    const bool poisoned = *status != 0;
    constexpr uint32_t kNone = 0xffffffffu;  // padding and places past the end; real keys stay below
    // (Places a list does not fill hold distance +infinity, which no scored code has unless `infinite`:
    //  the distances alone tell them apart, so all loads of a thread are independent of one another and
    //  in flight together -- one trip to memory instead of one per entry.)
    uint32_t dk[KPL];
    {
        float dv[KPL];
#pragma unroll
        for (int i = 0; i < KPL; ++i) {
            const int e = i * 1024 + tid;
            dv[i] = pd[e < total ? e : total - 1];
        }
#pragma unroll
        for (int i = 0; i < KPL; ++i) {
            const int e = i * 1024 + tid;
            const bool real = e < total && (dv[i] != __builtin_inff() || (infinite && pi[e] >= 0));
            dk[i] = real ? min(dist_key(dv[i]), kNone - 1u) : kNone;
        }
    }
    if (tid == 0) nsel = 0u;
    int turn = 0;
    // number of the workgroup's entries for which pred(i) holds (a second predicate is counted in
    // the high half of the word)
    auto count = [&](auto pred, auto... more) {
        uint32_t cnt = 0;
#pragma unroll
        for (int i = 0; i < KPL; ++i) {
            cnt += pred(i) ? 1u : 0u;
            ((cnt += more(i) ? 0x10000u : 0u), ...);
        }
        cnt = wave_sum_u32(cnt);
        if (lane == 0) part[turn][wave] = cnt;
        __syncthreads();
        uint32_t all = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) all += part[turn][w];
        turn ^= 1;
        return all;
    };
    // A bound on the k-th smallest key from single rows of the (sorted) lists: if t lists have their
    // r-th entry at or below v, at least t (r + 1) entries lie at or below v, so for any t <= nslice
    // the t-th smallest key of row ceil(k / t) - 1 bounds the k-th smallest of all.  Lists of equal
    // quality (the slices of a flat scan) make the widest t the sharpest -- with 256 lists the 100th
    // smallest head --, lists of unequal quality (the probed lists of an inverted file: the
    // nearest few hold nearly all of the answer) a small t on a deep row; wave w tries t = T >> w, T
    // the widest, down to t = 1, and the smallest of their values is taken.  That usually leaves a
    // few hundred entries of tens of thousands, which are ranked directly instead of being searched
    // bit by bit (three barriers instead of forty).
    __shared__ uint32_t bounds_s[16];
    {
        const int row0 = (k + nslice - 1) / nslice - 1;
        const uint32_t t_widest = (uint32_t)((k + row0) / (row0 + 1));  // (<= nslice)
        const uint32_t t = max(t_widest >> wave, 1u);
        const bool active = wave == 0 || (t_widest >> (wave - 1)) > 1u;  // (t = 1 is tried once)
        uint32_t b0 = kNone;
        if (active) {
            const int row = (k + (int)t - 1) / (int)t - 1;  // t (row + 1) >= k, row <= k - 1
            uint32_t rk[16];  // the row, 16 keys to a lane (nslice <= 1024)
            const int nreg = (nslice + 63) >> 6;  // (wave-uniform)
            {
                float rv[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int l = i * 64 + lane;
                    rv[i] = (i < nreg && l < nslice) ? pd[(int64_t)l * k + row] : __builtin_inff();
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) rk[i] = rv[i] != __builtin_inff() ? min(dist_key(rv[i]), kNone - 1u) : kNone;
            }
            b0 = 0;  // the t-th smallest key of the row (kNone when the row has fewer than t entries)
            for (int b = 31; b >= 0; --b) {
                const uint32_t mid = b0 | (1u << b);
                uint32_t cnt = 0;
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (i < nreg) cnt += rk[i] < mid ? 1u : 0u;
                if (wave_sum_u32(cnt) < t) b0 = mid;
            }
        }
        if (lane == 0) bounds_s[wave] = b0;
    }
    __syncthreads();
    uint32_t bound = bounds_s[0];
#pragma unroll
    for (int w = 1; w < 16; ++w) bound = min(bound, bounds_s[w]);
    // entries that exist (low half) and entries at or below the bound (high half), in one count
    // (at most 32768 entries: each half fits 16 bits)
    const uint32_t both = count([&](int i) { return dk[i] != kNone; }, [&](int i) { return bound != kNone && dk[i] <= bound; });
    const uint32_t have = both & 0xffffu;
    const uint32_t kk = have < (uint32_t)k ? have : (uint32_t)k;  // entries to return
    const uint32_t near = bound == kNone ? 1025u : both >> 16;
    if (kk > 0 && near <= 1024u) {
        // (near >= kk: the bound is at or above the k-th smallest key)
#pragma unroll
        for (int i = 0; i < KPL; ++i) {
            if (dk[i] > bound) continue;
            const uint32_t slot = atomicAdd(&nsel, 1u);
            selk[slot] = dk[i];
            seli[slot] = pi[i * 1024 + tid];
        }
        __syncthreads();
        if (tid < (int)near) {
            const uint32_t key = selk[tid];
            const int64_t id = seli[tid];
            const int rank = rank_among(key, id, (int)near);
            if (rank < (int)kk) {
                ids[q * k + rank] = poisoned ? (int64_t)-2 : id;
                dists[q * k + rank] = key_dist(key);
            }
        }
        if (tid >= (int)kk && tid < k) {
            ids[q * k + tid] = poisoned ? (int64_t)-2 : (int64_t)-1;
            dists[q * k + tid] = __builtin_inff();
        }
        return;
    }
    if (kk > 0) {
        uint32_t pivot = 0;  // the kk-th smallest key
        for (int b = 31; b >= 0; --b) {
            const uint32_t mid = pivot | (1u << b);
            if (count([&](int i) { return dk[i] < mid; }) < kk) pivot = mid;
        }
        const uint32_t below = count([&](int i) { return dk[i] < pivot; });
        const uint32_t upto = count([&](int i) { return dk[i] <= pivot; });
        int64_t last = INT64_MAX;  // entries at the pivot distance belong up to this id
        if (upto > kk) {
            int64_t eid[KPL];
#pragma unroll
            for (int i = 0; i < KPL; ++i) eid[i] = dk[i] == pivot ? pi[i * 1024 + tid] : INT64_MAX;
            const uint32_t want = kk - below;  // >= 1
            int64_t lp = 0;
            for (int b = 62; b >= 0; --b) {
                const int64_t mid = lp | ((int64_t)1 << b);
                if (count([&](int i) { return eid[i] < mid; }) < want) lp = mid;
            }
            last = lp;
        }
#pragma unroll
        for (int i = 0; i < KPL; ++i) {
            if (dk[i] > pivot) continue;
            const int64_t id = pi[i * 1024 + tid];
            if (dk[i] == pivot && id > last) continue;
            const uint32_t slot = atomicAdd(&nsel, 1u);
            if (slot < 1024u) {  // (exactly kk <= 1024 entries pass)
                selk[slot] = dist_key(pd[i * 1024 + tid]);
                seli[slot] = id;
            }
        }
    }
    __syncthreads();
    if (tid < (int)kk) {
        const uint32_t key = selk[tid];
        const int64_t id = seli[tid];
        const int rank = rank_among(key, id, (int)kk);
        ids[q * k + rank] = poisoned ? (int64_t)-2 : id;
        dists[q * k + rank] = key_dist(key);
    } else if (tid < k) {
        ids[q * k + tid] = poisoned ? (int64_t)-2 : (int64_t)-1;
        dists[q * k + tid] = __builtin_inff();
    }
}

bool merge_selects(int64_t nq, int nlists, int k)
{
    return (nq <= kMergeSelectQueries || (nq <= kMergeSelectManyQueries && nlists >= 32)) &&
           (int64_t)nlists * k <= kMergeSelectEntries && k >= kMergeSelectMinK && k <= 1024;
}

// One wave per query; the lists are spread over the lanes, OWN to a lane.
// infinite: codes at distance +infinity are listed by the selecting merge too (the other always does).
int launch_merge(const float *part_d, const int64_t *part_i, int64_t nq, int nlists, int k, bool infinite,
                 const int *status, const uint32_t *redo, int64_t *ids, float *dists, hipStream_t s)
{
    PSC_REQUIRE(nlists >= 1 && nlists <= 1024, "between 1 and 1024 partial lists per query, got %d", nlists);
    const dim3 grid((unsigned)nq), block(64);
    if (merge_selects(nq, nlists, k)) {
        if ((int64_t)nlists * k <= 8 * 1024)
            hipLaunchKernelGGL(merge_select_kernel<8>, grid, dim3(1024), 0, s, part_d, part_i, nlists, k, infinite, status,
                               redo, ids, dists);
        else
            hipLaunchKernelGGL(merge_select_kernel<32>, grid, dim3(1024), 0, s, part_d, part_i, nlists, k, infinite, status,
                               redo, ids, dists);
        PSC_HIP_TRY(hipGetLastError());
        return PSC_OK;
    }
    if (nlists <= 64)
        hipLaunchKernelGGL(merge_kernel<1>, grid, block, 0, s, part_d, part_i, nlists, k, (int64_t)0, status, redo, ids, dists);
    else if (nlists <= 128)
        hipLaunchKernelGGL(merge_kernel<2>, grid, block, 0, s, part_d, part_i, nlists, k, (int64_t)0, status, redo, ids, dists);
    else if (nlists <= 256)
        hipLaunchKernelGGL(merge_kernel<4>, grid, block, 0, s, part_d, part_i, nlists, k, (int64_t)0, status, redo, ids, dists);
    else
        hipLaunchKernelGGL(merge_kernel<16>, grid, block, 0, s, part_d, part_i, nlists, k, (int64_t)0, status, redo, ids, dists);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

__global__ void fill_padding_kernel(int64_t *ids, float *dists, int64_t total)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < total) {
        ids[e] = -1;
        dists[e] = __builtin_inff();
    }
}

// Start of a scan: every shared threshold at +infinity and, if asked, the status word cleared.
__global__ void init_scan_kernel(uint32_t *gthr, int64_t n, int *status)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) gthr[e] = kKeyInf;
    if (e == 0 && status) *status = 0;
}

// Hamming filter alone: per query the number of codes within ht (and optionally every distance).
// A workgroup column serves kFilterTQ queries at a time, so that a code is loaded once for all of
// them (their code words are the same for every lane: scalar registers).
constexpr int kFilterTQ = 16;
template <int M>
__global__ void __launch_bounds__(256)
hamming_filter_kernel(const uint8_t *__restrict__ qcodes, int64_t nq, const uint8_t *__restrict__ codes,
                      int64_t n, int ht, unsigned long long *__restrict__ nsurv,
                      uint8_t *__restrict__ hdist)
{
    constexpr int WPC = M / 4;
    const int64_t q0 = (int64_t)blockIdx.y * kFilterTQ;
    const int nvq = (int)((nq - q0) < kFilterTQ ? (nq - q0) : kFilterTQ);
    uint32_t qw[kFilterTQ][WPC];
#pragma unroll
    for (int t = 0; t < kFilterTQ; ++t) {
        const int64_t q = q0 + (t < nvq ? t : 0);
#pragma unroll
        for (int w = 0; w < WPC; ++w) qw[t][w] = ((const uint32_t *)qcodes)[q * WPC + w];
    }
    uint32_t local[kFilterTQ];
#pragma unroll
    for (int t = 0; t < kFilterTQ; ++t) local[t] = 0u;
    // (a thread counts at most n / (256 * gridDim.x) < 2^32 codes per query)
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        uint32_t cw[WPC];
#pragma unroll
        for (int w = 0; w < WPC; ++w) cw[w] = ((const uint32_t *)codes)[i * WPC + w];
#pragma unroll
        for (int t = 0; t < kFilterTQ; ++t) {
            int h = 0;
#pragma unroll
            for (int w = 0; w < WPC; ++w) h += __popc(cw[w] ^ qw[t][w]);
            if (hdist && t < nvq) hdist[(q0 + t) * n + i] = (uint8_t)h;
            local[t] += (h <= ht) ? 1u : 0u;
        }
    }
    // wave reduction, workgroup reduction, then one atomic per workgroup and query (many waves
    // adding to the same few counters would queue up behind each other)
    __shared__ uint32_t part[4][kFilterTQ];
#pragma unroll
    for (int t = 0; t < kFilterTQ; ++t) {
        uint32_t v = local[t];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v += (uint32_t)__shfl_xor((int)v, off, 64);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6][t] = v;
    }
    __syncthreads();
    if ((int)threadIdx.x < nvq) {
        const unsigned long long v = (unsigned long long)part[0][threadIdx.x] + part[1][threadIdx.x] +
                                     part[2][threadIdx.x] + part[3][threadIdx.x];
        if (v) atomicAdd(&nsurv[q0 + threadIdx.x], v);
    }
}

template <int M>
__global__ void __launch_bounds__(256)
hamming_histogram_kernel(const uint8_t *__restrict__ qcodes, const uint8_t *__restrict__ codes, int64_t n,
                         unsigned long long *__restrict__ hist)
{
    constexpr int NB = 8 * M + 1;
    __shared__ unsigned int wbins[4][NB];  // one set of bins per wave: fewer lanes fight over a counter
    unsigned int *bins = wbins[threadIdx.x >> 6];
    const int64_t q = blockIdx.y;
    constexpr int WPC = M / 4;
    for (int b = threadIdx.x; b < 4 * NB; b += 256) (&wbins[0][0])[b] = 0u;
    uint32_t qw[WPC];
#pragma unroll
    for (int w = 0; w < WPC; ++w) qw[w] = ((const uint32_t *)qcodes)[q * WPC + w];
    __syncthreads();
    // (a workgroup sees fewer than 2^32 codes: the grid has at least n / 2^31 columns)
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        int h = 0;
#pragma unroll
        for (int w = 0; w < WPC; ++w) h += __popc(((const uint32_t *)codes)[i * WPC + w] ^ qw[w]);
        atomicAdd(&bins[h], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < NB; b += 256) {
        const unsigned long long v = (unsigned long long)wbins[0][b] + wbins[1][b] + wbins[2][b] + wbins[3][b];
        if (v) atomicAdd(&hist[b], v);
    }
}

__global__ void zero_u64_kernel(unsigned long long *p, int64_t n)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) p[e] = 0;
}

template <int M, int TQ, int NW, bool IVF, bool SHARE>
int run_scan(const ScanArgs &a, int64_t ntiles, size_t lds, hipStream_t s)
{
    static bool configured = false;  // raise the dynamic-LDS ceiling once per instantiation
    if (!configured) {
        PSC_HIP_TRY(hipFuncSetAttribute((const void *)scan_kernel<M, TQ, NW, IVF, SHARE>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
        configured = true;
    }
    hipLaunchKernelGGL((scan_kernel<M, TQ, NW, IVF, SHARE>), dim3((unsigned)ntiles), dim3(NW * 64), lds, s, a);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

template <int M, int NW, bool SHARE, bool IVF = false>
int run_scan_mfma(const ScanArgs &a, int64_t ntiles, size_t lds, hipStream_t s)
{
    static bool configured = false;
    if (!configured) {
        PSC_HIP_TRY(hipFuncSetAttribute((const void *)scan_mfma_kernel<M, NW, SHARE, IVF>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
        configured = true;
    }
    hipLaunchKernelGGL((scan_mfma_kernel<M, NW, SHARE, IVF>), dim3((unsigned)ntiles), dim3(NW * 64), lds, s, a);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

template <int M, int TQ, int NW, bool SHARE, bool FILTER>
int run_adc(const ScanArgs &a, int64_t ntiles, size_t lds, hipStream_t s)
{
    static bool configured = false;
    if (!configured) {
        PSC_HIP_TRY(hipFuncSetAttribute((const void *)adc_kernel<M, TQ, NW, SHARE, FILTER>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
        configured = true;
    }
    hipLaunchKernelGGL((adc_kernel<M, TQ, NW, SHARE, FILTER>), dim3((unsigned)ntiles), dim3(NW * 64), lds, s, a);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

template <int M, bool DENSE, bool MARKED>
int run_scan_pool(const ScanArgs &a, float open, int *status, uint32_t *arrived, int64_t *ids, float *dists,
                  const MarkedQueries &marked, int64_t nwords, hipStream_t s)
{
    static std::atomic<bool> configured{false};
    if (!configured.load(std::memory_order_acquire)) {
        PSC_HIP_TRY(hipFuncSetAttribute((const void *)scan_pool_kernel<M, DENSE, MARKED>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                        (int)sizeof(SmallLds<M>)));
        configured.store(true, std::memory_order_release);
    }
    const int64_t queries = MARKED ? marked.few : a.nq;
    hipLaunchKernelGGL((scan_pool_kernel<M, DENSE, MARKED>), dim3((unsigned)(queries * a.nslice)), dim3(1024), sizeof(SmallLds<M>),
                       s, a, open, status, arrived, ids, dists, marked, nwords);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}
template <bool MARKED>
int dispatch_scan_pool(int m, bool dense, const ScanArgs &a, float open, int *status, uint32_t *arrived, int64_t *ids, float *dists,
                       const MarkedQueries &marked, int64_t nwords, hipStream_t s)
{
    if (m == 8)
        return dense ? run_scan_pool<8, true, MARKED>(a, open, status, arrived, ids, dists, marked, nwords, s)
                     : run_scan_pool<8, false, MARKED>(a, open, status, arrived, ids, dists, marked, nwords, s);
    return dense ? run_scan_pool<16, true, MARKED>(a, open, status, arrived, ids, dists, marked, nwords, s)
                 : run_scan_pool<16, false, MARKED>(a, open, status, arrived, ids, dists, marked, nwords, s);
}
// The slices of a marked query: as many as its last workgroup puts together, up to 16, of 16384 codes and more.  Small
// ones: where half of all codes are at one distance a query is dear (30 marks of 3000 queries x 200k codes, k = 100, whole
// search: slices of 8192 codes 731 us, 16384 775, 65536 1063); and few: workgroups that find nothing marked take time too
// (of that search of 400 us without marks 8, 5 and 4 us).
int marked_slices(int64_t n, int k)
{
    int slices = 16;
    while (slices > 1 && (slices * k > kSmallPool || n < (int64_t)slices * 16384)) slices /= 2;
    return slices;
}

template <bool SHARE, bool FILTER>
int dispatch_adc(int m, int tq, int nwaves, const ScanArgs &a, int64_t ntiles, size_t lds, hipStream_t s)
{
    if constexpr (FILTER) {
        if (m == 8 && tq == 8 && nwaves == 8) return run_adc<8, 8, 8, SHARE, true>(a, ntiles, lds, s);
    }
    if (nwaves != 16) {
        set_error("no kernel for tile shape m=%d tq=%d waves=%d", m, tq, nwaves);
        return PSC_EINVAL;
    }
    if (m == 8) {
        if (tq == 16) return run_adc<8, 16, 16, SHARE, FILTER>(a, ntiles, lds, s);
        if (tq == 8) return run_adc<8, 8, 16, SHARE, FILTER>(a, ntiles, lds, s);
        return run_adc<8, 4, 16, SHARE, FILTER>(a, ntiles, lds, s);
    }
    if (tq == 8) return run_adc<16, 8, 16, SHARE, FILTER>(a, ntiles, lds, s);
    return run_adc<16, 4, 16, SHARE, FILTER>(a, ntiles, lds, s);
}

}  // namespace

// Share of uniformly random b-bit codes within Hamming distance ht of a given one: what the
// launcher goes by when it picks the kernel (real codes differ, but not by enough to matter for
// a choice between two kernels that both give the same results).
double random_code_survival(int nbits, int ht)
{
    double c = 1.0, sum = 0.0;  // c = C(nbits, i) / 2^nbits, built up stepwise
    for (int i = 0; i < nbits; ++i) c *= 0.5;
    for (int i = 0; i <= ht && i <= nbits; ++i) {
        sum += c;
        c = c * (double)(nbits - i) / (double)(i + 1);
    }
    return sum;
}

namespace {
// The tile shapes plan_scan hands out (queries per tile x waves per workgroup).
template <bool IVF, bool SHARE>
int dispatch_scan(int m, int tq, int nwaves, const ScanArgs &a, int64_t ntiles, size_t lds, hipStream_t s)
{
    if constexpr (IVF) {
        if (m == 8 && tq == 4 && nwaves == 8) return run_scan<8, 4, 8, true, SHARE>(a, ntiles, lds, s);
        if (m == 8 && tq == 4 && nwaves == 16) return run_scan<8, 4, 16, true, SHARE>(a, ntiles, lds, s);
        if (m == 16 && tq == 8 && nwaves == 16) return run_scan<16, 8, 16, true, SHARE>(a, ntiles, lds, s);
        if (m == 16 && tq == 4 && nwaves == 16) return run_scan<16, 4, 16, true, SHARE>(a, ntiles, lds, s);
    } else {
        if (m == 8 && tq == 8 && nwaves == 8) return run_scan<8, 8, 8, false, SHARE>(a, ntiles, lds, s);
        if (m == 8 && tq == 16 && nwaves == 16) return run_scan<8, 16, 16, false, SHARE>(a, ntiles, lds, s);
        if (m == 8 && tq == 8 && nwaves == 16) return run_scan<8, 8, 16, false, SHARE>(a, ntiles, lds, s);
        if (m == 8 && tq == 4 && nwaves == 16) return run_scan<8, 4, 16, false, SHARE>(a, ntiles, lds, s);
        if (m == 16 && tq == 8 && nwaves == 16) return run_scan<16, 8, 16, false, SHARE>(a, ntiles, lds, s);
        if (m == 16 && tq == 4 && nwaves == 16) return run_scan<16, 4, 16, false, SHARE>(a, ntiles, lds, s);
    }
    set_error("no kernel for tile shape m=%d tq=%d waves=%d", m, tq, nwaves);
    return PSC_EINVAL;
}

constexpr size_t kLdsBudget = 160 * 1024;

thread_local char g_route[96] = "";

void note_route(const char *kernel, int m, int tq, int nwaves, int nslice, int64_t ntiles)
{
    snprintf(g_route, sizeof g_route, "%s m=%d tq=%d waves=%d slices=%d tiles=%lld", kernel, m, tq, nwaves, nslice,
             (long long)ntiles);
}

}  // namespace

std::atomic<int> g_filter_route{PSC_ROUTE_AUTO};

const char *last_scan_route() { return g_route; }

void note_scan_route(const char *text) { snprintf(g_route, sizeof g_route, "%s", text); }

// Tile shape and database slices.
// Shapes (queries per tile x waves per workgroup), per kind of scan, first one that fits:
//  * fused scan, 64-bit codes, more than 16 queries: 8 x 8, two workgroups per compute unit (one
//    stages its tables or waits on a list lock while the other filters; fewer waves per list
//    lock) -- measured 4% (clustered codes) to 11% (random codes) ahead of 16 x 16 at ht=24;
//    falls back to 16 x 16, 8 x 16, 4 x 16 as k grows (the lists share LDS with the tables);
//  * fused scan with the matrix-core filter (9 queries or more): 16 x 16 (k up to 136) at 64 bits, 8 x 16
//    at 128, the only shapes of scan_mfma_kernel;
//  * up to 4 / 8 / 16 queries: no more query slots than queries (every slot costs filter work),
//    which keeps a one-pass scan of few queries bound by memory bandwidth;
//  * grouped inverted-file jobs: 4 x 8, three workgroups per compute unit (tiles are short, so
//    their set-up and tail overlap better: 12.4 -> 9.3 ms on the 100M workload);
//  * dense route, with or without the Hamming test: the 16-wave shapes (70 against 76 ms for
//    8 x 8 at 64 bits).
int plan_scan(int m, int64_t nq, int64_t n, int k, int kind, ScanPlan *plan)
{
    if (m != 8 && m != 16) {
        set_error("m must be 8 or 16, got %d", m);
        return PSC_EINVAL;
    }
    if (k < 1 || k > PSC_MAX_K) {
        set_error("k must be in [1, %d], got %d", PSC_MAX_K, k);
        return PSC_EINVAL;
    }
    if (nq < 0 || n < 0 || n >= ((int64_t)1 << 40)) {
        set_error("bad sizes nq=%lld n=%lld", (long long)nq, (long long)n);
        return PSC_EINVAL;
    }
    ScanPlan p;
    p.kpad = (k + 3) / 4 * 4;
    struct Shape {
        int tq, nwaves;
        size_t max_lds;  // the shape is meant for this many bytes at most (several workgroups per unit)
    };
    const int tq_cap = nq <= 4 ? 4 : (nq <= 8 ? 8 : 16);
    Shape options[5];
    int nopt = 0;
    if (kind == kScanFusedMfma) {
        if (nq < kMfmaMinQueries) {
            set_error("the matrix-core filter takes at least %d queries", (int)kMfmaMinQueries);
            return PSC_EINVAL;
        }
        options[nopt++] = Shape{m == 8 ? 16 : 8, 16, kLdsBudget};
    } else {
        if (m == 8 && kind == kScanLists) options[nopt++] = Shape{4, 8, kLdsBudget / 2};
        if (m == 8 && kind == kScanFused && nq > 16)
            options[nopt++] = Shape{8, 8, kLdsBudget / 2};
        if (m == 8 && kind != kScanLists) options[nopt++] = Shape{16, 16, kLdsBudget};
        if (kind != kScanLists || m == 16) options[nopt++] = Shape{8, 16, kLdsBudget};
        options[nopt++] = Shape{4, 16, kLdsBudget};
    }
    p.tq = 0;
    for (int o = 0; o < nopt; ++o) {
        const int t = options[o].tq, nw = options[o].nwaves;
        if (t > tq_cap) continue;
        const size_t need = (size_t)t * m * 256 * 4 + (size_t)t * p.kpad * 8 + (size_t)t * 16 + (size_t)t * m * 5 +
                            (size_t)nw * ((kind == kScanFusedMfma ? kMfmaQueueCap : kQueueCap) + 1) * 8;
        if (need <= options[o].max_lds) {
            p.tq = t;
            p.nwaves = nw;
            p.lds_bytes = need;
            break;
        }
    }
    if (p.tq == 0) {
        set_error("no tile shape fits LDS for m=%d k=%d", m, k);
        return PSC_EINVAL;
    }
    // workgroups of this shape a compute unit holds at a time (LDS, and 32 waves)
    p.wgs_per_cu = (int)std::max<size_t>(1, std::min<size_t>(kLdsBudget / p.lds_bytes, (size_t)(32 / p.nwaves)));
    // (one workgroup per unit already saturates memory for a handful of queries, and every further
    //  slice costs list and merge work: measured best at 256 workgroups for 1 to 128 queries)
    const int64_t round = 256 * (int64_t)(nq <= 16 ? 1 : p.wgs_per_cu);
    const int64_t nqt = (nq + p.tq - 1) / p.tq;
    // Slices: one workgroup per (query tile, slice); the launch runs in rounds of `round`
    // workgroups.  Every slice of a query builds its own list of k, which costs insertions and
    // merge work, so the fewest slices win that keep the compute units busy.
    const int64_t block = 512;  // codes per wave and step, at most (64 lanes x 8 codes)
    const int64_t min_slice = p.nwaves * block;  // at least one block per wave
    const int64_t max_by_size = std::max<int64_t>(1, n / min_slice);
    const int64_t wg_limit = std::max<int64_t>(8 * round, nqt);
    int64_t want = 1, tiles_one = 0;
    if (nqt > 0 && nq <= 16) {
        // a handful of queries: score = share of the rounds' places that are used, less 1% per round.  Of
        // the slices that take the same number of rounds the most score best, so one candidate per round
        // is looked at (all 2048 slices, four plans to a call, took 45 of 1 query x 100k codes' 65 us)
        double best_score = -1.0;
        for (int64_t rounds = 1; rounds * round <= wg_limit; ++rounds) {
            const int64_t sN = rounds * round / nqt, wg = nqt * sN;
            if (sN < 1 || wg <= (rounds - 1) * round) continue;
            const double score = (double)wg / (double)(rounds * round) - 0.01 * (double)rounds;
            if (score > best_score + 1e-9) {
                best_score = score;
                want = sN;
            }
        }
    } else if (nqt > 0) {
        // Batches: the query tiles that fill whole rounds are scanned in one piece each, only the
        // tiles of the last, partial round are cut into slices (see flat_tile) -- or all tiles are
        // cut alike, whichever is estimated cheaper.  Time in units of "one workgroup scans the
        // whole database": the whole rounds, plus the rounds of the sliced tiles at 1/S each;
        // every extra list of a query is charged 4% (measured: two lists instead of one for all
        // queries cost about 8% at the headline size).
        double best_cost = 1e300;
        const int64_t whole_rounds_tiles = n <= kMaxSliceLen ? (nqt / round) * round : 0;
        for (int64_t t1 : {whole_rounds_tiles, (int64_t)0}) {
            const int64_t rest = nqt - t1;
            for (int64_t sN = 1; sN <= std::min<int64_t>(max_by_size, 1024) && rest * sN <= wg_limit; ++sN) {
                const double time = (double)t1 / (double)round +
                                    (rest ? (double)((rest * sN + round - 1) / round) / (double)sN : 0.0);
                const double extra = (double)(rest * (sN - 1)) / (double)nqt;
                const double cost = time * (1.0 + 0.04 * extra);
                if (cost < best_cost - 1e-12) {
                    best_cost = cost;
                    want = sN;
                    tiles_one = t1;
                }
                if (!rest) break;
            }
        }
    }
    int64_t nslice = std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(want, max_by_size), 1024));
    int64_t slice_len = (((n + nslice - 1) / nslice) + block - 1) / block * block;
    if (slice_len > kMaxSliceLen) {
        slice_len = kMaxSliceLen;
        nslice = (n + slice_len - 1) / slice_len;
        if (nslice > 1024) {
            set_error("database too large for one scan call");
            return PSC_EINVAL;
        }
    }
    if (slice_len == 0) slice_len = block;
    nslice = std::max<int64_t>(1, (n + slice_len - 1) / slice_len);
    p.nslice = (int)nslice;
    p.slice_len = slice_len;
    p.tiles_one = tiles_one;
    p.ntiles = tiles_one + (nqt - tiles_one) * nslice;
    const size_t dist_bytes = ((size_t)nq * nslice * k * sizeof(float) + 255) / 256 * 256;
    p.part_bytes = dist_bytes + (size_t)nq * nslice * k * sizeof(int64_t);
    // a query cut into many slices exchanges one word per 64th of them (see ScanArgs::pub_slots)
    p.pub_slots = shared_threshold_words(nslice);
    p.gthr_bytes = ((size_t)nq * p.pub_slots * sizeof(uint32_t) + 255) / 256 * 256;
    p.total_bytes = 256 + p.gthr_bytes + p.part_bytes;
    *plan = p;
    return PSC_OK;
}

int merge_partial_lists(const float *part_d, const int64_t *part_i, int64_t nq, int nlists, int k, const int *status,
                        int64_t *ids, float *dists, hipStream_t s)
{
    return launch_merge(part_d, part_i, nq, nlists, k, false, status, nullptr, ids, dists, s);
}

int shared_threshold_words(int64_t lists_per_query)
{
    return lists_per_query >= kManySlices ? (int)std::min<int64_t>(lists_per_query, 64) : 1;
}

size_t flat_scan_workspace_bytes(int m, int64_t nq, int64_t n, int k)
{
    size_t bytes = 0;
    for (int kind : {kScanFused, kScanDense, kScanDenseFiltered}) {
        ScanPlan p;
        if (plan_scan(m, nq, n, k, kind, &p) != PSC_OK) return 0;
        bytes = std::max(bytes, p.total_bytes);
    }
    ScanPlan p;  // the matrix-core route where it applies (it has shapes and slices of its own)
    if (nq >= kMfmaMinQueries && plan_scan(m, nq, n, k, kScanFusedMfma, &p) == PSC_OK)
        bytes = std::max(bytes, p.total_bytes);
    return bytes;
}

// The exchange between the lists of one query (ScanArgs::pub_slots), for `slots` words per query.
static void set_exchange(ScanArgs &a, int slots, int k)
{
    a.pub_slots = slots;
    a.pub_r = k;
    a.pub_kth = 1;
    if (slots > 1) {
        a.pub_r = std::min(k, std::max(1, (5 * k + 2 * slots - 1) / (2 * slots)));
        a.pub_kth = (k + a.pub_r - 1) / a.pub_r;
    }
}

// Whether a flat scan takes scan_pool_kernel, and in how many slices per query (0: it does not): two
// estimates in microseconds, from what each kernel does.
//  * pool: 256 workgroups run at a time; each takes its start, its selections, its codes and its survivors,
//    all together no less than memory gives (every query reads the codes for itself); several slices a merge
//    (pool_merge_cost).
//  * tiled: a round of workgroups takes a tile's set-up, its pairs and surviving pairs, and about k (1 +
//    ln(survivors / k)) insertions into each list, one after the other; then the merge.
// The survivors are those of random codes and a share for one's own cluster (1 % of all codes at ht =
// 3 m, falling with the threshold).  Coefficients fitted to 5634 random calls (3k .. 10M codes, random and
// clustered, x 1 .. 4000 queries, k = 1 .. 1000, thresholds 0 .. 8 m) before the last workgroup merged.  The rule as it
// is, on 3000 other calls (x 1 .. 1000 queries): 0.361 of the tiled kernels' time in geometric mean over 2000 calls of
// psc_scan, 0.436 over 1000 of psc_search (0.360 and 0.436 if the faster were always taken); the pool is
// taken and more than 5 % slower in 17 of 2396.  E.g. (pool / tiled, us): 500k x 83 queries, k = 1000 65 / 457; 165k
// x 97, k = 100 29 / 123; 4M x 75, k = 100 287 / 218.
struct ScanCosts {
    // pool: a workgroup, a selection, 100 keys kept, 1000 codes, 1000 survivors
    double group, select, kept, code, survivor;
    // tiled: the launches, a tile, 1000 pairs by either filter and 1000 surviving pairs (to 16 waves), an
    // insertion, the merge per result
    double launch, tile, pair, pair_mfma, surviving_pair, insertion, merge_k;
};
// Several slices: whether the query's last workgroup puts them together, and what that takes in microseconds (a merge
// launch: `launch`).  The last workgroup ranks up to kRankedKeys keys and searches among more; where the tables' kernel
// has not set its word (preset), a launch that sets it comes first, and with few results out of many keys a merge
// launch instead is the faster one (4M codes x 4 queries, k = 10, 64 slices 33.1 / 36.8 us; k = 100: 39.7 / 35.0).
static bool pool_merges_itself(int64_t slices, int64_t n, int k, bool preset)
{
    return slices * k <= kSmallPool && n < ((int64_t)1 << 31) && (preset || k > 16 || slices * k <= 256);
}
static double pool_merge_cost(int64_t slices, int64_t n, int k, bool preset, double launch)
{
    const double keys = (double)(slices * k);
    if (slices == 1) return 0.0;
    if (!pool_merges_itself(slices, n, k, preset)) return launch;
    return (preset ? 3.0 : 5.5) + (keys <= kRankedKeys ? 1.3e-5 * keys * keys : 6.0);
}
// The estimates in microseconds (pool: infinite where it is not taken at all) and the pool's slices.
struct ScanTimes {
    double pool = HUGE_VAL, tiled = 0.0;
    int64_t slices = 0;
};
static ScanTimes scan_times(int m, int64_t nq, int64_t n, int k, int ht, bool dense, bool mfma, bool preset, const ScanPlan &p,
                            double cached = 1e7)  // bytes a microsecond from the caches
{
    ScanTimes times;
    // (a workgroup per query: past 4096 queries the tiles are ahead; past the caches every query reads
    //  memory for itself: 50M codes of 64 bits, 1 query 138 / 179 us, 2 queries 205 / 181, 400M 786 / 644)
    const double bytes = (double)n * m;
    const bool pool_serves = nq <= 4096 && bytes <= (nq == 1 ? 400e6 : 128e6);
    static constexpr ScanCosts kCosts[2][2] = {
        {{1.4, 6.7, 2.3, 0.11, 0.58, 0.0, 24.0, 0.059, 0.0149, 0.45, 0.68, 0.25},
         {2.0, 8.0, 2.2, 0.126, 0.92, 9.0, 11.0, 0.19, 0.035, 0.76, 0.61, 0.25}},
        {{11.7, 0.0, 2.8, 0.385, 0.0, 0.0, 44.0, 0.213, 0.213, 0.0, 0.68, 1.7},
         {12.2, 0.0, 2.7, 0.742, 0.0, 0.0, 28.0, 0.346, 0.346, 0.0, 0.5, 1.4}}};
    const ScanCosts &c = kCosts[dense ? 1 : 0][m == 8 ? 0 : 1];
    const double in_cluster = 0.01 * std::pow((double)ht / (3 * m), 6);
    const double keep = ht >= 8 * m ? 1.0 : std::min(1.0, random_code_survival(8 * m, ht) + in_cluster);
    const double memory = (double)nq * bytes / (bytes < 128e6 ? cached : 5.8e6);
    // the slices: a merge against the codes of a workgroup (the plain estimate the fit's slices were chosen by)
    const double kilo = dense ? (m == 8 ? 0.37 : 0.72) : 0.13;
    double best = 1e300;
    int64_t slices = 0;
    for (int64_t sN = 1; pool_serves && sN <= 256 && (sN == 1 || (sN * nq <= 256 && sN * 8192 <= n)); sN *= 2) {
        if ((n + sN - 1) / sN > (1 << 24)) continue;
        const double t = std::max((double)((nq * sN + 255) / 256) * (10.0 + 1e-3 * kilo * (double)n / (double)sN), memory) +
                         pool_merge_cost(sN, n, k, preset, 10.0 + 1e-3 * (double)(sN * k));
        if (t < best) {
            best = t;
            slices = sN;
        }
    }
    if (slices != 0) {
        const double codes = (double)n / (double)slices;
        const double group = c.group + c.select * std::min(1.0, keep * codes / k) + 0.01 * c.kept * std::min(keep * codes, (double)k) +
                             1e-3 * codes * (c.code + c.survivor * keep);
        // (where the queries read more than 1.2 GB in all the estimate is low by about what a merge of their own saves:
        //  58 queries x 1.5M codes of 128 bits 155 / 125 us in tiles, 44 x 4.4M of 64 bits 168 / 133)
        const double launch_merge = merge_selects(nq, (int)slices, k) ? 17.0 + 2.1e-3 * (double)(slices * k) : 10.0 + 0.31 * k;
        const double merged = (double)nq * bytes > 1.2e9 && slices > 1 ? launch_merge : pool_merge_cost(slices, n, k, preset, launch_merge);
        times.pool = 10.5 + std::max((double)((nq * slices + 255) / 256) * group, memory) + merged;
        times.slices = slices;
    }
    auto tile_time = [&](double len) {
        const double survivors = keep * len, insertions = std::min(survivors, k * (1.0 + std::log(std::max(1.0, survivors / k))));
        return c.tile + c.insertion * insertions +
               1e-3 * len * p.tq * 16.0 / p.nwaves * ((mfma ? c.pair_mfma : c.pair) + c.surviving_pair * keep);
    };
    const double at_a_time = 256.0 * p.wgs_per_cu, sliced = (double)(p.ntiles - p.tiles_one) / at_a_time;
    const double scan = (double)p.tiles_one / at_a_time * tile_time((double)n) +
                        (p.tiles_one > 0 ? sliced : std::max(1.0, sliced)) * tile_time((double)p.slice_len);
    const double merge = merge_selects(nq, p.nslice, k) ? 13.0 + 5e-4 * (double)p.nslice * k : c.merge_k * k;
    times.tiled = c.launch + std::max(scan, bytes / 5.8e6) + merge;
    return times;
}
static int pool_scan_slices(int m, int64_t nq, int64_t n, int k, int ht, bool dense, bool mfma, bool preset, const ScanPlan &p,
                            size_t ws_bytes)
{
    const ScanTimes t = scan_times(m, nq, n, k, ht, dense, mfma, preset, p);
    if (t.slices == 0 || t.pool > 0.95 * t.tiled) return 0;
    const size_t need = 256 + ((size_t)nq * t.slices * k * sizeof(float) + 255) / 256 * 256 + (size_t)nq * t.slices * k * sizeof(int64_t);
    return need <= ws_bytes ? (int)t.slices : 0;
}

// Which kernel serves a flat scan, and its plan.
struct ScanRoute {
    bool dense = false, mfma = false;
    ScanPlan plan;
};
static int scan_route(int m, int64_t nq, int64_t n, int k, int ht, size_t ws_bytes, ScanRoute *r)
{
    // survivor share from which scoring every pair is the faster route: the dense kernel takes the
    // same time whatever the threshold (it tests only the pairs that beat the k-th best), the fused
    // one grows with the survivors (10M x 10k random codes, k = 100, fused / dense: 64-bit codes ht = 29:
    // 52.1 / 68.8 ms, 30: 67.2 / 69.0, 31: 83.7 / 69.0; 128-bit codes ht = 61: 124 / 136, 62: 148 / 136)
    const double dense_from = 0.34;
    r->dense = ht >= 8 * m || random_code_survival(8 * m, ht) >= dense_from;
    ScanPlan &p = r->plan;
    int rc = PSC_EINVAL;
    const bool dense = r->dense;
    // Matrix-core filter: 9 queries or more and k small enough for its tile of 16 (128 bits: 8).  128 bits: ahead
    // at every threshold that is not the dense route's (10M random codes, 2000 queries, k = 100, matrix cores
    // / xor-popcount; ht = 40: 3.0 / 5.4 ms, 48: 3.2 / 5.5, 56: 8.3 / 10.1, 60: 20.7 / 21.0).  64 bits: so
    // too while few pairs survive (ht = 24: 2.9 / 4.6); with a tenth or more of them surviving the lists
    // decide, and the smaller tiles of the other keep more of them moving until there are some 5e8 pairs (2000
    // x 10M ht = 26: 4.5 / 6.5 ms, 28: 8.2 / 10.1, 29: 10.7 / 12.7; 93 x 55k, k = 1, ht = 28: 67 / 41 us).
    // psc_set_filter_route overrides the rule (for measurements).
    const bool enough = nq >= kMfmaMinQueries;
    bool &mfma = r->mfma;
    mfma = !dense && enough && (m == 16 || random_code_survival(64, ht) < 0.10 || (double)nq * (double)n >= 5e8);
    const int forced = g_filter_route.load(std::memory_order_relaxed);
    if (forced == PSC_ROUTE_POPCOUNT) mfma = false;
    if (forced == PSC_ROUTE_MFMA) mfma = !dense && enough;
    if (mfma) {
        rc = plan_scan(m, nq, n, k, kScanFusedMfma, &p);
        // (k too large for the shape, or a workspace that holds only the popcount kernel's plan: that one
        // takes over)
        mfma = rc == PSC_OK && ws_bytes >= p.total_bytes;
    }
    if (!mfma)
        rc = plan_scan(m, nq, n, k, !dense ? kScanFused : (ht >= 8 * m ? kScanDense : kScanDenseFiltered), &p);
    return rc;
}

double estimated_scan_time(int m, int64_t nq, int64_t n, int k, int ht, size_t ws_bytes)
{
    ScanRoute r;
    if (scan_route(m, nq, n, k, ht, ws_bytes, &r) != PSC_OK) return 0.0;
    const ScanTimes t = scan_times(m, nq, n, k, ht, r.dense, r.mfma, true, r.plan);
    if (t.pool > 0.95 * t.tiled) return t.tiled;
    // (two workgroups a compute unit, the caches give the filtered scan of 128-bit codes more than the route's estimate has
    //  them give: 600 queries x 200k, k = 200, ht 48 192 us by that and 130 in fact, 1200 x 400k 768 and 407)
    if (m == 16 && !r.dense && nq >= 512) return scan_times(m, nq, n, k, ht, r.dense, r.mfma, true, r.plan, 1.8e7).pool;
    return t.pool;
}

int launch_scan(int m, const float *lut_dev, const uint8_t *qcodes_dev, int64_t nq,
                const uint8_t *codes_dev, int64_t n, int ht, int k, int64_t skip_first,
                bool clear_status, bool preset, int64_t *ids_dev, float *dists_dev, void *ws, size_t ws_bytes,
                hipStream_t s, const MarkedQueries *marked)
{
    PSC_REQUIRE(ht >= 0, "ht must be >= 0, got %d", ht);
    ScanRoute route;
    int rc = scan_route(m, nq, n, k, ht, ws_bytes, &route);
    if (rc != PSC_OK) return rc;
    const ScanPlan &p = route.plan;
    const bool dense = route.dense, mfma = route.mfma;
    if (nq == 0) return PSC_OK;
    PSC_REQUIRE(ids_dev && dists_dev, "null result pointer");
    if (n == 0) {
        const int64_t total = nq * k;
        hipLaunchKernelGGL(fill_padding_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s,
                           ids_dev, dists_dev, total);
        PSC_HIP_TRY(hipGetLastError());
        return PSC_OK;
    }
    PSC_REQUIRE(lut_dev && qcodes_dev && codes_dev, "null input pointer");
    PSC_REQUIRE(((uintptr_t)codes_dev & 15) == 0 && ((uintptr_t)qcodes_dev & 15) == 0 &&
                    ((uintptr_t)lut_dev & 15) == 0,
                "codes, query codes and tables must be 16-byte aligned");
    PSC_REQUIRE(ws && ws_bytes >= p.total_bytes, "workspace too small: need %zu bytes, got %zu",
                p.total_bytes, ws_bytes);
    PSC_REQUIRE(((uintptr_t)ws & 255) == 0, "workspace must be 256-byte aligned");
    PSC_REQUIRE(p.ntiles <= 0x7fffffffLL, "too many tiles");

    ScanArgs a;
    a.lut = lut_dev;
    a.qcodes = qcodes_dev;
    a.codes = codes_dev;
    a.skip_first = skip_first;
    a.nq = nq;
    a.n = n;
    a.slice_len = p.slice_len;
    a.nslice = p.nslice;
    a.tiles_one = p.tiles_one;
    a.k = k;
    a.kpad = p.kpad;
    const int nbits = 8 * m;
    const int ht_eff = ht > nbits ? nbits : ht;
    a.bias = 0x7fffffffu - (uint32_t)ht_eff;
    a.status = (int *)ws;
    a.gthr = (uint32_t *)((char *)ws + 256);
    a.job_q = nullptr;
    a.redo = marked != nullptr ? marked->redo : nullptr;
    a.part_d = (float *)((char *)ws + 256 + p.gthr_bytes);
    a.part_i = (int64_t *)((char *)a.part_d + (((size_t)nq * p.nslice * k * sizeof(float) + 255) / 256 * 256));
    // which entry the lists of a many-slice query publish, and which of the published values bounds
    // the k-th best: pub_kth words x pub_r entries >= k, with pub_kth about 0.4 of the words (the
    // value then sits near the (1.3 k)-th best of everything scanned so far)
    set_exchange(a, p.pub_slots, k);
    // (codes at distance +infinity are listed where the merge of the tiled kernels' lists would list them, whichever kernel
    //  answers)
    const bool infinite = !merge_selects(nq, p.nslice, k);
    const float open = infinite ? HUGE_VALF : FLT_MAX;
    const int64_t nwords = nq * p.pub_slots;
    bool words_set = false;
    if (marked != nullptr) {
        ScanArgs few = a;
        few.nslice = marked_slices(n, k);
        few.slice_len = ((n + few.nslice - 1) / few.nslice + 63) / 64 * 64;
        few.nslice = (int)((n + few.slice_len - 1) / few.slice_len);
        const size_t entries = (size_t)marked->few * few.nslice * k, dist_bytes = (entries * sizeof(float) + 255) / 256 * 256;
        few.part_d = (float *)marked->scratch;
        few.part_i = (int64_t *)((char *)marked->scratch + dist_bytes);
        if (few.slice_len <= (1 << 24) && (few.nslice == 1 || few.nslice * k <= kSmallPool) &&
            dist_bytes + entries * sizeof(int64_t) <= marked->scratch_bytes) {
            rc = dispatch_scan_pool<true>(m, dense, few, open, clear_status ? a.status : nullptr, few.nslice > 1 ? marked->arrived : nullptr,
                                          ids_dev, dists_dev, *marked, nwords, s);
            if (rc != PSC_OK) return rc;
            words_set = true;
        }
    }
    const int pool_slices = g_filter_route.load(std::memory_order_relaxed) == PSC_ROUTE_AUTO && skip_first < 0
                                ? pool_scan_slices(m, nq, n, k, ht, dense, mfma, preset, p, ws_bytes)
                                : 0;
    if (pool_slices > 0) {
        a.nslice = pool_slices;
        a.slice_len = ((n + pool_slices - 1) / pool_slices + 63) / 64 * 64;
        a.nslice = (int)((n + a.slice_len - 1) / a.slice_len);  // (no empty slice)
        // the slices' keys are put together by the query's last workgroup where they fit its pool (and the
        // words it is told by fit the workspace beside them), by a merge launch otherwise
        const size_t dist_bytes = ((size_t)nq * a.nslice * k * sizeof(float) + 255) / 256 * 256;
        const size_t key_bytes = dist_bytes + (size_t)nq * a.nslice * k * sizeof(int64_t);
        const size_t words = ((size_t)nq * sizeof(uint32_t) + 255) / 256 * 256;
        // (several slices: at most 128 queries)
        const bool self_merge = a.nslice > 1 && pool_merges_itself(a.nslice, n, k, preset) &&
                                256 + words + key_bytes <= ws_bytes;
        uint32_t *arrived = self_merge ? a.gthr : nullptr;
        a.part_d = (float *)((char *)ws + 256 + (self_merge ? words : 0));
        a.part_i = (int64_t *)((char *)a.part_d + dist_bytes);
        if (self_merge && !preset && !words_set) {
            hipLaunchKernelGGL(init_scan_kernel, dim3((unsigned)((nq + 255) / 256)), dim3(256), 0, s, arrived, nq, (int *)nullptr);
            PSC_HIP_TRY(hipGetLastError());
        }
        int *status = clear_status && !words_set ? a.status : nullptr;
        rc = dispatch_scan_pool<false>(m, dense, a, open, status, arrived, ids_dev, dists_dev, MarkedQueries{}, 0, s);
        if (rc != PSC_OK) return rc;
        note_route(dense ? "scan_pool_kernel+all" : "scan_pool_kernel", m, 1, 16, a.nslice, nq * a.nslice);
        if (a.nslice == 1 || self_merge) return PSC_OK;
        return launch_merge(a.part_d, a.part_i, nq, a.nslice, k, infinite, a.status, a.redo, ids_dev, dists_dev, s);
    }
    if (!words_set)
        hipLaunchKernelGGL(init_scan_kernel, dim3((unsigned)((nwords + 255) / 256)), dim3(256), 0, s, a.gthr, nwords,
                           clear_status ? a.status : (int *)nullptr);
    // A single query leaves three of the narrowest tile's four query slots empty: they take copies of
    // its tables and code, every wave feeds the list of slot wave % 4, and the four lists are merged
    // when the slice ends -- a list's lock is then shared by 4 waves instead of 16 while the lists
    // fill.
    a.spread_lists = (nq == 1 && skip_first < 0) ? 1 : 0;
    a.list_tab = nullptr;
    a.queries = nullptr;
    a.coarse = nullptr;
    a.job_qcodes = nullptr;
    a.dim = 0;
    a.nlist = 0;
    a.tiles = nullptr;
    a.ntiles = nullptr;
    a.list_off = nullptr;
    a.ext_ids = nullptr;
    a.job_slot = nullptr;
    if (ht >= nbits)  // nothing to filter: the pure-ADC kernel
        rc = p.nslice >= 4 ? dispatch_adc<true, false>(m, p.tq, p.nwaves, a, p.ntiles, p.lds_bytes, s)
                           : dispatch_adc<false, false>(m, p.tq, p.nwaves, a, p.ntiles, p.lds_bytes, s);
    else if (dense)
        rc = p.nslice >= 4 ? dispatch_adc<true, true>(m, p.tq, p.nwaves, a, p.ntiles, p.lds_bytes, s)
                           : dispatch_adc<false, true>(m, p.tq, p.nwaves, a, p.ntiles, p.lds_bytes, s);
    else if (mfma)
        rc = m == 8 ? (p.nslice >= 4 ? run_scan_mfma<8, 16, true>(a, p.ntiles, p.lds_bytes, s)
                                     : run_scan_mfma<8, 16, false>(a, p.ntiles, p.lds_bytes, s))
                    : (p.nslice >= 4 ? run_scan_mfma<16, 16, true>(a, p.ntiles, p.lds_bytes, s)
                                     : run_scan_mfma<16, 16, false>(a, p.ntiles, p.lds_bytes, s));
    else
        rc = p.nslice >= 4 ? dispatch_scan<false, true>(m, p.tq, p.nwaves, a, p.ntiles, p.lds_bytes, s)
                           : dispatch_scan<false, false>(m, p.tq, p.nwaves, a, p.ntiles, p.lds_bytes, s);
    if (rc != PSC_OK) return rc;
    note_route(ht >= nbits ? "adc_kernel" : dense ? "adc_kernel+filter" : mfma ? "scan_mfma_kernel" : "scan_kernel",
               m, p.tq, p.nwaves, p.nslice, p.ntiles);
    return launch_merge(a.part_d, a.part_i, nq, p.nslice, k, false, a.status, a.redo, ids_dev, dists_dev, s);
}

// Which filter the grouped inverted-file scan takes.  The matrix-core kernel needs 64-bit codes,
// k small enough for its 16-job tile and enough jobs per list
// to fill its tiles (a tile costs the same filter work whether 16 or 4 of its slots are taken).
// It pays only while next to nothing survives the test: its one 16-wave workgroup per compute
// unit cannot overlap one tile's set-up and list work with another tile's filtering as three
// 8-wave workgroups do, and a list is 24k codes, not 10M.  Measured on 100M vectors / 4096 lists
// / 10k queries x 64 probes, k = 100, whole search, xor/popcount against matrix cores:
// ht = 0: 5.2 / 4.5 ms, 16: 5.4 / 4.9, 20: 7.1 / 9.0, 24: 8.6 / 10.5 (k = 1: 6.2 / 6.2).
// Hence thresholds that let fewer than one random pair in 10^4 through (ht <= 17).
// psc_set_filter_route overrides the rule where the kernel can run at all.
bool ivf_scan_on_matrix_cores(int m, int ht, int k, int64_t njobs, int nlist, int64_t max_list_len, ScanPlan *plan)
{
    if (m != 8 || ht >= 64 || njobs < kMfmaMinQueries) return false;
    bool take = njobs >= 12 * (int64_t)nlist && random_code_survival(64, ht) < 1e-4;
    const int forced = g_filter_route.load(std::memory_order_relaxed);
    if (forced == PSC_ROUTE_POPCOUNT) take = false;
    if (forced == PSC_ROUTE_MFMA) take = true;
    if (!take) return false;
    ScanPlan p;
    if (plan_scan(m, njobs, max_list_len, k, kScanFusedMfma, &p) != PSC_OK) return false;  // (k too large)
    *plan = p;
    return true;
}

// Inverted-file scan: one workgroup per tile descriptor (up to `max_tiles`; the actual count is
// read on the device), partial lists written at job_slot[job] * k, then one merge per query
// over its nprobe partial lists.
int launch_ivf_scan(int m, int tq, int nwaves, int kpad, size_t lds_bytes, const float *lut_dev,
                    const float *list_tab_dev,
                    const float *queries_dev, const float *coarse_dev, int dim, int nlist,
                    uint8_t *job_qcodes_dev, const uint8_t *codes_dev, int64_t n, int ht, int k,
                    const void *tiles_dev, const int *ntiles_dev, int64_t max_tiles,
                    const int64_t *list_off_dev, const int32_t *ext_ids_dev, const int32_t *job_slot_dev,
                    const int32_t *job_q_dev, uint32_t *gthr_dev, float *part_d, int64_t *part_i, int *status,
                    int64_t nq, int nprobe, int64_t *ids_dev, float *dists_dev, bool on_matrix_cores,
                    bool one_job_per_tile, hipStream_t s)
{
    PSC_REQUIRE(((uintptr_t)codes_dev & 15) == 0 && ((uintptr_t)job_qcodes_dev & 15) == 0 &&
                    ((uintptr_t)lut_dev & 15) == 0 && ((uintptr_t)list_tab_dev & 15) == 0,
                "codes, query codes and tables must be 16-byte aligned");
    PSC_REQUIRE(max_tiles <= 0x7fffffffLL, "too many tiles");
    PSC_REQUIRE(dim % m == 0, "dim must be a multiple of m");
    ScanArgs a;
    a.lut = lut_dev;
    a.qcodes = nullptr;
    a.list_tab = list_tab_dev;
    a.queries = queries_dev;
    a.coarse = coarse_dev;
    a.job_qcodes = job_qcodes_dev;
    a.dim = dim;
    a.nlist = nlist;
    a.codes = codes_dev;
    a.skip_first = -1;
    a.nq = 0;
    a.n = n;
    a.slice_len = 0;
    a.nslice = 1;
    a.tiles_one = 0;
    a.k = k;
    a.kpad = kpad;
    const int nbits = 8 * m;
    a.bias = 0x7fffffffu - (uint32_t)(ht > nbits ? nbits : ht);
    a.part_d = part_d;
    a.part_i = part_i;
    a.status = status;
    a.tiles = (const IvfTile *)tiles_dev;
    a.ntiles = ntiles_dev;
    a.list_off = list_off_dev;
    a.ext_ids = ext_ids_dev;
    a.job_slot = job_slot_dev;
    a.job_q = job_q_dev;
    a.gthr = gthr_dev;
    a.spread_lists = one_job_per_tile ? 1 : 0;
    // Tiles of one job each all start together and warm up side by side: they exchange as the
    // slices of a flat scan do.  Grouped tiles of a large batch run one after the other; there a
    // job mostly inherits the k-th best of the query's nearest lists, which one word carries, and
    // reading more than that on every change of a list costs more than it prunes (measured on 100M
    // vectors, 10k queries x 64 probes: 8.3 ms with one word, 21.9 ms with 64).
    set_exchange(a, one_job_per_tile ? shared_threshold_words(nprobe) : 1, k);  // (gthr_dev holds that many words per query)
    const int64_t nwords = nq * a.pub_slots;
    hipLaunchKernelGGL(init_scan_kernel, dim3((unsigned)((nwords + 255) / 256)), dim3(256), 0, s, gthr_dev, nwords,
                       a.status);
    if (max_tiles > 0) {
        int rc;
        if (on_matrix_cores) {
            PSC_REQUIRE(m == 8 && tq == 16 && nwaves == 16, "the matrix-core scan has one tile shape");
            rc = run_scan_mfma<8, 16, true, true>(a, max_tiles, lds_bytes, s);
        } else {
            rc = dispatch_scan<true, true>(m, tq, nwaves, a, max_tiles, lds_bytes, s);
        }
        if (rc != PSC_OK) return rc;
    }
    note_route(on_matrix_cores ? (list_tab_dev ? "scan_mfma_kernel+lists" : "scan_mfma_kernel+lists+direct-tables")
                               : (list_tab_dev ? "scan_kernel+lists" : "scan_kernel+lists+direct-tables"),
               m, tq, nwaves, 1, max_tiles);
    return launch_merge(part_d, part_i, nq, nprobe, k, false, status, nullptr, ids_dev, dists_dev, s);
}

int launch_hamming_filter(int m, const uint8_t *qcodes_dev, int64_t nq, const uint8_t *codes_dev,
                          int64_t n, int ht, int64_t *nsurv_dev, uint8_t *hdist_dev, hipStream_t s)
{
    if (m != 8 && m != 16) {
        set_error("m must be 8 or 16, got %d", m);
        return PSC_EINVAL;
    }
    PSC_REQUIRE(nq >= 0 && n >= 0 && ht >= 0, "bad sizes");
    if (nq == 0) return PSC_OK;
    PSC_REQUIRE(nsurv_dev && qcodes_dev, "null pointer");
    PSC_REQUIRE(nq <= 65535 * (int64_t)kFilterTQ, "too many queries for one filter call");
    hipLaunchKernelGGL(zero_u64_kernel, dim3((unsigned)((nq + 255) / 256)), dim3(256), 0, s,
                       (unsigned long long *)nsurv_dev, nq);
    if (n == 0) return PSC_OK;
    PSC_REQUIRE(codes_dev, "null pointer");
    PSC_REQUIRE(((uintptr_t)codes_dev & 3) == 0 && ((uintptr_t)qcodes_dev & 3) == 0, "codes must be 4-byte aligned");
    const unsigned gx = (unsigned)std::min<int64_t>((n + 255) / 256, 1024);
    const unsigned gy = (unsigned)((nq + kFilterTQ - 1) / kFilterTQ);
    if (m == 8)
        hipLaunchKernelGGL((hamming_filter_kernel<8>), dim3(gx, gy), dim3(256), 0, s, qcodes_dev, nq,
                           codes_dev, n, ht, (unsigned long long *)nsurv_dev, hdist_dev);
    else
        hipLaunchKernelGGL((hamming_filter_kernel<16>), dim3(gx, gy), dim3(256), 0, s, qcodes_dev, nq,
                           codes_dev, n, ht, (unsigned long long *)nsurv_dev, hdist_dev);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

int launch_hamming_histogram(int m, const uint8_t *qcodes_dev, int64_t nq, const uint8_t *codes_dev,
                             int64_t n, int64_t *hist_dev, hipStream_t s)
{
    if (m != 8 && m != 16) {
        set_error("m must be 8 or 16, got %d", m);
        return PSC_EINVAL;
    }
    PSC_REQUIRE(nq >= 0 && n >= 0 && hist_dev, "bad sizes or null histogram");
    PSC_REQUIRE(nq <= 65535, "at most 65535 queries per histogram call");
    hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(256), 0, s, (unsigned long long *)hist_dev, (int64_t)(8 * m + 1));
    if (nq == 0 || n == 0) return PSC_OK;
    PSC_REQUIRE(qcodes_dev && codes_dev, "null pointer");
    PSC_REQUIRE(((uintptr_t)codes_dev & 3) == 0 && ((uintptr_t)qcodes_dev & 3) == 0, "codes must be 4-byte aligned");
    // (64k codes or more per workgroup: every workgroup ends with up to 8m + 1 global additions)
    const unsigned gx = (unsigned)std::max<int64_t>(std::min<int64_t>((n + 65535) / 65536, 2048), (n >> 31) + 1);
    if (m == 8)
        hipLaunchKernelGGL((hamming_histogram_kernel<8>), dim3(gx, (unsigned)nq), dim3(256), 0, s, qcodes_dev,
                           codes_dev, n, (unsigned long long *)hist_dev);
    else
        hipLaunchKernelGGL((hamming_histogram_kernel<16>), dim3(gx, (unsigned)nq), dim3(256), 0, s, qcodes_dev,
                           codes_dev, n, (unsigned long long *)hist_dev);
    PSC_HIP_TRY(hipGetLastError());
    return PSC_OK;
}

}  // namespace psc
