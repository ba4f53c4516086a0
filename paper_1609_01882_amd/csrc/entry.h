// Result-list entries and the wave helpers of the kernels that make them.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#define PSC_LDS __attribute__((address_space(3)))

namespace psc {
namespace {

__device__ __forceinline__ uint64_t ballot64(bool p) { return __ballot(p); }

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63); }

__device__ __forceinline__ int prefix_count(uint64_t mask)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// One list entry = (sortable distance key, id) packed in 64 bits, key in the high word, so that
// the unsigned 64-bit order is the (distance, id) order.  The key is the usual order-preserving
// map of float bits to unsigned (negative values flip all bits, others flip the sign bit);
// -0 is folded into +0 first so that equal distances get equal keys.
__device__ __forceinline__ uint32_t dist_key(float d)
{
    const uint32_t u = __float_as_uint(d + 0.0f);
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ float key_dist(uint32_t key)
{
    return __uint_as_float(key ^ ((key >> 31) ? 0x80000000u : 0xffffffffu));
}
constexpr uint32_t kKeyInf = 0xff800000u;  // dist_key(+infinity)
constexpr uint64_t kNoEntry = ~0ull;       // above every entry
__device__ __forceinline__ uint64_t pack_entry(float d, uint32_t id)
{
    return ((uint64_t)dist_key(d) << 32) | id;
}
__device__ __forceinline__ float entry_dist(uint64_t e) { return key_dist((uint32_t)(e >> 32)); }
__device__ __forceinline__ uint32_t entry_id(uint64_t e) { return (uint32_t)e; }

}  // namespace
}  // namespace psc
