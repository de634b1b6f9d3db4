// The decoupled look-back of a single-sweep encoder: every workgroup of a user publishes its size, then reads its
// predecessors' entries until it meets one that already knows its running total.  Workgroups take their position from a
// ticket counter, so every predecessor is running and publishes without waiting for anyone.  An entry carries everything a
// successor needs, so it is written and read with relaxed device-scope atomics; one lane makes both stores to it, for only
// that lane's program order keeps the size from landing after the running total.
// (k_encode_fused of the byte alphabets has the same steps written out: called from here they moved its registers, all of
// which it needs, and sixteen users' round of 25.6 M elements took 1192 us instead of 1177.)
#ifndef CO3_LOOKBACK_H
#define CO3_LOOKBACK_H
#include "co3_internal.h"

namespace co3 {

// look-back entry: flag in the top two bits, size in bits below
constexpr uint64_t kLbAgg = 1ull << 62;      // size of this workgroup alone
constexpr uint64_t kLbPrefix = 2ull << 62;   // size of this workgroup and all before it
constexpr uint64_t kLbStalled = 3ull << 62;
constexpr uint64_t kLbValue = (1ull << 62) - 1;

// By the lane that later replaces the entry (lookback_finish).
__device__ inline void lookback_publish(uint64_t *state, uint32_t b, uint32_t own)
{
    __hip_atomic_store(&state[b], (b == 0 ? kLbPrefix : kLbAgg) | own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The nearest 64 predecessor entries, requested now and looked at later; by a whole wavefront.
__device__ inline uint64_t lookback_first(const uint64_t *state, uint32_t b, uint32_t lane)
{
    uint64_t v = kLbPrefix;  // before the first workgroup: running total 0
    if ((int64_t)b - 1 - (int64_t)lane >= 0)
        v = __hip_atomic_load(&state[b - 1 - lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return v;
}

// The sizes of all earlier workgroups; false: an entry stayed empty for spin_limit polls, or was marked as stalled.
__device__ inline bool lookback_collect(const uint64_t *state, uint32_t b, uint64_t lb_first, uint32_t lane,
                                        uint32_t spin_limit, uint64_t &prefix)
{
    prefix = 0;
    int64_t pos = (int64_t)b - 1;
    while (pos >= 0) {
        const int64_t idx = pos - (int64_t)lane;
        uint64_t v = kLbPrefix;  // before the first workgroup: running total 0
        if (idx >= 0) {
            uint32_t spins = 0;
            v = pos == (int64_t)b - 1 ? lb_first
                                      : __hip_atomic_load(&state[idx], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            while ((v >> 62) == 0 && spins < spin_limit) {
                __builtin_amdgcn_s_sleep(1);
                v = __hip_atomic_load(&state[idx], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ++spins;
            }
        }
        // lane 0 holds the nearest predecessor; sum up to and including the first running total
        const uint64_t has_prefix = __ballot((v >> 62) == 2);
        const int stop = has_prefix ? (int)__builtin_ctzll(has_prefix) : 63;
        const bool bad = (int)lane <= stop && ((v >> 62) == 0 || (v >> 62) == 3);
        if (__any(bad)) return false;
        uint64_t val = ((int)lane <= stop) ? (v & kLbValue) : 0ull;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) val += __shfl_xor(val, o, 64);
        prefix += val;
        if (has_prefix) break;
        pos -= 64;
    }
    return true;
}

// The entry's last value, by the lane that published its size.
__device__ inline void lookback_finish(uint64_t *state, uint32_t b, bool ok, uint64_t prefix, uint32_t own, uint64_t *status)
{
    if (!ok) {
        __hip_atomic_store(&state[b], kLbStalled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_STALLED), 1ull);
    } else if (b != 0) {
        __hip_atomic_store(&state[b], kLbPrefix | (prefix + own), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

uint32_t lookback_polls();   // polls of one predecessor entry before giving up (k_fused.hip)

}  // namespace co3
#endif
