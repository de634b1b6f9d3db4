// Operations of a wavefront's 64 lanes together: sums, the layer of a chunk.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "co3_internal.h"

namespace co3 {

__device__ inline uint32_t wave_inclusive_scan_dpp(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);   // row_shr 1, 2, 4, 8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);   // row_bcast 15, 31
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);
    return x;
}

// The layer of a user's chunk, the same in all lanes.  64 layers are looked at with a load, where halves would be a chain of one load
// for every doubling.  (segs[nseg].chunk_start = nchunks > chunk; an empty layer begins where the one behind it does.)
__device__ inline uint32_t wave_find_chunk_segment(const SegDev *segs, uint32_t nseg, uint64_t chunk)
{
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t lo = 0, n = nseg;   // among lo .. lo + n - 1, of which the first begins at or before the chunk
    while (n > 1u) {
        const uint32_t step = (n + 63u) >> 6, at = lane * step;
        const uint32_t c = (uint32_t)__popcll(__ballot(at < n && segs[lo + (at < n ? at : 0u)].chunk_start <= chunk)) - 1u;
        lo += c * step;
        n = n - c * step < step ? n - c * step : step;
    }
    return lo;
}

}  // namespace co3
