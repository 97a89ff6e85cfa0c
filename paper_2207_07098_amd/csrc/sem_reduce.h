// Wave reductions on the vector ALUs (gfx950) and the ordering of LDS accesses
// between the lanes of one wave.  __shfl_xor goes through the LDS pipe (two
// permutes of 32 bits per step of a double); DPP moves do not, and their
// latency hides behind the next value's.
#pragma once

#include <hip/hip_runtime.h>

namespace sem {

// What a lane wrote to LDS before it, every lane of its wave reads after it.
// The hardware runs a wave's LDS operations in order; the fences keep the
// compiler from exchanging a store with another lane's load (the barrier alone
// is no memory operation to it).  They cost no instruction at this scope.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// v of the lane that the DPP control selects, 0.0 where it selects none.
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// Sum over the 64 lanes of a full wave in a fixed order; lane 63 holds it.
__device__ __forceinline__ double wave_sum63(double v) {
    v += dpp_mov<0x111>(v);        // row_shr:1  -- sums of 2, 4, 8, 16 lanes
    v += dpp_mov<0x112>(v);        // row_shr:2
    v += dpp_mov<0x114>(v);        // row_shr:4
    v += dpp_mov<0x118>(v);        // row_shr:8     (lane 15 of each row)
    v += dpp_mov<0x142>(v);        // row_bcast:15  (lanes 31 and 63)
    v += dpp_mov<0x143>(v);        // row_bcast:31  (lane 63)
    return v;
}

// The same sum for every lane.
__device__ __forceinline__ double wave_total(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, wave_sum63(v));
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, 63);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), 63);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

}  // namespace sem
