// Device helpers shared by the kernel sources.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace cut {

// Gather of one element of a row through a buffer resource built (on the
// scalar unit) from the uniform row address: the lane's byte offset is the only
// per-lane operand, so a gather costs no vector address arithmetic.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* row, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(row), (short)0, (int)bytes, 0x00020000);
}
template <class T>
__device__ __forceinline__ T buf_load(__amdgpu_buffer_rsrc_t r, uint32_t voff, int32_t soff) {
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, soff, 0));
    } else {
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, soff, 0));
    }
}

// One state element idx of classic RK4 with right-hand side f at stage `stage`:
// stage 0 starts the accumulator, 1-2 add to it, 3 finishes the step (and
// updates z); returns the next stage state.  z and the accumulator are touched
// once per stage: streamed with non-temporal hints so they do not displace
// gathered rows.
__device__ inline double rk_combine(int stage, double ds, double* z, double* acc, int64_t idx, double f) {
    const double zk = __builtin_nontemporal_load(z + idx);
    double nxt;
    if (stage == 0) {
        __builtin_nontemporal_store(zk + (ds / 6.0) * f, acc + idx);
        nxt = zk + 0.5 * ds * f;
    } else if (stage == 1) {
        __builtin_nontemporal_store(__builtin_nontemporal_load(acc + idx) + (ds / 3.0) * f, acc + idx);
        nxt = zk + 0.5 * ds * f;
    } else if (stage == 2) {
        __builtin_nontemporal_store(__builtin_nontemporal_load(acc + idx) + (ds / 3.0) * f, acc + idx);
        nxt = zk + ds * f;
    } else {
        nxt = __builtin_nontemporal_load(acc + idx) + (ds / 6.0) * f;
        __builtin_nontemporal_store(nxt, z + idx);
    }
    return nxt;
}

}  // namespace cut
