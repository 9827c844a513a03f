// Wave-wide reductions in registers (gfx950), shared by the fix-up and the hard decisions.
#pragma once
#include "device_common.hpp"

namespace dm {

// Wave-wide max / sum of one float per lane, every lane receiving the result, in VALU only
// (the whole wave must be active): v_permlane32_swap and v_permlane16_swap pair lanes 32 and 16
// apart (the two outputs hold the pair in both lanes), then DPP row rotations by 8, 4, 2, 1
// combine the 16 lanes of each row.  No LDS round trips on the callers' dependent chains.
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}

template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

template <typename Op>
__device__ __forceinline__ float wave_reduce_f(float v, Op op) {
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    v = op(__builtin_bit_cast(float, (uint32_t)a[0]), __builtin_bit_cast(float, (uint32_t)a[1]));
    const uint32_t w = __builtin_bit_cast(uint32_t, v);
    const auto b = __builtin_amdgcn_permlane16_swap(w, w, false, false);
    v = op(__builtin_bit_cast(float, (uint32_t)b[0]), __builtin_bit_cast(float, (uint32_t)b[1]));
    v = op(v, dpp_f<0x128>(v));  // row_ror:8
    v = op(v, dpp_f<0x124>(v));  // row_ror:4
    v = op(v, dpp_f<0x122>(v));  // row_ror:2
    v = op(v, dpp_f<0x121>(v));  // row_ror:1
    return v;
}

__device__ __forceinline__ float wave_max_f(float v) {
    return wave_reduce_f(v, [](float x, float y) { return fmaxf(x, y); });
}

__device__ __forceinline__ float wave_sum_f(float v) {
    return wave_reduce_f(v, [](float x, float y) { return x + y; });
}

// The same for 32-bit integers.
template <typename Op>
__device__ __forceinline__ uint32_t wave_reduce_u32(uint32_t v, Op op) {
    return __builtin_bit_cast(uint32_t, wave_reduce_f(__builtin_bit_cast(float, v), [op](float x, float y) {
        return __builtin_bit_cast(float, op(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y)));
    }));
}

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
    return wave_reduce_u32(v, [](uint32_t x, uint32_t y) { return min(x, y); });
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
    return wave_reduce_u32(v, [](uint32_t x, uint32_t y) { return x + y; });
}

// Error counts of received block `blk` (symbol errors, bit errors per lane) summed over the wave
// and added to slot `slot` of counts [n_blk][kAccSlots][2].
__device__ __forceinline__ void hard_flush(unsigned long long* counts, int blk, int slot, int lane, uint32_t se,
                                           uint32_t be) {
    se = wave_sum_u32(se);
    be = wave_sum_u32(be);
    unsigned long long* c = counts + ((size_t)blk * kAccSlots + slot) * 2;
    if (lane == 0) {
        if (se) atomicAdd(c, (unsigned long long)se);
        if (be) atomicAdd(c + 1, (unsigned long long)be);
    }
}

}  // namespace dm
