// Sums over a wave's 64 lanes without LDS.
#pragma once

#include <hip/hip_runtime.h>

namespace efem {

template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xF, 0xF, true);
    const uint32_t hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Sum over the 64 lanes; every lane gets the total.  Bound by the chain of
// exchanges: four within a row of 16 by lane permutes in the vector unit, then
// two that swap rows and halves.  Through LDS (six exchanges of two words, each
// a round trip) an FP64 CG iteration of 12^3 hexahedra took 17.9 us against 16.0,
// of 32^3 19.9 and 18.0 (64 to 256 iterations).
__device__ __forceinline__ double wave_sum(double v)
{
    v += dpp_mov<0xB1>(v);    // lane ^ 1
    v += dpp_mov<0x4E>(v);    // lane ^ 2
    v += dpp_mov<0x141>(v);   // mirrored half rows: the other quad's sum
    v += dpp_mov<0x140>(v);   // mirrored rows: the other half row's
    auto swap = [](double a, bool halves) {
        const uint64_t b = __builtin_bit_cast(uint64_t, a);
        const uint32_t lo = (uint32_t)b, hi = (uint32_t)(b >> 32);
        const auto l = halves ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                              : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto h = halves ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                              : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        return __builtin_bit_cast(double, (uint64_t)h[0] << 32 | l[0])
               + __builtin_bit_cast(double, (uint64_t)h[1] << 32 | l[1]);
    };
    v = swap(v, false);
    return swap(v, true);
}

}  // namespace efem
