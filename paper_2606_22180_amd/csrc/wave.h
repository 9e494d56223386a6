// Sums over the 64 lanes of a wavefront without LDS: gfx950's lane swaps for
// distances 32 and 16, DPP moves within a row of 16 lanes below that.  A
// __shfl_xor is a ds_bpermute, a trip through the LDS pipe of about 100
// cycles per step of a dependent chain; these are vector instructions.
//
// Every sum is the butterfly over distances 32, 16, 8, 4, 2, 1 (or its tail),
// so a value's rounding does not depend on which of these functions made it.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace felog {

constexpr int kDppQuadXor1 = 0xB1;   // quad_perm:[1,0,3,2]
constexpr int kDppQuadXor2 = 0x4E;   // quad_perm:[2,3,0,1]
constexpr int kDppRowShl4 = 0x104, kDppRowShr4 = 0x114, kDppRowRor8 = 0x128;

__device__ __forceinline__ uint32_t lo32(double x)
{
    return (uint32_t)(unsigned long long)__double_as_longlong(x);
}
__device__ __forceinline__ uint32_t hi32(double x)
{
    return (uint32_t)((unsigned long long)__double_as_longlong(x) >> 32);
}
__device__ __forceinline__ double make_f64(uint32_t lo, uint32_t hi)
{
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

template <int CTRL, int BANKS = 0xf>
__device__ __forceinline__ uint32_t dpp(uint32_t old, uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)x, CTRL, 0xf, BANKS, false);
}

// The value of lane (own ^ X), X = 1, 2, 4 or 8.
template <int X>
__device__ __forceinline__ uint32_t from_xor(uint32_t x)
{
    if constexpr (X == 1) return dpp<kDppQuadXor1>(0u, x);
    else if constexpr (X == 2) return dpp<kDppQuadXor2>(0u, x);
    else if constexpr (X == 8) return dpp<kDppRowRor8>(0u, x);
    else {
        // lanes 0-3 and 8-11 of a row (banks 0, 2) from 4 lanes up, the others from 4 down
        static_assert(X == 4, "distance");
        return dpp<kDppRowShr4, 0xa>(dpp<kDppRowShl4, 0x5>(0u, x), x);
    }
}
template <int X>
__device__ __forceinline__ double from_xor(double x)
{
    return make_f64(from_xor<X>(lo32(x)), from_xor<X>(hi32(x)));
}

// Lanes whose bit X (16 or 32) is clear get a's sum over the lane pair
// (own, own ^ X), the others b's.
template <int X>
__device__ __forceinline__ double pair_sums(double a, double b)
{
    if constexpr (X == 32) {
        const auto l = __builtin_amdgcn_permlane32_swap(lo32(a), lo32(b), false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(hi32(a), hi32(b), false, false);
        return make_f64(l[0], h[0]) + make_f64(l[1], h[1]);
    } else if constexpr (X == 16) {
        const auto l = __builtin_amdgcn_permlane16_swap(lo32(a), lo32(b), false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(hi32(a), hi32(b), false, false);
        return make_f64(l[0], h[0]) + make_f64(l[1], h[1]);
    } else {
        const bool up = (__lane_id() & X) != 0;
        const double keep = up ? b : a, send = up ? a : b;
        return keep + from_xor<X>(send);
    }
}

// The value's sum over the lane pairs (own, own ^ X), in every lane.
template <int X>
__device__ __forceinline__ double xor_sum(double x)
{
    if constexpr (X >= 16) return pair_sums<X>(x, x);
    else return x + from_xor<X>(x);
}

// Sum over the 64 lanes, in every lane.
__device__ __forceinline__ double wave_total(double x)
{
    x = xor_sum<32>(x);
    x = xor_sum<16>(x);
    x = xor_sum<8>(x);
    x = xor_sum<4>(x);
    x = xor_sum<2>(x);
    return xor_sum<1>(x);
}

__device__ __forceinline__ double read_lane(double x, int lane)
{
    return make_f64((uint32_t)__builtin_amdgcn_readlane((int)lo32(x), lane),
                    (uint32_t)__builtin_amdgcn_readlane((int)hi32(x), lane));
}

}  // namespace felog
