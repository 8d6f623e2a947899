// Sums over the 64 lanes of a wave (gfx950), every lane receiving the total.
//
// The lanes are added in butterfly order, partners 32, 16, 8, 4, 2, 1 apart:
// both partners form the same sum, so all lanes end with the same bits.  The
// exchanges stay in the vector unit: v_permlane32_swap and v_permlane16_swap
// hand each lane its partner 32 or 16 lanes away (the two results of a swap
// of a value with itself are the partners' values), and DPP row rotations by
// 8, 4, 2, 1 the nearer ones -- after the step at distance 2 k the values
// repeat every 2 k lanes inside a row of 16, so the lane k places round the
// row holds the partner's value.  A ds_bpermute exchange goes through the
// LDS pipe and is waited for, twice per step for a double; every CG kernel does
// three such sums on its critical path.

#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace mpcg {

template <int CTRL> __device__ inline uint32_t dpp_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}

constexpr int kRowRor8 = 0x128, kRowRor4 = 0x124, kRowRor2 = 0x122, kRowRor1 = 0x121;

// The sum of a lane's value and its partner's, for each step's exchange.
struct LanePair {
    uint32_t a, b;
};
template <int STEP> __device__ inline LanePair lane_pair(uint32_t v)
{
    if (STEP == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return {(uint32_t)r[0], (uint32_t)r[1]};
    }
    if (STEP == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return {(uint32_t)r[0], (uint32_t)r[1]};
    }
    if (STEP == 8) return {v, dpp_u32<kRowRor8>(v)};
    if (STEP == 4) return {v, dpp_u32<kRowRor4>(v)};
    if (STEP == 2) return {v, dpp_u32<kRowRor2>(v)};
    return {v, dpp_u32<kRowRor1>(v)};
}

template <int STEP> __device__ inline double lane_add(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const LanePair lo = lane_pair<STEP>((uint32_t)u), hi = lane_pair<STEP>((uint32_t)(u >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi.a << 32) | lo.a) +
           __builtin_bit_cast(double, ((uint64_t)hi.b << 32) | lo.b);
}

template <int STEP> __device__ inline float lane_add(float v)
{
    const LanePair p = lane_pair<STEP>(__builtin_bit_cast(uint32_t, v));
    return __builtin_bit_cast(float, p.a) + __builtin_bit_cast(float, p.b);
}

template <typename T> __device__ inline T wave_sum_all(T v)
{
    v = lane_add<32>(v);
    v = lane_add<16>(v);
    v = lane_add<8>(v);
    v = lane_add<4>(v);
    v = lane_add<2>(v);
    return lane_add<1>(v);
}

// Integer sum and extremes over the wave by the same exchanges.
template <int STEP, typename F> __device__ inline int lane_fold(int v, const F &f)
{
    const LanePair p = lane_pair<STEP>((uint32_t)v);
    return f((int)p.a, (int)p.b);
}
template <typename F> __device__ inline int wave_fold(int v, const F &f)
{
    v = lane_fold<32>(v, f);
    v = lane_fold<16>(v, f);
    v = lane_fold<8>(v, f);
    v = lane_fold<4>(v, f);
    v = lane_fold<2>(v, f);
    return lane_fold<1>(v, f);
}

// Sum over the wave of x * y, valid in lane 0: the products are rounded once
// except lane l's own (l < 32), which enters its first addition unrounded
// (one fma with the rounded product of lane l + 32).
template <typename T> __device__ inline T wave_dot(T x, T y);
template <> __device__ inline double wave_dot<double>(double x, double y)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, x * y);
    const LanePair lo = lane_pair<32>((uint32_t)u), hi = lane_pair<32>((uint32_t)(u >> 32));
    double v = fma(x, y, __builtin_bit_cast(double, ((uint64_t)hi.b << 32) | lo.b));
    v = lane_add<16>(v);
    v = lane_add<8>(v);
    v = lane_add<4>(v);
    v = lane_add<2>(v);
    return lane_add<1>(v);
}
template <> __device__ inline float wave_dot<float>(float x, float y)
{
    const LanePair p = lane_pair<32>(__builtin_bit_cast(uint32_t, x * y));
    float v = fmaf(x, y, __builtin_bit_cast(float, p.b));
    v = lane_add<16>(v);
    v = lane_add<8>(v);
    v = lane_add<4>(v);
    v = lane_add<2>(v);
    return lane_add<1>(v);
}

}  // namespace mpcg
