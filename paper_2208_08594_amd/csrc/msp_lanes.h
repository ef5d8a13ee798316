// Sums across the lanes of a wavefront without LDS: register moves within rows
// of 16 lanes (DPP) and swaps between rows.  Each add_N returns v plus the
// value of the lane N away (xor), the sum a butterfly of __shfl_xor takes, at the
// latency of two register instructions instead of an LDS round trip.
#pragma once

#include <hip/hip_runtime.h>

namespace msp {

template <int CTRL>
__device__ __forceinline__ int lane_move(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ float lane_move(float v)
{
    return __int_as_float(lane_move<CTRL>(__float_as_int(v)));
}
template <int CTRL>
__device__ __forceinline__ double lane_move(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = lane_move<CTRL>((int)b), hi = lane_move<CTRL>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
constexpr int kMoveXor1 = 0xB1, kMoveXor2 = 0x4E;       // quad_perm 1,0,3,2 and 2,3,0,1
constexpr int kMoveRor4 = 0x124, kMoveRor8 = 0x128;     // row_ror: 8 is xor 8, 4 is xor 4 of
                                                        // values of period 8
constexpr int kMoveHalfMirror = 0x141, kMoveMirror = 0x140;  // xor 4 (8) of values that are
                                                             // equal in each four (eight)

// v of the lane 16 (32) away, by xor, plus v
__device__ __forceinline__ float add_16(float v)
{
    const unsigned b = __float_as_uint(v);
    const auto s = __builtin_amdgcn_permlane16_swap(b, b, false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ __forceinline__ float add_32(float v)
{
    const unsigned b = __float_as_uint(v);
    const auto s = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ __forceinline__ double join(unsigned lo, unsigned hi)
{
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double add_16(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const auto l = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32),
                                                    false, false);
    return join(l[0], h[0]) + join(l[1], h[1]);
}
__device__ __forceinline__ double add_32(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const auto l = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32),
                                                    false, false);
    return join(l[0], h[0]) + join(l[1], h[1]);
}

// sum over the wave, in every lane: pairs 32, 16, 8, 4, 2, 1 apart, in that order
template <typename T>
__device__ __forceinline__ T wave_sum(T v)
{
    v = add_32(v);
    v = add_16(v);
    v += lane_move<kMoveRor8>(v);
    v += lane_move<kMoveRor4>(v);
    v += lane_move<kMoveXor2>(v);
    v += lane_move<kMoveXor1>(v);
    return v;
}

// sum over the lanes of equal lane mod 8: pairs 8, 16, 32 apart
template <typename T>
__device__ __forceinline__ T sum_of_rows8(T v)
{
    v += lane_move<kMoveRor8>(v);
    v = add_16(v);
    return add_32(v);
}

// sum over 8 (64) consecutive lanes: pairs 1, 2, 4 (8, 16, 32) apart
template <int L, typename T>
__device__ __forceinline__ T group_sum(T v)
{
    static_assert(L == 8 || L == 64, "8 or 64 lanes");
    v += lane_move<kMoveXor1>(v);
    v += lane_move<kMoveXor2>(v);
    v += lane_move<kMoveHalfMirror>(v);
    if (L == 64) {
        v += lane_move<kMoveMirror>(v);
        v = add_16(v);
        v = add_32(v);
    }
    return v;
}

}  // namespace msp
