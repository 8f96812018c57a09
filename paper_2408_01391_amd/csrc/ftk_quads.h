// Rows by pieces of four features, and sums over groups of lanes.
#pragma once

#include <hip/hip_runtime.h>

namespace ftk {

// rows need no more than element alignment: 16-byte loads from 4- or 8-byte aligned addresses
typedef float float4e __attribute__((ext_vector_type(4), aligned(4)));
typedef double double2e __attribute__((ext_vector_type(2), aligned(8)));

template <typename T>
struct Quad {
    T v[4];
};
template <typename T>
__device__ __forceinline__ Quad<T> load_quad(const T *p)
{
    Quad<T> q;
    if constexpr (sizeof(T) == 4) {
        const float4e f = *reinterpret_cast<const float4e *>(p);
#pragma unroll
        for (int e = 0; e < 4; ++e) q.v[e] = f[e];
    } else {
        const double2e f = *reinterpret_cast<const double2e *>(p);
        const double2e h = *reinterpret_cast<const double2e *>(p + 2);
        q.v[0] = f[0];
        q.v[1] = f[1];
        q.v[2] = h[0];
        q.v[3] = h[1];
    }
    return q;
}

// Sum over the L lanes of a group (every lane gets it; the same additions whatever the values).
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
template <int L, typename V>
__device__ __forceinline__ V group_sum(V v)
{
    v += dpp_move<0xB1>(v);                            // lane ^ 1
    if constexpr (L >= 4) v += dpp_move<0x4E>(v);      // lane ^ 2
    if constexpr (L >= 8) v += dpp_move<0x141>(v);     // the other four of eight
    if constexpr (L >= 16) v += dpp_move<0x140>(v);    // the other eight of sixteen
    if constexpr (L >= 32) v += __shfl_xor(v, 16, 64);
    if constexpr (L >= 64) v += __shfl_xor(v, 32, 64);
    return v;
}

}  // namespace ftk
