// Reductions across the lanes of a wave on DPP and the row swaps, without the
// round trips of shuffles through LDS.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace sw {

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

// Sum over the 64 lanes: butterflies inside each row of 16 lanes on DPP,
// then the four row totals.  Fixed order, so the result is deterministic.
__device__ __forceinline__ float wave_sum_f(float v) {
    v += dpp_f<0xb1>(v);   // quad_perm [1,0,3,2]
    v += dpp_f<0x4e>(v);   // quad_perm [2,3,0,1]
    v += dpp_f<0x141>(v);  // row_half_mirror
    v += dpp_f<0x140>(v);  // row_mirror
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
    return (r0 + r1) + (r2 + r3);
}

// The values of lanes i and i ^ 32 (i ^ 16), in either order.
__device__ __forceinline__ uint2 swap32(unsigned v) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return make_uint2(r[0], r[1]);
}
__device__ __forceinline__ uint2 swap16(unsigned v) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return make_uint2(r[0], r[1]);
}

// Sum over the 64 lanes in the order of butterflies over lane distances 32, 16,
// .. 1, the same bits on every lane.  After the first steps lanes that differ in
// the upper bits alone hold the same value, so a rotation by four in a row of 16
// is as good as the exchange.
__device__ __forceinline__ float wave_butterfly_sum(float v) {
    uint2 p = swap32(__float_as_uint(v));
    v = __uint_as_float(p.x) + __uint_as_float(p.y);
    p = swap16(__float_as_uint(v));
    v = __uint_as_float(p.x) + __uint_as_float(p.y);
    v += dpp_f<0x128>(v);  // row_ror:8
    v += dpp_f<0x124>(v);  // row_ror:4
    v += dpp_f<0x4e>(v);   // quad_perm [2,3,0,1]
    v += dpp_f<0xb1>(v);   // quad_perm [1,0,3,2]
    return v;
}

__device__ __forceinline__ void argmin_merge(double &v, int &i, double v2, int i2) {
    if (v2 < v || (v2 == v && i2 < i)) {
        v = v2;
        i = i2;
    }
}

// Smallest (v, i) over the 64 lanes, by v and then by i, on every lane; a NaN
// never is.
__device__ __forceinline__ void wave_argmin(double &v, int &i) {
    auto row = [&](auto ctrl) {
        constexpr int C = decltype(ctrl)::value;
        const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), C, 0xf, 0xf, false);
        const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), C, 0xf, 0xf, false);
        argmin_merge(v, i, __hiloint2double(hi, lo),
                     __builtin_amdgcn_mov_dpp(i, C, 0xf, 0xf, false));
    };
    row(std::integral_constant<int, 0xb1>{});   // quad_perm [1,0,3,2]
    row(std::integral_constant<int, 0x4e>{});   // quad_perm [2,3,0,1]
    row(std::integral_constant<int, 0x124>{});  // row_ror:4
    row(std::integral_constant<int, 0x128>{});  // row_ror:8
    auto rows = [&](auto swap) {
        const uint2 h = swap(__double2hiint(v)), l = swap(__double2loint(v)), k = swap(i);
        v = __hiloint2double((int)h.x, (int)l.x);
        i = (int)k.x;
        argmin_merge(v, i, __hiloint2double((int)h.y, (int)l.y), (int)k.y);
    };
    rows([](unsigned x) { return swap16(x); });
    rows([](unsigned x) { return swap32(x); });
}

}  // namespace sw
