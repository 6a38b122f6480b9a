// Wave-wide combinations without the LDS unit (a general shuffle goes through it).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mvla {

// value of another lane by a data-parallel-primitive control (16-lane rows), 32-bit halves of a double
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
    const long long v = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo));
}

// Sum over the 64 lanes, in all of them; the additions of a butterfly over lane distances 32, 16, 8, 4, 2, 1
// (once lanes 8 apart agree, a rotation by 4 fetches the same value as lane xor 4 does, and so on).
__device__ __forceinline__ double wave_sum_f64(double x) {
    {
        const long long v = __double_as_longlong(x);
        const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(v >> 32), (uint32_t)(v >> 32), false, false);
        x = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
            __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
    }
    {
        const long long v = __double_as_longlong(x);
        const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(v >> 32), (uint32_t)(v >> 32), false, false);
        x = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
            __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
    }
    x += dpp_f64<0x128>(x);   // row_ror:8
    x += dpp_f64<0x124>(x);
    x += dpp_f64<0x122>(x);
    x += dpp_f64<0x121>(x);
    return x;
}

// The same for 32-bit floats.
__device__ __forceinline__ float wave_sum_f32(float x) {
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xf, 0xf, false));   // row_ror:8
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xf, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x122, 0xf, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x121, 0xf, 0xf, false));
    return x;
}

// Sum over the 64 lanes, in all of them.
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x) {
    const auto h = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    x = h[0] + h[1];
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = r[0] + r[1];
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, false);   // row_ror:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x122, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x121, 0xf, 0xf, false);
    return x;
}

}  // namespace mvla
