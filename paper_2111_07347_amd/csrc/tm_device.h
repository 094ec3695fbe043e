// Device helpers: 64-lane wavefront reductions and broadcasts.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace tmlib {

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Uniform (scalar) copy of a wave-uniform value.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// v combined over the wave's lanes by f, in all of them: along the rows of 16
// lanes, then across them (data-parallel moves of the vector unit; the LDS
// crossbar, which shuffles go through, takes ten times as long per step), read
// from the last lane. A lane without a partner combines its value with itself,
// so f(x, x) has to be x (a maximum or minimum).
template <typename F>
__device__ __forceinline__ int wave_fold(int v, F f) {
    auto step = [&](auto ctrl, auto rows) {
        v = f(v, __builtin_amdgcn_update_dpp(v, v, ctrl.value, rows.value, 0xf, false));
    };
    using std::integral_constant;
    step(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});    // row_shr:1
    step(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});    // row_shr:2
    step(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});    // row_shr:4
    step(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});    // row_shr:8
    step(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});    // row_bcast:15
    step(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});    // row_bcast:31
    return __builtin_amdgcn_readlane(v, 63);
}

// The wave's maximum (no NaN).
__device__ __forceinline__ float wave_max(float v) {
    return __int_as_float(wave_fold(__float_as_int(v), [](int x, int y) {
        return __float_as_int(fmaxf(__int_as_float(x), __int_as_float(y)));
    }));
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

__device__ __forceinline__ unsigned long long ballot(bool p) { return __ballot(p); }

// Orders a wave's LDS accesses across its lanes: what a lane wrote before
// is seen by the wave's reads after (the compiler may not move memory
// operations across it; the hardware keeps a wave's LDS operations in order).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace tmlib
