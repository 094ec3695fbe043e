// Arithmetic shared by the window bounds (tm_bound.hip) and the search that
// refines them (tm_search.hip): rounding up to float16, and the scales that
// keep window maxima and weights inside its range.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>

namespace tmlib {

constexpr int kWeightExp = 10;           // float16 weights carry w * 2^10
constexpr int kImageExp = 14;            // window maxima are scaled below 2^14
constexpr int kSearchWindows = 8;        // windows of shifts per template of the search

// Least A = max |P| with window bounds. From here on the scales of
// window_scale and the sums they undo are normal float32 numbers, and what
// the exact score loses to subnormal products (2^-150 each) is far below the
// bounds' margin; a fainter pattern is scored exhaustively.
constexpr float kFaint = 0x1p-100f;

// Powers of 2: P * image <= 2^kImageExp for |P| <= A (A >= kFaint), and the
// factor that takes a sum of scaled weights and maxima back.
struct WindowScale { float image, undo; };

__host__ __device__ __forceinline__ WindowScale window_scale(float A) {
    int e = 0;
    (void)frexpf(A, &e);                 // A = m 2^e, m in [0.5, 1)
    return {ldexpf(1.0f, kImageExp - e), ldexpf(1.0f, e - kImageExp - kWeightExp)};
}

// 1 / pn rounded up (0 for pn <= 0).
__host__ __device__ __forceinline__ float inverse_up(double pn) {
    if (!(pn > 0.0)) return 0.0f;
    const double ip = 1.0 / pn;
    const float f = static_cast<float>(ip);
    return static_cast<double>(f) < ip ? nextafterf(f, INFINITY) : f;
}

// Whether a pattern with intensities has no window bounds: too faint, 1 / ||P||
// (rounded either way, 0 for no norm) at the end of the range, past which its
// scores are infinite, or subnormal, or a norm that is not its own and so far
// off that the product of the bounds' factors (about A / ||P|| / 2^24) could
// leave the normal numbers.
__host__ __device__ __forceinline__ bool no_window_bounds(float A, float inv) {
    return A > 0.0f && (A < kFaint || inv > 0x1p127f ||
                        (inv > 0.0f && (inv < 0x1p-125f || !(A * inv >= 0x1p-40f && A * inv <= 0x1p100f))));
}

__host__ __device__ __forceinline__ float h2f(uint32_t bits16) {
    return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(bits16)));
}

// float16 bits of the smallest float16 >= x (x >= 0; past the range: inf).
__host__ __device__ __forceinline__ uint32_t f16_up(float x) {
    const _Float16 h = static_cast<_Float16>(x);
    uint16_t b = __builtin_bit_cast(uint16_t, h);
    if (static_cast<float>(h) < x) ++b;
    return b;
}

// n u / (1 - n u), u the unit roundoff of float32: bounds the relative error
// of n roundings in a row.
inline double gamma32(double n) {
    const double u = std::ldexp(1.0, -24);
    return n * u / (1.0 - n * u);
}

}  // namespace tmlib
