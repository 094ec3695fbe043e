// Pattern preprocessing before indexing (Section 4.1: the direct beam is
// centred, the diffuse background removed by a difference of Gaussians, the
// result smoothed by a Gaussian blur and low intensities set to zero; the
// discussion names parallelising these steps as an open optimisation).
//
//   centre_kernel  one workgroup per pattern: the maximum of the square box
//                  |x - W/2| <= r_box, |y - H/2| <= r_box, then the
//                  intensity-weighted centroid (float64) of the box pixels
//                  >= frac times that maximum.
//   filter_kernel  everything else in one pass over the pattern.
//
// Gaussians: exp(-t^2 / (2 sigma^2)) on |t| <= floor(4 sigma + 0.5),
// normalised in float64 on the host, applied in float32; mirror boundary
// (... c b a | a b c ...) by folding indices modulo 2n. A symmetric filter
// keeps that extension, so the blur of a difference of Gaussians is the
// difference of two separable filters, K1 = G(blur) G(min) and K2 = G(blur)
// G(max), whose taps are convolved in float64 on the host: one pass along x
// and one along y in all.
//
// filter_kernel: a workgroup of 4 waves owns 32 columns of a pattern and goes
// down its rows in blocks of 32. Per block the centred rows, out(x, y) = in(x +
// cx - W/2, y + cy - H/2) (bilinear, zero outside), are staged in LDS with
// mirrored halos; the correlations along x and y are products with banded
// Toeplitz matrices on the matrix cores (v_mfma_f32_16x16x4_f32: float32 in and
// out), one 16 x 16 tile per wave. Rows filtered along x wait in a ring until
// the reach of the filters along y is there. The Toeplitz operands are read
// from a zero-padded tap table in LDS (entry k - n), and rows outside the
// image are ring rows at the mirrored index. A 16-column tile of a filter of
// radius r takes 16 + 2 r products per output, against 2 r + 1 of the filter
// alone; the vector units' share is the staging.
// Measured (1024 uint16 patterns of 256 x 256, sigma 1 / 6 / 1, all steps):
// 478 us, 37 % of it matrix-core issue, against 1061 us of separate row and
// column passes for the difference and the blur on the vector units (ten image
// sizes of HBM traffic). Strips of 64 columns and 8 waves take 453 us, but
// their rings exceed the LDS at the largest reach.
//
// A zero tap still multiplies in a matrix product: non-finite pixels are
// staged as 0 and kept as bits of the columns that their reach along x covers;
// outputs that such a row reaches along y become infinite or NaN as the sum of
// positive taps times these pixels is, and the difference of two such sums.
#include <algorithm>
#include <cmath>

#include "tm_internal.h"

namespace {

constexpr int kMaxRadius = 64;            // sigma <= 15.9
constexpr int kMaxReach = 2 * kMaxRadius; // of a filter and the blur
constexpr int kThreads = 256;             // 4 waves: 2 x 2 tiles of 16 x 16
constexpr int kTile = 32;                 // columns of a strip, rows of a block
constexpr int kCentreThreads = 256;
constexpr int kXcds = 8;
constexpr int kMaxGrid = 1 << 22;         // workgroups of a launch

// A symmetric filter: its reach, that rounded up to a multiple of 4 (0 taps
// past the reach) and w[t], 0 <= t <= r.
struct Filter {
    int reach, r;
    float w[kMaxReach + 1];
};

__device__ __forceinline__ int mirror(int i, int n) {
    if (static_cast<unsigned>(i) < static_cast<unsigned>(n)) return i;
    if (i < 0 && i >= -n) return -i - 1;
    if (i >= n && i < 2 * n) return 2 * n - 1 - i;
    // images narrower than the halo: fold modulo the period 2n
    const int p = 2 * n;
    int j = i % p;
    if (j < 0) j += p;
    return j < n ? j : p - 1 - j;
}

template <typename Tin>
__global__ void __launch_bounds__(kCentreThreads)
centre_kernel(const Tin* __restrict__ patterns, int H, int W, int r_box, double frac,
              double* __restrict__ centre) {
    __shared__ double red[4][kCentreThreads / 64];
    const int b = blockIdx.x;
    const Tin* img = patterns + static_cast<size_t>(b) * H * W;
    const double x0 = 0.5 * W, y0 = 0.5 * H;
    const int xl = max(0, static_cast<int>(ceil(x0 - r_box))), xh = min(W - 1, static_cast<int>(floor(x0 + r_box)));
    const int yl = max(0, static_cast<int>(ceil(y0 - r_box))), yh = min(H - 1, static_cast<int>(floor(y0 + r_box)));
    const int bw = xh - xl + 1, n = (xh >= xl && yh >= yl) ? bw * (yh - yl + 1) : 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double m = -INFINITY;
    for (int i = threadIdx.x; i < n; i += kCentreThreads) {
        const int y = yl + i / bw, x = xl + i % bw;
        m = fmax(m, static_cast<double>(img[static_cast<size_t>(y) * W + x]));
    }
    for (int o = 32; o >= 1; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
    if (lane == 0) red[0][wave] = m;
    __syncthreads();
    m = red[0][0];
    for (int w = 1; w < kCentreThreads / 64; ++w) m = fmax(m, red[0][w]);
    __syncthreads();
    double s = 0.0, sx = 0.0, sy = 0.0;
    const double thr = frac * m;
    for (int i = threadIdx.x; i < n; i += kCentreThreads) {
        const int y = yl + i / bw, x = xl + i % bw;
        const double v = static_cast<double>(img[static_cast<size_t>(y) * W + x]);
        if (v >= thr) {
            s += v;
            sx += v * x;
            sy += v * y;
        }
    }
    for (int o = 32; o >= 1; o >>= 1) {
        s += __shfl_xor(s, o, 64);
        sx += __shfl_xor(sx, o, 64);
        sy += __shfl_xor(sy, o, 64);
    }
    if (lane == 0) {
        red[1][wave] = s;
        red[2][wave] = sx;
        red[3][wave] = sy;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double ts = 0.0, tx = 0.0, ty = 0.0;
        for (int w = 0; w < kCentreThreads / 64; ++w) {
            ts += red[1][w];
            tx += red[2][w];
            ty += red[3][w];
        }
        const bool ok = n > 0 && m > 0.0;
        centre[2 * b] = ok ? tx / ts : x0;
        centre[2 * b + 1] = ok ? ty / ts : y0;
    }
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Zero-padded taps of a filter for the Toeplitz operands: entry 15 + d holds
// tap d - r (0 <= d <= 2 r), zeros 15 deep on either side.
__host__ __device__ constexpr int table_len(int r) { return 2 * r + 1 + 30; }

// Rows of the ring: a block's filters along y run when the blocks that hold
// their reach are there, and still find the rows before the block.
__host__ __device__ constexpr int blocks_ahead(int r) { return (r + kTile - 1) / kTile; }
__host__ __device__ constexpr int ring_rows(int r) {
    return (kTile * (blocks_ahead(r) + 1) + r + kTile - 1) / kTile * kTile;
}

// Product of a 16 x (16 + 2 r) and a (16 + 2 r) x 16 operand (4 | r, an even
// number of steps of 4), one of them banded: from both ends of k toward the
// middle in two sums, so that the small taps are added first (less rounding)
// and two products are in flight. a(k) and b(k) point to a lane's element at
// k; SA and SB floats further (back) lies that of the next (last) step, which
// holds for b as far as `whole` says: whole(k, d) for the 4 steps from k in
// direction d.
template <int SA, int SB, typename FA, typename FB, typename FW>
__device__ __forceinline__ f32x4 banded(int r, FA a, FB b, FW whole) {
    f32x4 lo = {0.0f, 0.0f, 0.0f, 0.0f}, hi = lo;
    const int pairs = 2 + r / 4, e = 12 + 2 * r;
    int p = 0;
#pragma unroll 1
    for (; p + 4 <= pairs; p += 4) {
        const int k = 4 * p, l = e - 4 * p;
        if (!whole(k, 1) || !whole(l, -1)) break;
        const float *al = a(k), *bl = b(k), *ah = a(l), *bh = b(l);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            lo = __builtin_amdgcn_mfma_f32_16x16x4f32(al[SA * u], bl[SB * u], lo, 0, 0, 0);
            hi = __builtin_amdgcn_mfma_f32_16x16x4f32(ah[-SA * u], bh[-SB * u], hi, 0, 0, 0);
        }
    }
#pragma unroll 1
    for (; p < pairs; ++p) {
        lo = __builtin_amdgcn_mfma_f32_16x16x4f32(*a(4 * p), *b(4 * p), lo, 0, 0, 0);
        hi = __builtin_amdgcn_mfma_f32_16x16x4f32(*a(e - 4 * p), *b(e - 4 * p), hi, 0, 0, 0);
    }
    return lo + hi;
}

// Place of column n of a ring row: in odd rows the halves change places, so
// that the 2 rows that half a wave reads do not meet in an LDS bank.
__device__ __forceinline__ int ring_at(int row, int n) {
    return row * kTile + (n ^ ((row & 1) << 4));
}

// Floats of a staged row: rows 2 (mod 4) apart put the 16 x 2 elements that
// half a wave reads in different banks.
__host__ __device__ constexpr int staged_pitch(int R) { return (kTile + 2 * R) / 4 * 4 + 2; }

// TWO: out = K1 - K2, else K1 alone. Dynamic LDS: staged block, rings, tables,
// bits of non-finite pixels.
template <typename Tin, bool TWO>
__global__ void __launch_bounds__(kThreads, 4)
filter_kernel(const Tin* __restrict__ in, const double* __restrict__ centre, int B, int H, int W,
              int strips, Filter f1, Filter f2, bool thresh, float threshold,
              float* __restrict__ out) {
    extern __shared__ float lds[];
    // the strips of a pattern run on one XCD (workgroups go round the XCDs)
    const int q = blockIdx.x / kXcds;
    const int b = q / strips * kXcds + static_cast<int>(blockIdx.x) % kXcds;
    if (b >= B) return;
    const int x0 = (q % strips) * kTile;
    const int r1 = f1.r, r2 = TWO ? f2.r : 0, R = max(r1, r2);
    const int cols = kTile + 2 * R, cpitch = staged_pitch(R);
    const int ring = ring_rows(R), ahead = blocks_ahead(R);
    float* c = lds;                                   // [kTile][cpitch]
    float* ring1 = c + kTile * cpitch;                // [ring][kTile]
    float* ring2 = ring1 + ring * kTile;
    float* t1 = TWO ? ring2 + ring * kTile : ring2;
    float* t2 = t1 + table_len(r1);
    uint32_t* bad = reinterpret_cast<uint32_t*>(TWO ? t2 + table_len(r2) : t2);   // [ring][4], then any
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ti = wave >> 1, tj = wave & 1;          // this wave's tile
    const int m16 = lane & 15, k4 = lane >> 4;
    for (int i = tid; i < table_len(r1); i += kThreads) {
        const int d = abs(i - 15 - r1);
        t1[i] = d <= r1 ? f1.w[d] : 0.0f;
    }
    if (TWO)
        for (int i = tid; i < table_len(r2); i += kThreads) {
            const int d = abs(i - 15 - r2);
            t2[i] = d <= r2 ? f2.w[d] : 0.0f;
        }
    for (int i = tid; i <= 4 * ring; i += kThreads) bad[i] = 0u;
    const Tin* img = in + static_cast<size_t>(b) * H * W;
    // shift of the centred pattern: whole pixels and fractions
    const double dx = centre ? centre[2 * b] - 0.5 * W : 0.0;
    const double dy = centre ? centre[2 * b + 1] - 0.5 * H : 0.0;
    const double xf = floor(dx), yf = floor(dy);
    const float fx = static_cast<float>(dx - xf), fy = static_cast<float>(dy - yf);
    const int sx = static_cast<int>(fmax(fmin(xf, 1e6), -1e6));
    const int sy = static_cast<int>(fmax(fmin(yf, 1e6), -1e6));
    const int n_blocks = (H + kTile - 1) / kTile;
    constexpr int kRun = 8;                           // rows a thread stages in a column
    const float inv_cols = 1.0f / static_cast<float>(cols);
    float* dst = out + static_cast<size_t>(b) * H * W;
    for (int blk = 0; blk < n_blocks + ahead; ++blk) {
        if (blk < n_blocks) {
            // ---- stage: tasks of one column and kRun rows
            const int y0 = blk * kTile;
            if constexpr (sizeof(Tin) == 4) {
                __syncthreads();                      // the bits of this block's ring rows are free
                if (tid < 4 * kTile) bad[4 * (y0 % ring) + tid] = 0u;
                __syncthreads();
            }
            // all rows of the block inside the image: plain strides
            const bool inside = y0 + sy >= 0 && y0 + sy + kTile < H;
            for (int task = tid; task < cols * (kTile / kRun); task += kThreads) {
                const int g = static_cast<int>((static_cast<float>(task) + 0.5f) * inv_cols);
                const int i = task - g * cols;
                const int x = mirror(x0 - R + i, W) + sx, ya = y0 + g * kRun + sy;
                // a pair of neighbours inside the image and their weights
                const int xp = min(max(x, 0), max(W - 2, 0));
                const bool lo0 = x == xp && x < W, lo1 = x + 1 == xp, hi0 = x == xp + 1 && x < W, hi1 = x == xp && xp + 1 < W;
                const float wl = lo0 ? 1.0f - fx : lo1 ? fx : 0.0f, wh = hi0 ? 1.0f - fx : hi1 ? fx : 0.0f;
                // (byte offsets within a pattern fit 32 bits: H, W <= 8192)
                const int second = W > 1 ? 1 : 0;
                auto px = [&](int row, int o) {
                    return static_cast<float>(*reinterpret_cast<const Tin*>(
                        reinterpret_cast<const char*>(img) +
                        static_cast<uint32_t>(row * W + xp + o) * static_cast<uint32_t>(sizeof(Tin))));
                };
                float a[kRun + 1];
                auto blend = [&](float l, float h) {
                    if constexpr (sizeof(Tin) == 4) {     // a pixel without weight may be non-finite
                        l = wl != 0.0f ? l : 0.0f;
                        h = wh != 0.0f ? h : 0.0f;
                    }
                    return wl * l + wh * h;
                };
                if (inside) {
                    float l[kRun + 1], h[kRun + 1];
#pragma unroll
                    for (int u = 0; u <= kRun; ++u) {
                        l[u] = px(ya + u, 0);
                        h[u] = px(ya + u, second);
                    }
#pragma unroll
                    for (int u = 0; u <= kRun; ++u) a[u] = blend(l[u], h[u]);
                } else {
#pragma unroll
                    for (int u = 0; u <= kRun; ++u) {
                        const int row = min(max(ya + u, 0), H - 1);
                        const float v = blend(px(row, 0), px(row, second));
                        a[u] = ya + u >= 0 && ya + u < H ? v : 0.0f;
                    }
                }
                float* cp = c + g * kRun * cpitch + i;
#pragma unroll
                for (int u = 0; u < kRun; ++u) {
                    float v = fy != 0.0f ? (1.0f - fy) * a[u] + fy * a[u + 1] : a[u];
                    if (sizeof(Tin) == 4 && !(fabsf(v) <= 3.402823466e38f)) {
                        // columns n within the reach of filter f; +inf and
                        // -inf apart, NaN is both
                        uint32_t* row = &bad[4 * ((y0 + g * kRun + u) % ring)];
                        for (int f = 0; f < (TWO ? 2 : 1); ++f) {
                            const int d = f ? f2.reach : f1.reach;
                            const int n0 = max(0, i - R - d), n1 = min(kTile - 1, i - R + d);
                            if (n0 > n1) continue;
                            const uint32_t m = (0xffffffffu >> (31 - n1)) & (0xffffffffu << n0);
                            if (!(v <= 0.0f)) atomicOr(row + 2 * f, m);
                            if (!(v >= 0.0f)) atomicOr(row + 2 * f + 1, m);
                        }
                        bad[4 * ring] = 1u;
                        v = 0.0f;
                    }
                    cp[u * cpitch] = v;
                }
            }
            __syncthreads();
            // ---- along x: tile (ti, tj) of both filters
            const float* ca = c + (16 * ti + m16) * cpitch + 16 * tj + k4;
            auto along_x = [&](const float* t, int r) {
                const float *p = ca + (R - r), *w = t + 15 + k4 - m16;
                return banded<4, 4>(r, [&](int k) { return p + k; }, [&](int k) { return w + k; },
                                    [](int, int) { return true; });
            };
            const f32x4 a1 = along_x(t1, r1);
            f32x4 a2 = a1;
            if (TWO) a2 = along_x(t2, r2);
            const int slot = y0 % ring;               // blocks do not straddle the ring's end
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int o = ring_at(slot + 16 * ti + 4 * k4 + v, 16 * tj + m16);
                ring1[o] = a1[v];
                if (TWO) ring2[o] = a2[v];
            }
        }
        __syncthreads();
        if (blk < ahead) continue;
        // ---- along y: rows of block blk - ahead
        const int y0 = (blk - ahead) * kTile + 16 * ti;
        const int n = 16 * tj + m16;
        auto along_y = [&](const float* rg, const float* t, int r) {
            const float *w = t + 15 + k4 - m16, *lane_rg = rg + ring_at(k4, n);
            auto tap = [&](int k) { return w + k; };
            if (y0 >= r && y0 + 16 + r <= H) {        // uniform: no row is mirrored
                // (4 | r, y0 and the ring: the 4 rows of a step lie together)
                const int first = (y0 - r) % ring;
                auto slot = [&](int k) { return first + k - (first + k >= ring ? ring : 0); };
                return banded<4, 4 * kTile>(r, tap, [&](int k) { return lane_rg + slot(k) * kTile; },
                                             [&](int k, int d) { return d > 0 ? slot(k) + 12 < ring : slot(k) >= 12; });
            }
            // (the rows in question lie within a ring's length of this one)
            const int s0 = max(0, y0 - r) / ring * ring;
            return banded<4, 0>(r, tap, [&](int k) {
                int slot = mirror(y0 - r + k + k4, H) - s0;
                slot += slot < 0 ? ring : 0;
                slot -= slot >= ring ? ring : 0;
                return rg + ring_at(slot, n);
            }, [](int, int) { return false; });
        };
        f32x4 acc = along_y(ring1, t1, r1);
        if (TWO) acc -= along_y(ring2, t2, r2);
        const bool any_bad = sizeof(Tin) == 4 && bad[4 * ring] != 0u;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int y = y0 + 4 * k4 + v, x = x0 + n;
            float z = acc[v];
            if (any_bad && y < H) {
                auto reached = [&](int f, int reach) {
                    uint32_t pos = 0, neg = 0;
                    for (int d = -reach; d <= reach; ++d) {
                        const uint32_t* row = &bad[4 * (mirror(y + d, H) % ring) + 2 * f];
                        pos |= row[0];
                        neg |= row[1];
                    }
                    const float inf = __int_as_float(0x7f800000);
                    return ((pos >> n) & 1u ? inf : 0.0f) - ((neg >> n) & 1u ? inf : 0.0f);
                };
                z += reached(0, f1.reach);
                if (TWO) z -= reached(1, f2.reach);
            }
            if (thresh && z < threshold) z = 0.0f;
            if (y < H && x < W) dst[static_cast<size_t>(y) * W + x] = z;
        }
    }
}

// Normalised taps of G(sigma) in float64, w[r + t] for |t| <= r (sigma 0: the
// identity); returns r.
int gaussian(double sigma, double (&w)[2 * kMaxRadius + 1]) {
    const int r = sigma > 0.0 ? static_cast<int>(4.0 * sigma + 0.5) : 0;
    double s = 0.0;
    for (int i = -r; i <= r; ++i) s += w[i + r] = r ? std::exp(-static_cast<double>(i) * i / (2.0 * sigma * sigma)) : 1.0;
    for (int i = 0; i <= 2 * r; ++i) w[i] /= s;
    return r;
}

// The filter G(a) G(b).
Filter make_filter(double a, double b) {
    double u[2 * kMaxRadius + 1], v[2 * kMaxRadius + 1];
    const int ru = gaussian(a, u), rv = gaussian(b, v);
    Filter f{};
    f.reach = ru + rv;
    f.r = (f.reach + 3) & ~3;
    for (int t = 0; t <= f.reach; ++t) {
        double w = 0.0;
        for (int i = std::max(-ru, t - rv); i <= std::min(ru, t + rv); ++i) w += u[i + ru] * v[t - i + rv];
        f.w[t] = static_cast<float>(w);
    }
    return f;
}

template <typename Tin>
int run(const Tin* in, int B, int H, int W, const tm_preprocess_opts& o, float* out,
        double* centre_out, hipStream_t s) {
    const bool dog = o.sigma_max > 0.0;
    const Filter f1 = make_filter(dog ? o.sigma_min : 0.0, o.sigma_blur);
    const Filter f2 = dog ? make_filter(o.sigma_max, o.sigma_blur) : Filter{};
    double* cen = centre_out;
    tmlib::Scratch mem;
    if (!cen && o.r_box >= 0) mem.add(cen, 2 * static_cast<size_t>(B));
    const bool scratch = !centre_out && o.r_box >= 0;
    if (scratch)
        if (int r = mem.allocate(s)) return r;
    const int R = std::max(f1.r, f2.r), ring = ring_rows(R);
    const size_t lds = sizeof(float) *
                       (static_cast<size_t>(kTile) * staged_pitch(R) +
                        static_cast<size_t>(ring) * kTile * (dog ? 2 : 1) + table_len(f1.r) +
                        (dog ? table_len(f2.r) : 0) + 4 * ring + 1);
    auto kern = dog ? filter_kernel<Tin, true> : filter_kernel<Tin, false>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    const int strips = (W + kTile - 1) / kTile;
    const int chunk = kMaxGrid / (strips * kXcds) * kXcds;    // patterns of a launch
    for (int b0 = 0; e == hipSuccess && b0 < B; b0 += chunk) {
        const int n = std::min(chunk, B - b0);
        const Tin* cin = in + static_cast<size_t>(b0) * H * W;
        double* cc = cen ? cen + 2 * static_cast<size_t>(b0) : nullptr;
        if (cc)    // with r_box < 0 the box is empty and the centre is (W/2, H/2)
            hipLaunchKernelGGL(centre_kernel<Tin>, dim3(n), dim3(kCentreThreads), 0, s, cin, H, W,
                               o.r_box, o.frac, cc);
        hipLaunchKernelGGL(kern, dim3((n + kXcds - 1) / kXcds * kXcds * strips), dim3(kThreads), lds, s,
                           cin, o.r_box >= 0 ? cc : nullptr, n, H, W, strips, f1, f2,
                           static_cast<bool>(std::isfinite(o.threshold)), static_cast<float>(o.threshold),
                           out + static_cast<size_t>(b0) * H * W);
        e = hipGetLastError();
        if (b0 > B - chunk) break;                            // (b0 stays in int)
    }
    const int r = e == hipSuccess ? TM_OK : tmlib::hip_fail(e, "preprocess kernel launch");
    return scratch ? mem.release(s, r) : r;
}

}  // namespace

extern "C" int tm_preprocess(const void* patterns, tm_dtype dtype, int32_t B, int32_t H,
                             int32_t W, const tm_preprocess_opts* opts, float* out,
                             double* centre_out, void* hip_stream) {
    tmlib::clear_error();
    if (!opts) { tmlib::set_error("opts is NULL"); return TM_EINVAL; }
    if (B < 0) { tmlib::set_error("B=%d < 0", B); return TM_EINVAL; }
    if (H < 1 || W < 1 || H > 8192 || W > 8192) { tmlib::set_error("H=%d, W=%d outside [1, 8192]", H, W); return TM_EINVAL; }
    if (dtype != TM_U16 && dtype != TM_F32) { tmlib::set_error("unknown dtype %d", static_cast<int>(dtype)); return TM_EINVAL; }
    const tm_preprocess_opts& o = *opts;
    if (o.r_box > 4096) { tmlib::set_error("r_box=%d too large", o.r_box); return TM_EINVAL; }
    if (!std::isfinite(o.frac) || !std::isfinite(o.sigma_min) || !std::isfinite(o.sigma_max) ||
        !std::isfinite(o.sigma_blur) || o.sigma_min < 0.0 || o.sigma_max < 0.0 ||
        o.sigma_blur < 0.0 || std::isnan(o.threshold)) {
        tmlib::set_error("frac and sigmas must be finite, sigmas >= 0, threshold not NaN");
        return TM_EINVAL;
    }
    if (o.sigma_max > 0.0 && !(o.sigma_min < o.sigma_max)) {
        tmlib::set_error("difference of Gaussians needs sigma_min < sigma_max");
        return TM_EINVAL;
    }
    for (double sg : {o.sigma_min, o.sigma_max, o.sigma_blur}) {
        if (static_cast<int>(4.0 * sg + 0.5) > kMaxRadius) {
            tmlib::set_error("Gaussian sigma %g above %g (radius %d)", sg, (kMaxRadius - 0.5) / 4.0,
                             kMaxRadius);
            return TM_EINVAL;
        }
    }
    if (B > 0 && (!patterns || !out)) { tmlib::set_error("patterns and out must be non-NULL"); return TM_EINVAL; }
    if (int r = tmlib::require_device()) return r;
    if (B == 0) return TM_OK;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (dtype == TM_F32)
        return run(static_cast<const float*>(patterns), B, H, W, o, out, centre_out, s);
    return run(static_cast<const uint16_t*>(patterns), B, H, W, o, out, centre_out, s);
}
