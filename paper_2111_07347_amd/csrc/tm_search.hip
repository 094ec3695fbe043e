// Exact top-N search of a pattern by refinement of bounds, one workgroup per
// pattern (several for small batches).
//
// The result is the plain path's top-N, bit for bit: scores come from the same
// float32 sums in the same record order, and a (template, window of shifts)
// pair is left out only when an upper bound of its scores lies below a lower
// bound q of the N-th best score.
//
//   1. Window image. The circle of shifts is cut into W = 8 windows of w =
//      ceil(n / 8); M[j, x] = max(0, max of wlen columns from x), wlen = w + W w
//      - n, scaled and rounded up to float16. Entry (j, r) of the image in LDS
//      holds the W halves M[j, r + i w]: a pixel at column q w + r finds the
//      bounds of all windows in one entry, half i standing for window (i - q)
//      mod W (for i < q the column lies W w - n past the window's, which wlen
//      covers).
//   2. Seeds: the templates with the largest bounds at hand get the exact score
//      of their best window; the N-th best of these is q.
//   3. Templates whose bound reaches q, the largest bounds first, get their W
//      window bounds; the windows that reach q are scored exactly in batches,
//      and q rises with each batch.
//
// The bounds at hand are, by kind of search:
//   kQc     the window bounds of tm_bound.hip (dense libraries);
//   kAll    bounds of all templates from the image, kept in LDS (sparse
//           libraries, where that is little work);
//   kItems  the same for a listed part of the library (a pre-filter's).
//
// A template's window records are sorted by the sector q of their column.
// Window bounds of a few templates go W lanes to a template, lane o summing
// sector o's records for all windows (few per lane: their loads are in flight
// together); the all-template pass goes one template to a lane, 64 templates
// with alike sector counts to a chunk, so that the turn from halves to
// windows is the same in all lanes and costs nothing.
//
// What bounds it: wave instructions (about 40 thousand per pattern of a
// 4000-template FCC library, of which a third are the all-template pass) and
// the latency of short dependent phases, hidden by 16 to 32 waves per CU.
// Measured (256 x 256 patterns, top-5, search alone, before -> now; before:
// the plain scan, or the pre-filter's candidate scan): 16384 patterns x 2000
// FCC templates 8.3 -> 2.1 ms; 256 patterns 0.29 -> 0.14 ms; 1024 patterns x
// 20000 orthorhombic templates, BF16 pre-filter keeping a tenth, candidate
// pass 8.5 -> 1.7 ms; one pattern x 20000 templates against the certified
// passes after the bound kernel 0.42 -> 0.13 ms.
//
// Rigour in finite precision is that of tm_bound.hip: image and weights
// rounded up to float16 with exact products, float32 sums widened by 1 / (1 -
// gamma), the plain path's own rounding covered by the margin c_t A (the
// sum's first term). A pattern that is too faint for these scales
// (tm_window.h) is left to the plain scan.
#include <algorithm>
#include <array>
#include <climits>
#include <cmath>
#include <cstring>
#include <numeric>
#include <type_traits>

#include "tm_device.h"
#include "tm_internal.h"
#include "tm_topn.h"
#include "tm_window.h"

namespace {

using tmlib::f16_up;
using tmlib::gamma32;
using tmlib::h2f;
using tmlib::kWeightExp;

constexpr int W = tmlib::kSearchWindows; // windows of shifts per template
constexpr int kUnit = 4;                 // window records per unit (one 16-byte load)
constexpr int kExactPad = 8;             // exact records are padded to whole batches of 8
constexpr int kBatch = 64;               // candidates scored between updates of q
constexpr int kMaxWork = 128;            // largest batch (a histogram bin may hold more)
constexpr int kSeedPicks = 32;           // columns of Qc that seed the search, about
constexpr int kMaxSeeds = 256;           //   and at the most
constexpr int kPend = 32;                // columns of Qc per wave and round
constexpr int kSel = 256;                // listed columns per round (kAll, kItems)
constexpr uint32_t kDone = 0xffffu;      // a bound that is dealt with
constexpr double kSparse = 24;           // most records per template of a sparse library
constexpr double kItemsSparse = 150000;  // a list's pixels x shift slots from which a search pays:
constexpr double kItemsDense = 450000;   //   sparse and dense libraries (see search_items_pays)
constexpr int kAllTemplates = 32768;     // most templates bounded in the workgroup (2 bytes each)
constexpr int kAllSteps = 8192;          // and most steps of 64 records for that
constexpr int kBuildWaves = 8;           // waves that build the image (row buffers share the lists' LDS)
constexpr int kMaxRows = 1023;           // touched-row index: 10 bits
constexpr int kMaxCols = 12;             // columns per lane (n_theta <= 768)
constexpr int kFillGrid = 512;           // workgroups that fill the chip (two per CU)
constexpr size_t kThreePerCu = 53 * 1024;   // LDS of three workgroups per CU
constexpr size_t kTwoPerCu = 80 * 1024;  // and of two
constexpr double kWindowCost = 8;        // wave instructions of a window per record
constexpr double kWindowMore = 150;      //   and besides, about
constexpr int kMinGive = 64;             // windows scored before a pattern is given up,
constexpr int kMaxGive = 160;            //   at the least and at the most (of a small batch)
constexpr size_t kMaxLds = 159 * 1024;   // of a workgroup, static part apart
constexpr int kSplitGrid = 128;          // workgroups up to which a pattern is split
constexpr int kMaxParts = 16;            // workgroups per pattern of a small batch
constexpr int kPartColumns = 2048;       // columns that are worth a workgroup

enum Kind { kQc, kAll, kItems };

// Candidate list of a workgroup: what one round may add, and the picks.
constexpr int entries(Kind kind, int nw) { return kind == kQc ? nw * kPend + kMaxSeeds : kSel; }

struct SearchArgs {
    const float* polar;
    const double* norms;
    const int* rows;                     // null: polar holds the touched rows only
    int Rs, n, n_rows, w, wlen, scr;
    int pitch;                           // floats of an LDS row of intensities (two turns)
    const uint4* recs;                   // window records, 4 per unit
    const uint4* head;                   // per column: first unit, margin factor x 2^10, units
                                         // per sector (8 bits each)
    const uint2* xrecs;                  // exact records: row and column, weight
    const int2* xhead;                   // [Tp] first exact record and their number (padded)
    const int* tid;                      // template of a column, -1 none
    const int* col;                      // [Tp] column of a template
    float dfac;
    const float* amax;                   // kQc: [B] max |P| over the touched rows
    const float* Qc;                     // kQc: bounds [B, n_cs], and per pattern n_list large
    int n_cs, n_valid;                   //   ones with their columns
    const float* lq;
    const int* lc;
    int n_list;
    const uint32_t* drecs;               // kAll: records by step and lane
    const uint4* dchunk;                 //   per 64 columns: first step, steps per sector
    int n_chunks;
    const int* items;                    // kItems: templates [B, n_items], ascending
    int n_items;
    int lists_end;                       // LDS entries (16 bytes) of image and lists
    int Tp, N, parts;
    int* give;                           // [B, parts]: set where the search is given up after
    int give_up;                         //   more than give_up windows
    int* top_t;                          // [B, parts, N]
    int* top_s;
    float* top_q;
};

struct Ctl {
    int cnt;                             // candidates listed
    int live, maxu, cut, work;           // selection of a batch
    int windows;                         // windows scored in it
    float q;                             // lower bound of the N-th best score
    int hist[64];
};

// LDS behind the image: lists and selection state; the image is built with
// row buffers in the same place.
template <Kind KIND, int NW>
struct Lists {
    uint2 ent[entries(KIND, NW)];        // template; float16 bound | window mask << 16
    uint4 work[kMaxWork];                // a batch: template, first record, records, windows;
                                         // then template, shift, score
    uint16_t pend[KIND == kQc ? NW * kPend : kSel];   // columns waiting for their bounds
    Ctl ctl;
};

// Suffix sums over a histogram of 64 bins (one wave): the highest bin from
// which on there are at least `want` entries, 0 if there is none.
__device__ __forceinline__ int cut_bin(const int* hist, int want, int lane) {
    int x = hist[lane];
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_down(x, d, 64);
        if (lane + d < 64) x += up;
    }
    const unsigned long long m = tmlib::ballot(x >= want);
    return m ? 63 - __clzll(static_cast<long long>(m)) : 0;
}

// Place of this lane in a list that takes one entry of every lane with
// `take` (a counter in LDS).
__device__ __forceinline__ int place(int* counter, bool take, int lane) {
    const unsigned long long m = tmlib::ballot(take);
    if (!m) return 0;
    int base = 0;
    if (lane == 0) base = atomicAdd(counter, __popcll(m));
    return __builtin_amdgcn_readfirstlane(base) + __popcll(m & ((1ull << lane) - 1));
}

// Exact records c .. c + 63 of a template, one per lane: column and offset of
// the row (in polar, or in the LDS rows), weight.
template <bool LROWS>
__device__ __forceinline__ uint2 exact_records(const SearchArgs& a, int r0, int nr, int c, int lane) {
    uint2 x = make_uint2(0u, 0u);
    if (c + lane < nr) x = a.xrecs[r0 + c + lane];
    const uint32_t k = x.x & 1023u, crow = (x.x >> 10) & 1023u;
    if constexpr (LROWS) return make_uint2(crow * static_cast<uint32_t>(a.pitch) + k, x.y);
    const uint32_t row = a.rows ? x.x >> 20 : crow;
    return make_uint2(row * static_cast<uint32_t>(a.n) << 10 | k, x.y);
}

// Exact best score of a template (records r0 .. r0 + nr - 1, the first 64 in
// `first`) over the windows of mask (all uniform): lanes are shifts, the sum
// of every shift in record order as in the plain path. Returns the raw
// maximum (before 1 / ||P||) and its smallest shift. The records come 64 at a
// time, one per lane in one load, and go to all lanes through scalar
// registers (scalar loads would be waited for batch by batch).
// With rows of two turns in LDS the shifts of all windows fill the lanes and
// no column wraps.
__device__ __forceinline__ float exact_lds(const SearchArgs& a, const float* __restrict__ rows,
                                           int r0, int nr, uint2 first, unsigned mask, int lane,
                                           int& best_s) {
    const int total = __popc(mask) * a.w;
    const float inv = 1.0f / static_cast<float>(a.w);
    float bm = -INFINITY;
    int bs = INT_MAX;
#pragma unroll 1
    for (int v0 = 0; v0 < total; v0 += 64) {
        const int v = v0 + lane;
        const int wi = static_cast<int>((static_cast<float>(v) + 0.5f) * inv);
        int S = 0, i = 0;
        for (unsigned m = mask; m; m &= m - 1, ++i)
            if (wi == i) S = __ffs(static_cast<int>(m)) - 1;
        const int sh = S * a.w + v - wi * a.w;
        const bool ok = v < total && sh < a.n;
        const float* p = rows + (ok ? sh : 0);
        float acc = 0.0f;
#pragma unroll 1
        for (int c = 0; c < nr; c += 64) {
            const uint2 x = c == 0 ? first : exact_records<true>(a, r0, nr, c, lane);
            const int m = min(64, nr - c);           // a multiple of kExactPad
#pragma unroll 1
            for (int u0 = 0; u0 < m; u0 += kExactPad) {
                float y[kExactPad];
#pragma unroll
                for (int u = 0; u < kExactPad; ++u) y[u] = p[__builtin_amdgcn_readlane(x.x, u0 + u)];
#pragma unroll
                for (int u = 0; u < kExactPad; ++u)
                    acc = fmaf(__uint_as_float(__builtin_amdgcn_readlane(x.y, u0 + u)), y[u], acc);
            }
        }
        if (ok && acc > bm) {
            bm = acc;
            bs = sh;
        }
    }
    const float wm = tmlib::wave_max(bm);
    best_s = tmlib::wave_fold(bm == wm ? bs : INT_MAX, [](int x, int y) { return min(x, y); });
    return wm;
}

// The same from polar, V windows at a time (their first shifts sh0): the
// intensities of a batch of records are in flight while the one before is
// summed.
template <int V>
__device__ __forceinline__ void exact_windows(const SearchArgs& a, const float* __restrict__ src, int r0,
                                              int nr, uint2 first, const int (&sh0)[V], int lane,
                                              float& best, int& bs) {
    constexpr int NB = V == 1 ? 8 : 4;           // records per batch
#pragma unroll 1
    for (int d0 = 0; d0 < a.w; d0 += 64) {       // (windows of more than 64 shifts: n > 512)
        const int d = d0 + lane;
        const int dl = d < a.w ? d : 0;
        float acc[V];
#pragma unroll
        for (int k = 0; k < V; ++k) acc[k] = 0.0f;
#pragma unroll 1
        for (int c = 0; c < nr; c += 64) {
            const uint2 x = c == 0 ? first : exact_records<false>(a, r0, nr, c, lane);
            const int m = min(64, nr - c);       // a multiple of kExactPad
            auto load = [&](int u0, float (&p)[NB][V]) {
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const uint32_t y = __builtin_amdgcn_readlane(x.x, u0 + u);
#pragma unroll
                    for (int k = 0; k < V; ++k) {
                        int c0 = static_cast<int>(y & 1023u) + sh0[k];  // first column, mod n
                        c0 -= c0 >= a.n ? a.n : 0;
                        const int turn = a.n - c0;                      // shifts before the wrap
                        p[u][k] = (src + (y >> 10) + c0)[dl >= turn ? dl - a.n : dl];
                    }
                }
            };
            auto sum = [&](int u0, const float (&p)[NB][V]) {
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const float w = __uint_as_float(__builtin_amdgcn_readlane(x.y, u0 + u));
#pragma unroll
                    for (int k = 0; k < V; ++k) acc[k] = fmaf(w, p[u][k], acc[k]);
                }
            };
            float pa[NB][V], pb[NB][V];
            load(0, pa);
#pragma unroll 1
            for (int u = 0; u < m; u += 2 * NB) {
                if (u + NB < m) load(u + NB, pb);
                sum(u, pa);
                if (u + NB >= m) break;
                if (u + 2 * NB < m) load(u + 2 * NB, pa);
                sum(u + NB, pb);
            }
        }
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const float v = d < a.w && sh0[k] + d < a.n ? acc[k] : -INFINITY;
            const float wm = tmlib::wave_max(v);
            const int s = sh0[k] + d0 + __ffsll(static_cast<long long>(tmlib::ballot(v == wm))) - 1;
            if (wm > best || (wm == best && s < bs)) {
                best = wm;
                bs = s;
            }
        }
    }
}

__device__ __forceinline__ float exact_polar(const SearchArgs& a, const float* __restrict__ src,
                                             int r0, int nr, uint2 first, unsigned mask, int lane,
                                             int& best_s) {
    float best = -INFINITY;
    int bs = INT_MAX;
#pragma unroll 1
    while (mask) {
        const int lowest = (__ffs(static_cast<int>(mask)) - 1) * a.w;
        const unsigned rest = mask & (mask - 1);
        if (!rest) {
            const int sh0[1] = {lowest};
            exact_windows<1>(a, src, r0, nr, first, sh0, lane, best, bs);
            break;
        }
        int sh0[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {            // past the last window: the lowest again
            sh0[k] = mask ? (__ffs(static_cast<int>(mask)) - 1) * a.w : lowest;
            mask &= mask - 1;
        }
        exact_windows<4>(a, src, r0, nr, first, sh0, lane, best, bs);
    }
    best_s = bs;
    return best;
}

// x[i] = x[i + D] (mod W) in the lanes with bit D of o.
template <int D>
__device__ __forceinline__ void turn(float (&x)[W], int o) {
    float y[W];
#pragma unroll
    for (int i = 0; i < W; ++i) y[i] = (o & D) ? x[(i + D) & (W - 1)] : x[i];
#pragma unroll
    for (int i = 0; i < W; ++i) x[i] = y[i];
}

// Lanes o and o ^ D add up the D values that lane o keeps (the upper ones
// with bit D).
template <int D>
__device__ __forceinline__ void exchange(float (&x)[W], int o) {
#pragma unroll
    for (int i = 0; i < D; ++i) {
        const float keep = (o & D) ? x[i + D] : x[i];
        const float give = (o & D) ? x[i] : x[i + D];
        x[i] = keep + __shfl_xor(give, D, 64);
    }
}

// Sum of the 8 bytes of x.
__device__ __forceinline__ int byte_sum(unsigned long long x) {
    x = (x & 0x00ff00ff00ff00ffull) + ((x >> 8) & 0x00ff00ff00ff00ffull);
    return static_cast<int>((x * 0x0001000100010001ull) >> 48);
}

// The W halves of an image entry times a weight, added to acc; half i goes to
// acc[i - o mod W].
__device__ __forceinline__ void add_entry(const uint4* __restrict__ img, uint32_t rec, int o,
                                          float (&acc)[W]) {
    const float w = h2f(rec >> 16);
    const uint4 x = img[rec & 0xffffu];
    const uint32_t v[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int i = 0; i < W; ++i)
        acc[(i - o) & (W - 1)] = fmaf(w, h2f(i & 1 ? v[i >> 1] >> 16 : v[i >> 1]), acc[(i - o) & (W - 1)]);
}

// Window sums of the templates of 64 / W columns per wave, W lanes each (col
// < 0: none): lane o of a template sums the records of sector o for all
// windows (half i of an entry: window i - o), then the lanes' sums are turned
// by o and reduced so that lane S ends with window S's, margin included,
// still scaled.
__device__ __forceinline__ float window_sum(const SearchArgs& a, const uint4* __restrict__ img,
                                            int col, float Ahat, int lane) {
    const int o = lane & (W - 1);
    int nu = 0;
    const uint4* p = a.recs;
    float init = 0.0f;
    if (col >= 0) {
        const uint4 h = a.head[col];
        const unsigned long long c = static_cast<unsigned long long>(h.w) << 32 | h.z;
        nu = static_cast<int>(c >> (8 * o)) & 255;
        p += static_cast<int>(h.x) + byte_sum(c & ((1ull << (8 * o)) - 1));
        if (o == 0) init = __uint_as_float(h.y) * Ahat;
    }
    float acc[W];
#pragma unroll
    for (int i = 0; i < W; ++i) acc[i] = init;
    constexpr int kAhead = 2;                    // units loaded together
#pragma unroll 1
    for (int i = 0; tmlib::ballot(i < nu); i += kAhead) {
        uint4 r[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            r[k] = make_uint4(0u, 0u, 0u, 0u);
            if (i + k < nu) r[k] = p[i + k];
        }
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            if (k > 0 && !tmlib::ballot(i + k < nu)) break;   // uniform
            add_entry(img, r[k].x, 0, acc);
            add_entry(img, r[k].y, 0, acc);
            add_entry(img, r[k].z, 0, acc);
            add_entry(img, r[k].w, 0, acc);
        }
    }
    // window S from half (S + o) mod W, then halve the windows held with each
    // exchange: lane S ends with window S
    turn<4>(acc, o);
    turn<2>(acc, o);
    turn<1>(acc, o);
    exchange<4>(acc, o);
    exchange<2>(acc, o);
    exchange<1>(acc, o);
    return acc[0];
}

// Largest window sums of the 64 templates of a chunk, one per lane.
__device__ __forceinline__ float max_window(const SearchArgs& a, const uint4* __restrict__ img,
                                            int chunk, float Ahat, int lane) {
    const uint4 h = a.dchunk[chunk];
    const uint32_t* p = a.drecs + static_cast<size_t>(h.x) * 64 + lane;
    const float init = __uint_as_float(a.head[chunk * 64 + lane].y) * Ahat;
    float acc[W];
#pragma unroll
    for (int S = 0; S < W; ++S) acc[S] = init;
    uint32_t r0 = p[0], r1 = p[64], r2 = p[128], r3 = p[192];   // four steps ahead
    p += 256;
#pragma unroll
    for (int o = 0; o < W; ++o) {
        const int m = static_cast<int>((o < 4 ? h.z : h.w) >> (8 * (o & 3))) & 255;
#pragma unroll 1
        for (int i = 0; i < m; ++i) {
            const uint32_t rec = r0;
            r0 = r1;
            r1 = r2;
            r2 = r3;
            r3 = *p;
            p += 64;
            add_entry(img, rec, o, acc);
        }
    }
    float m = acc[0];
#pragma unroll
    for (int S = 1; S < W; ++S) m = fmaxf(m, acc[S]);
    return m;
}

// LROWS: the touched rows' intensities stay in LDS (two turns each).
template <Kind KIND, int NW, int MC, bool LROWS>
__global__ void __launch_bounds__(NW * 64, 8)
search_kernel(const SearchArgs a) {
    extern __shared__ uint4 smem[];
    __shared__ float red[NW];
    constexpr int NT = NW * 64;
    constexpr int G = 64 / W;                // templates per wave and evaluation
    constexpr int kEntries = entries(KIND, NW);
    uint4* img = smem;
    Lists<KIND, NW>& L = *reinterpret_cast<Lists<KIND, NW>*>(smem + a.n_rows * a.w);
    Ctl& C = L.ctl;
    // behind the lists: the rows, then the bounds at hand
    float* lrows = reinterpret_cast<float*>(smem + a.lists_end);
    uint16_t* ub = reinterpret_cast<uint16_t*>(lrows + (LROWS ? a.n_rows * a.pitch : 0));
    const int b = blockIdx.x, part = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = tmlib::uniform(tid >> 6);
    const int n = a.n, N = a.N;
    const float* src = a.polar + static_cast<size_t>(b) * a.Rs * n;
    const size_t o_out = (static_cast<size_t>(b) * a.parts + part) * N;
    const double pn = a.norms[b];
    // a non-finite norm: flagged as the plain path flags it
    if ((__double_as_longlong(pn) & 0x7ff0000000000000LL) == 0x7ff0000000000000LL) {
        for (int i = tid; i < N; i += NT) {
            a.top_t[o_out + i] = -1;
            a.top_s[o_out + i] = -1;
            a.top_q[o_out + i] = __int_as_float(0x7fc00000);
        }
        if (tid == 0) a.give[b * a.parts + part] = 0;
        return;
    }
    const float invP = pn > 0.0 ? static_cast<float>(1.0 / pn) : 0.0f;
    // A = max |P| over the touched rows
    float A = 0.0f;
    if constexpr (KIND != kQc) {
        for (int r0 = wave; r0 < a.n_rows; r0 += 2 * NW) {
            float v[2][MC];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int r = min(r0 + k * NW, a.n_rows - 1);
                const float* row = src + static_cast<size_t>(a.rows ? a.rows[r] : r) * n;
#pragma unroll
                for (int i = 0; i < MC; ++i) v[k][i] = lane + 64 * i < n ? row[lane + 64 * i] : 0.0f;
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int r = r0 + k * NW;
#pragma unroll
                for (int i = 0; i < MC; ++i) {
                    A = fmaxf(A, fabsf(v[k][i]));
                    const int c = lane + 64 * i;
                    if (LROWS && c < n && r < a.n_rows) {
                        lrows[r * a.pitch + c] = v[k][i];
                        lrows[r * a.pitch + n + c] = v[k][i];
                    }
                }
            }
        }
        A = tmlib::wave_max(A);
        if (lane == 0) red[wave] = A;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < NW; ++w) A = fmaxf(A, red[w]);
        __syncthreads();
    } else {
        A = a.amax[b];
    }
    // no intensity on the touched rows, or 1 / ||P|| = 0: every score is 0 and
    // the ranking goes by template index, so that the first N are the answer
    const bool flat = !(A > 0.0f) || invP == 0.0f;
    // no bounds at this scale: left to the plain scan
    if (!flat && tmlib::no_window_bounds(A, invP)) {
        if (tid == 0) a.give[b * a.parts + part] = 1;
        return;
    }
    float scale = 1.0f;
    if (!flat) {
        scale = tmlib::window_scale(A).image;
        // ---- the window image, row by row: clamped, scaled, rounded-up
        // float16 values of a row and a halo of H columns in rb, maxima of its
        // aligned blocks of o columns in bm; lane l takes the o columns from
        // x0 = o l: the part that all their windows share, then suffix maxima
        // of the head and prefix maxima of the tail
        const int o = (n + 63) / 64;
        const int H = a.wlen + o, nb = (n + H) / o;
        const int q = (a.wlen - o) / o, rq = a.wlen - o - q * o;
        uint16_t* rb = reinterpret_cast<uint16_t*>(&L) + static_cast<size_t>(wave) * a.scr;
        uint16_t* bm = rb + n + H;
        const uint32_t magic = (1u << 20) / a.w + 1;   // x / w for x < 800
        auto load_row = [&](int rr, float (&v)[MC]) {
            const int r = min(rr, a.n_rows - 1);
            const float* row = src + static_cast<size_t>(a.rows ? a.rows[r] : r) * n;
#pragma unroll
            for (int i = 0; i < MC; ++i) v[i] = lane + 64 * i < n ? row[lane + 64 * i] : 0.0f;
        };
        auto build_row = [&](int r, const float (&v)[MC]) {
#pragma unroll
            for (int i = 0; i < MC; ++i) {
                const int c = lane + 64 * i;
                if (c < n) {
                    const uint16_t h = static_cast<uint16_t>(f16_up(fmaxf(v[i], 0.0f) * scale));
                    rb[c] = h;
                    if (c < H) rb[n + c] = h;
                }
            }
            tmlib::wave_sync();
            for (int k = lane; k < nb; k += 64) {
                uint32_t m = 0;
                for (int d = 0; d < o; ++d) m = max(m, static_cast<uint32_t>(rb[k * o + d]));
                bm[k] = static_cast<uint16_t>(m);
            }
            tmlib::wave_sync();
            uint16_t* dst = reinterpret_cast<uint16_t*>(img + r * a.w);
            const int x0 = o * lane;
            if (x0 < n) {
                uint32_t hv[MC], tv[MC];
#pragma unroll
                for (int d = 0; d < MC; ++d) {
                    hv[d] = rb[x0 + min(d, o - 1)];
                    tv[d] = rb[x0 + a.wlen - 1 + min(max(d, 1), o - 1)];
                }
                uint32_t common = hv[MC - 1];
                for (int k = 1; k <= q; ++k) common = max(common, static_cast<uint32_t>(bm[lane + k]));
                for (int k = 0; k < rq; ++k)
                    common = max(common, static_cast<uint32_t>(rb[x0 + o * (q + 1) + k]));
                uint32_t out[MC];
                uint32_t hmax = common, tmax = common;
#pragma unroll
                for (int d = MC - 1; d >= 0; --d) {
                    if (d < o - 1) hmax = max(hmax, hv[d]);
                    out[d] = hmax;
                }
#pragma unroll
                for (int d = 1; d < MC; ++d) {
                    if (d < o) tmax = max(tmax, tv[d]);
                    out[d] = max(out[d], tmax);
                }
#pragma unroll
                for (int d = 0; d < MC; ++d) {
                    const int x = x0 + d;
                    if (d < o && x < n) {
                        const int i = static_cast<int>((static_cast<uint32_t>(x) * magic) >> 20);
                        dst[(x - i * a.w) * W + i] = static_cast<uint16_t>(out[d]);
                        // columns past n (W w > n) repeat the first ones
                        const int y = x + n;
                        if (y < W * a.w) {
                            const int iy = static_cast<int>((static_cast<uint32_t>(y) * magic) >> 20);
                            dst[(y - iy * a.w) * W + iy] = static_cast<uint16_t>(out[d]);
                        }
                    }
                }
            }
            tmlib::wave_sync();
        };
        // the next row is in flight while one is worked on (loads past the
        // last row repeat it)
        float va[MC], vb[MC];
        if (wave < kBuildWaves) load_row(wave, va);
#pragma unroll 1
        for (int r = wave < kBuildWaves ? wave : a.n_rows; r < a.n_rows; r += 2 * kBuildWaves) {
            load_row(r + kBuildWaves, vb);
            build_row(r, va);
            if (r + kBuildWaves >= a.n_rows) break;
            load_row(r + 2 * kBuildWaves, va);
            build_row(r + kBuildWaves, vb);
        }
    }
    __syncthreads();
    const float Ahat = h2f(f16_up(A * scale));
    // bound = sum to_q, to_q = out_scale dfac invP_up (1 + 2^-18), out_scale the
    // inverse of the scales, a power of 2: the last factor more than restores
    // the roundings (of normal numbers: see no_window_bounds)
    const float to_q = a.dfac * tmlib::inverse_up(pn) * (1.0f + 0x1p-18f) / (scale * static_cast<float>(1 << kWeightExp));
    if (tid == 0) {
        C.cnt = flat && part == 0 ? N : 0;
        C.q = -INFINITY;
    }
    if (flat && tid < N) {
        int t = tid;
        if constexpr (KIND == kItems) t = a.items[static_cast<size_t>(b) * a.n_items + tid];
        L.ent[tid] = make_uint2(static_cast<uint32_t>(t), ((1u << W) - 1) << 16);
    }
    __syncthreads();
    // Window bounds of the templates of G columns; those that reach q are
    // listed with their windows (seed: with the best window alone, whatever q).
    auto evaluate = [&](int col, bool seed) {
        const int t = col >= 0 ? a.tid[col] : -1;
        const float u = window_sum(a, img, col, Ahat, lane) * to_q;
        float U = u;
#pragma unroll
        for (int d = W / 2; d >= 1; d >>= 1) U = fmaxf(U, __shfl_xor(U, d, 64));
        const unsigned long long hit = tmlib::ballot(seed ? u == U : u >= C.q);
        unsigned mask = static_cast<unsigned>(hit >> (lane & ~(W - 1))) & ((1u << W) - 1);
        if (seed) mask &= 0u - mask;
        const bool take = t >= 0 && mask != 0 && (lane & (W - 1)) == 0;
        const int at = place(&C.cnt, take, lane);
        if (take && at < kEntries)
            L.ent[at] = make_uint2(static_cast<uint32_t>(t), f16_up(fmaxf(U, 0.0f)) | (mask << 16));
    };
    int windows = 0;                             // scored in the last batch
    // The live candidates (bound >= q) with the largest bounds, at least
    // `want` of them if there are so many and at most kMaxWork, scored
    // exactly: their number (0: none live). All threads call; ends with the
    // results in place.
    auto score_batch = [&](int want) -> int {
        const int cnt = min(C.cnt, kEntries);
        const float q = C.q;
        __syncthreads();
        if (tid < 64) C.hist[tid] = 0;
        if (tid == 0) {
            C.live = 0;
            C.maxu = 0;
            C.cut = 0;
            C.work = 0;
            C.windows = 0;
        }
        __syncthreads();
        int live = 0, mu = 0;
        for (int i = tid; i < cnt; i += NT) {
            const uint32_t y = L.ent[i].y;
            if ((y >> 16) && h2f(y) >= q) {
                ++live;
                mu = max(mu, static_cast<int>(y & 0xffffu));
            }
        }
        if (live) {
            atomicAdd(&C.live, live);
            atomicMax(&C.maxu, mu);
        }
        __syncthreads();
        live = C.live;
        if (live == 0) return 0;
        const int lo = q > 0.0f ? static_cast<int>(__builtin_bit_cast(uint16_t, static_cast<_Float16>(q))) : 0;
        const float range = 63.0f / static_cast<float>(max(1, C.maxu - lo));
        auto bin = [&](uint32_t y) {
            return min(63, max(0, static_cast<int>(static_cast<float>(static_cast<int>(y & 0xffffu) - lo) * range)));
        };
        if (live > want) {
            for (int i = tid; i < cnt; i += NT) {
                const uint32_t y = L.ent[i].y;
                if ((y >> 16) && h2f(y) >= q) atomicAdd(&C.hist[bin(y)], 1);
            }
            __syncthreads();
            if (wave == 0) {
                const int c = cut_bin(C.hist, want, lane);
                if (lane == 0) C.cut = c;
            }
            __syncthreads();
        }
        const int cut = C.cut;
        for (int i0 = 0; i0 < cnt; i0 += NT) {
            const int i = i0 + tid;
            const uint32_t y = i < cnt ? L.ent[i].y : 0u;
            const bool take = (y >> 16) && h2f(y) >= q && bin(y) >= cut;
            const int at = place(&C.work, take, lane);
            if (take && at < kMaxWork) {
                const int t = static_cast<int>(L.ent[i].x);
                const int2 h = a.xhead[t];
                L.work[at] = make_uint4(static_cast<uint32_t>(t), static_cast<uint32_t>(h.x),
                                        static_cast<uint32_t>(h.y), y >> 16);
                L.ent[i].y = y & 0xffffu;        // done
            }
        }
        __syncthreads();
        const int nw = min(C.work, kMaxWork);
        // the next template's records are loaded while one is scored
        auto item = [&](int i, int& r0, int& nr) {
            const uint4 x = L.work[min(i, kMaxWork - 1)];
            r0 = tmlib::uniform(static_cast<int>(x.y));
            nr = i < nw ? tmlib::uniform(static_cast<int>(x.z)) : 0;
            return static_cast<unsigned>(tmlib::uniform(static_cast<int>(x.w)));
        };
        int r0, nr;
        unsigned mask = item(wave, r0, nr);
        uint2 rec = exact_records<LROWS>(a, r0, nr, 0, lane);
#pragma unroll 1
        for (int i = wave; i < nw; i += NW) {
            int r1, nr1;
            const unsigned mask1 = item(i + NW, r1, nr1);
            const uint2 rec1 = exact_records<LROWS>(a, r1, nr1, 0, lane);
            int s = 0;
            float wm;
            if constexpr (LROWS)
                wm = exact_lds(a, lrows, r0, nr, rec, mask, lane, s);
            else
                wm = exact_polar(a, src, r0, nr, rec, mask, lane, s);
            if (lane == 0) {
                atomicAdd(&C.windows, __popc(mask));
                L.work[i].y = static_cast<uint32_t>(s);
                L.work[i].z = __float_as_uint(wm * invP);
            }
            r0 = r1;
            nr = nr1;
            mask = mask1;
            rec = rec1;
        }
        __syncthreads();
        windows = C.windows;
        return nw;
    };
    tmlib::TopState st = tmlib::topn_init();     // wave 0's list
    const int n_seed_scored = min(kMaxWork, max(16, (2 * N + 15) & ~15));
    // Scores the candidates listed; seeds only set q. A pattern with very
    // many candidates (hardly any structure, or a threshold that many
    // templates reach) is given up: a plain scan of all its templates by
    // many workgroups costs less than going on here.
    int scored = 0;
    bool gone = false;
    auto drain = [&](bool seed) {
#pragma unroll 1
        for (;;) {
            const int nw = score_batch(seed ? n_seed_scored : kBatch);
            if (nw == 0) break;
            if (wave == 0 && seed && nw >= N) {
                // the N-th best (every lane ranks up to two results)
#pragma unroll
                for (int h = 0; h < kMaxWork / 64; ++h) {
                    const int i = lane + 64 * h;
                    if (i < nw) {
                        const float Q = __uint_as_float(L.work[i].z);
                        int rank = 0;
                        for (int j = 0; j < nw; ++j) {
                            const float x = __uint_as_float(L.work[j].z);
                            rank += (x > Q || (x == Q && j < i)) ? 1 : 0;
                        }
                        if (rank == N - 1) C.q = Q;
                    }
                }
            }
            if (wave == 0 && !seed) {
                for (int i = 0; i < nw; ++i) {
                    const uint4 x = L.work[i];
                    const float Q = __uint_as_float(x.z);
                    const int t = static_cast<int>(x.x);
                    if (st.cnt < N || tmlib::topn_beats(st, Q, t))
                        tmlib::topn_insert(st, Q, t, static_cast<int>(x.y), lane, N);
                }
                if (lane == 0 && st.cnt == N && st.thr > C.q) C.q = st.thr;
            }
            __syncthreads();
            if (seed) break;
            scored += windows;
            if (scored > a.give_up) {
                gone = true;
                break;
            }
        }
        __syncthreads();
        if (tid == 0) C.cnt = 0;
    };
    if constexpr (KIND != kQc) {
        // ---- bounds of this part's columns (kAll: chunks of 64) or items
        const int n_all = KIND == kItems ? a.n_items : a.n_chunks;
        const int first = static_cast<int>(static_cast<long long>(n_all) * part / a.parts);
        const int last = static_cast<int>(static_cast<long long>(n_all) * (part + 1) / a.parts);
        const int* items = KIND == kItems ? a.items + static_cast<size_t>(b) * a.n_items + first : nullptr;
        const int n_ub = flat ? 0 : (KIND == kItems ? last - first : (last - first) * 64);
        auto column = [&](int i) { return KIND == kItems ? a.col[items[i]] : first * 64 + i; };
        if constexpr (KIND == kAll) {
#pragma unroll 1
            for (int c = wave; c * 64 < n_ub; c += NW) {
                const float u = max_window(a, img, first + c, Ahat, lane) * to_q;
                ub[c * 64 + lane] =
                    static_cast<uint16_t>(a.tid[(first + c) * 64 + lane] >= 0 ? f16_up(u) : kDone);
            }
        } else {
#pragma unroll 1
            for (int j0 = wave * G; j0 < n_ub; j0 += NW * G) {
                const int j = j0 + lane / W;
                float U = window_sum(a, img, j < n_ub ? column(j) : -1, Ahat, lane) * to_q;
#pragma unroll
                for (int d = W / 2; d >= 1; d >>= 1) U = fmaxf(U, __shfl_xor(U, d, 64));
                if (j < n_ub && (lane & (W - 1)) == 0) ub[j] = static_cast<uint16_t>(f16_up(U));
            }
        }
        __syncthreads();
        // ---- rounds: the columns with the largest bounds, first as seeds
#pragma unroll 1
        for (bool seed = !flat;; seed = false) {
            const int want = seed ? n_seed_scored : kBatch;
            const float q = C.q;
            __syncthreads();
            if (tid < 64) C.hist[tid] = 0;
            if (tid == 0) {
                C.live = 0;
                C.maxu = 0;
                C.cut = 0;
                C.work = 0;
            }
            __syncthreads();
            int live = 0, mu = 0;
            for (int i = tid; i < n_ub; i += NT) {
                const uint32_t u = ub[i];
                if (u != kDone && h2f(u) >= q) {
                    ++live;
                    mu = max(mu, static_cast<int>(u));
                }
            }
            if (live) {
                atomicAdd(&C.live, live);
                atomicMax(&C.maxu, mu);
            }
            __syncthreads();
            live = C.live;
            if (live == 0 && !flat) break;
            // Given up: after a batch, where more live than windows may be
            // scored; right after the seeds, where half of the templates
            // live (noise, another crystal): a batch of those takes all its
            // windows and settles nothing. 16384 patterns of noise, 2000 FCC
            // templates: 12.2 ms without this, 9.8 with (8.0 scanned at
            // once); one in eight of noise: 5.5, 3.4. From two fifths on,
            // unit weights lose (2.52 ms, 2.64), from three fifths another
            // crystal's patterns (9.88, 9.94).
            if (!seed && (scored > 0 ? live > a.give_up : live > n_ub / 2)) {
                gone = true;
                break;
            }
            const int top = C.maxu;
            // bins of float16 bits: one per 16 down from the largest (a
            // factor of 2 holds 1024)
            auto bin = [&](uint32_t u) { return max(0, 63 - (top - static_cast<int>(u)) / 16); };
            if (live > want) {
                for (int i = tid; i < n_ub; i += NT) {
                    const uint32_t u = ub[i];
                    if (u != kDone && h2f(u) >= q) {
                        const int k = bin(u);
                        if (k > 0) atomicAdd(&C.hist[k], 1);
                    }
                }
                __syncthreads();
                if (wave == 0) {
                    const int c = cut_bin(C.hist, want, lane);
                    if (lane == 0) C.cut = c;
                }
                __syncthreads();
            }
            const int cut = C.cut;
            for (int i0 = 0; i0 < n_ub; i0 += NT) {
                const int i = i0 + tid;
                const uint32_t u = i < n_ub ? ub[i] : kDone;
                const bool take = u != kDone && h2f(u) >= q && bin(u) >= cut;
                const int at = place(&C.work, take, lane);
                if (take && at < kSel) {
                    L.pend[at] = static_cast<uint16_t>(i);
                    if (!seed) ub[i] = static_cast<uint16_t>(kDone);
                }
            }
            __syncthreads();
            const int ns = min(C.work, kSel);
#pragma unroll 1
            for (int j0 = wave * G; j0 < ns; j0 += NW * G) {
                const int j = j0 + lane / W;
                evaluate(j < ns ? column(L.pend[j]) : -1, seed);
            }
            __syncthreads();
            drain(seed);
            __syncthreads();
            if (flat || gone) break;
        }
    } else {
        // ---- seeds: about kSeedPicks columns of the largest listed bounds
        int n_seed = 0;
        if (!flat) {
            const size_t lo = static_cast<size_t>(b) * a.n_list;
            float m = 0.0f;
            for (int i = tid; i < a.n_list; i += NT) m = fmaxf(m, a.lq[lo + i]);
            m = tmlib::wave_max(m);
            if (lane == 0) red[wave] = m;
            if (tid < 64) C.hist[tid] = 0;
            if (tid == 0) {
                C.cut = 0;
                C.work = 0;
            }
            __syncthreads();
#pragma unroll
            for (int w = 0; w < NW; ++w) m = fmaxf(m, red[w]);
            const float to_bin = m > 0.0f ? 128.0f / m : 0.0f;   // bins over [max / 2, max]
            auto bin = [&](float v) { return min(63, max(0, static_cast<int>(v * to_bin) - 64)); };
            for (int i = tid; i < a.n_list; i += NT)
                if (a.lc[lo + i] >= 0) atomicAdd(&C.hist[bin(a.lq[lo + i])], 1);
            __syncthreads();
            if (wave == 0) {
                const int c = cut_bin(C.hist, max(kSeedPicks, n_seed_scored), lane);
                if (lane == 0) C.cut = c;
            }
            __syncthreads();
            const int cut = C.cut;
            // picked columns wait at the entry list's end
            for (int i0 = 0; i0 < a.n_list; i0 += NT) {
                const int i = i0 + tid;
                const int c = i < a.n_list ? a.lc[lo + i] : -1;
                const bool take = c >= 0 && c < a.n_valid && bin(a.lq[lo + i]) >= cut;
                const int at = place(&C.work, take, lane);
                if (take && at < kMaxSeeds) L.ent[kEntries - 1 - at].x = static_cast<uint32_t>(c);
            }
            __syncthreads();
            n_seed = min(C.work, kMaxSeeds);
        }
        // ---- rounds: the seeds first, then every template whose bound in Qc
        // reaches q. A segment of 64 blocks of 64 columns is tested at a time
        // (its loads independent of each other): lane i keeps block i's hits.
        // Then up to kPend of them per wave and round get their window bounds.
        const float* row = a.Qc + static_cast<size_t>(b) * a.n_cs;
        const int w_all = a.parts * NW, w_me = part * NW + wave;
        const int lo = flat ? 0 : static_cast<int>(static_cast<long long>(a.n_valid) * w_me / w_all);
        const int hi = flat ? 0 : static_cast<int>(static_cast<long long>(a.n_valid) * (w_me + 1) / w_all);
        uint16_t* pend = L.pend + wave * kPend;
        constexpr int kSeg = 64 * 64;
        int seg = lo - kSeg, left = 0, done = 0, before = 0;
        unsigned long long hits = 0;
        const int share = (n_seed + NW - 1) / NW;
#pragma unroll 1
        for (bool seed = !flat;; seed = false) {
            int k = 0;
            if (seed) {
                k = max(0, min(share, n_seed - wave * share));
            } else {
#pragma unroll 1
                while (left == 0 && seg + kSeg < hi) {        // uniform
                    seg += kSeg;
                    const float q = C.q;
                    hits = 0;
                    constexpr int kAhead = 8;
#pragma unroll 1
                    for (int k0 = 0; k0 < 64 && seg + 64 * k0 < hi; k0 += kAhead) {
                        float v[kAhead];
#pragma unroll
                        for (int j = 0; j < kAhead; ++j) v[j] = row[min(seg + 64 * (k0 + j) + lane, hi - 1)];
#pragma unroll
                        for (int j = 0; j < kAhead; ++j) {
                            const unsigned long long m =
                                tmlib::ballot(seg + 64 * (k0 + j) + lane < hi && v[j] >= q);
                            if (lane == k0 + j) hits = m;
                        }
                    }
                    const int own = __popcll(hits);
                    int x = own;                              // hits before this lane's
#pragma unroll
                    for (int d = 1; d < 64; d <<= 1) {
                        const int up = __shfl_up(x, d, 64);
                        if (lane >= d) x += up;
                    }
                    before = x - own;
                    left = __builtin_amdgcn_readlane(x, 63);
                    done = 0;
                }
                k = min(left, kPend);
                // hits done .. done + k - 1 in order
                int at = before - done;
                for (unsigned long long m = hits; m && at < k; m &= m - 1, ++at)
                    if (at >= 0) pend[at] = static_cast<uint16_t>(64 * lane + __ffsll(static_cast<long long>(m)) - 1);
                left -= k;
                done += k;
                tmlib::wave_sync();
            }
#pragma unroll 1
            for (int j0 = 0; j0 < k; j0 += G) {
                const int j = j0 + lane / W;
                int col = -1;
                if (j < k)
                    col = seed ? static_cast<int>(L.ent[kEntries - 1 - (wave * share + j)].x) : seg + pend[j];
                evaluate(col, seed);
            }
            const bool more = left > 0 || seg + kSeg < hi;
            const int any = __syncthreads_or(more ? 1 : 0);
            if (seed || C.cnt > kEntries - NW * kPend || !any) drain(seed);
            if (!any || gone) break;
            __syncthreads();
        }
    }
    if (tid == 0) a.give[b * a.parts + part] = gone ? 1 : 0;
    if (wave == 0 && lane < N && !gone) {
        const bool ok = lane < st.cnt;
        a.top_t[o_out + lane] = ok ? st.t : (a.parts > 1 ? INT_MAX : -1);
        a.top_s[o_out + lane] = ok ? st.s : (a.parts > 1 ? 0 : -1);
        a.top_q[o_out + lane] = ok ? st.q : -INFINITY;
    }
}

// The parts' lists of a split search merged into the pattern's rows, one
// wave per pattern (score descending, ties to the lower template index).
// give, full: optional.
__global__ void __launch_bounds__(256)
merge_parts(const double* __restrict__ norms, int B, int parts, int N,
            const int* __restrict__ pt, const int* __restrict__ ps, const float* __restrict__ pq,
            const int* __restrict__ give, int* __restrict__ full, int* __restrict__ top_t,
            int* __restrict__ top_s, float* __restrict__ top_q) {
    const int lane = threadIdx.x & 63;
    const int b = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (b >= B) return;
    const size_t e0 = static_cast<size_t>(b) * parts * N, o = static_cast<size_t>(b) * N;
    // given up by any part: by all (the plain scan writes the rows)
    const bool any = give && tmlib::ballot(lane < parts && give[b * parts + lane] != 0) != 0;
    if (full && lane == 0) full[b] = any ? 1 : 0;
    if (any) return;
    const double pn = norms[b];
    if ((__double_as_longlong(pn) & 0x7ff0000000000000LL) == 0x7ff0000000000000LL) {
        if (lane < N) {
            top_t[o + lane] = -1;
            top_s[o + lane] = -1;
            top_q[o + lane] = __int_as_float(0x7fc00000);
        }
        return;
    }
    float prev_q = INFINITY;
    int prev_t = -1;
    for (int r = 0; r < N; ++r) {
        float bq = -INFINITY;
        int bt = INT_MAX, bs = 0;
        for (int c = lane; c < parts * N; c += 64) {
            const float q = pq[e0 + c];
            const int t = pt[e0 + c];
            const bool after = q < prev_q || (q == prev_q && t > prev_t);
            const bool better = q > bq || (q == bq && t < bt);
            if (after && better) { bq = q; bt = t; bs = ps[e0 + c]; }
        }
#pragma unroll
        for (int x = 32; x >= 1; x >>= 1) {
            const float oq = __shfl_xor(bq, x, 64);
            const int ot = __shfl_xor(bt, x, 64);
            const int os = __shfl_xor(bs, x, 64);
            if (oq > bq || (oq == bq && ot < bt)) { bq = oq; bt = ot; bs = os; }
        }
        if (lane == 0) {
            top_t[o + r] = bt == INT_MAX ? -1 : bt;
            top_s[o + r] = bt == INT_MAX ? -1 : bs;
            top_q[o + r] = bq;
        }
        prev_q = bq;
        prev_t = bt;
    }
}

// Shifts per window and columns per window maximum.
int window_width(int n) { return (n + W - 1) / W; }
int window_reach(int n) { return (W + 1) * window_width(n) - n; }

// Per-wave scratch of the image build, in halves.
size_t scratch_halves(int n) {
    const int o = (n + 63) / 64;
    const int H = window_reach(n) + o;
    return static_cast<size_t>(n + H + (n + H) / o + 7) / 8 * 8;
}

// LDS of image and lists.
template <Kind KIND, int NW>
size_t lds_bytes(const tm_library* L) {
    const int n = L->n_theta;
    const size_t image = static_cast<size_t>(L->n_rows) * window_width(n) * W * 2;
    const size_t rest = std::max(sizeof(Lists<KIND, NW>), kBuildWaves * scratch_halves(n) * sizeof(uint16_t));
    return (image + rest + 15) / 16 * 16;
}

}  // namespace

// ------------------------------------------------------------ library data

int tmlib::search_prepare(tm_library* L, const std::vector<uint32_t>& recs,
                          const std::vector<int32_t>& seg, const std::vector<int32_t>& rows,
                          const std::vector<int32_t>& band_off, hipStream_t s, size_t& bytes) {
    L->search = L->sr_all = false;
    const int n = L->n_theta, Tp = L->Tp;
    int dev = 0, attr = 0;
    if (!L->bound || L->n_rows > kMaxRows || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&attr, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        return TM_OK;
    const size_t max_lds = static_cast<size_t>(attr) - 1024;
    if (lds_bytes<kQc, 16>(L) > max_lds || static_cast<size_t>(L->n_rows) * window_width(n) > 65535)
        return TM_OK;
    const int n_cls = L->n_cls, n_bands = L->n_bands;
    auto each_record = [&](int32_t t, auto&& fn) {   // the plain path's records in its order
        for (int band = 0; band < n_bands; ++band) {
            const size_t s0 = (static_cast<size_t>(t) * n_bands + band) * n_cls;
            for (int32_t r = seg[s0]; r < seg[s0 + n_cls]; ++r) {
                const uint32_t o = recs[2 * static_cast<size_t>(r)];
                fn(band_off[band] + o / static_cast<uint32_t>(L->row_width),
                   o % static_cast<uint32_t>(L->row_width), recs[2 * static_cast<size_t>(r) + 1]);
            }
        }
    };
    // Sparse libraries: columns of their own, templates with alike sector
    // counts side by side, 64 to a chunk; a chunk takes the largest count of
    // each sector in steps. Where that is little work, the search kernel
    // bounds all templates by itself.
    const int w = window_width(n);
    std::vector<int32_t> tid = L->bnd_tid;
    std::vector<uint32_t> chunk, wrec, xrec, drec;
    if (static_cast<double>(L->n_spots) <= kSparse * Tp && Tp <= kAllTemplates &&
        lds_bytes<kAll, 16>(L) + 2 * static_cast<size_t>(Tp) + 256 <= max_lds) {
        std::vector<std::array<uint8_t, W>> sc(Tp);
        bool fits = true;
        for (int32_t t = 0; t < Tp; ++t) {
            int c[W] = {0};
            each_record(t, [&](uint32_t, uint32_t k, uint32_t) { ++c[k / w]; });
            for (int q = 0; q < W; ++q) {
                fits = fits && c[q] <= 255;
                sc[t][q] = static_cast<uint8_t>(std::min(c[q], 255));
            }
        }
        std::vector<int32_t> order(Tp);
        std::iota(order.begin(), order.end(), 0);
        std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) { return sc[x] > sc[y]; });
        uint32_t steps = 0;
        for (int32_t i0 = 0; i0 < Tp; i0 += 64) {
            uint32_t m[W] = {0}, packed[2] = {0u, 0u};
            for (int32_t i = i0; i < std::min(Tp, i0 + 64); ++i)
                for (int q = 0; q < W; ++q) m[q] = std::max<uint32_t>(m[q], sc[order[i]][q]);
            const uint32_t start = steps;
            for (int q = 0; q < W; ++q) {
                packed[q / 4] |= m[q] << (8 * (q % 4));
                steps += m[q];
            }
            chunk.insert(chunk.end(), {start, 0u, packed[0], packed[1]});
        }
        L->sr_all = fits && steps <= static_cast<uint32_t>(kAllSteps);
        if (L->sr_all) {
            tid.assign((static_cast<size_t>(Tp) + 63) / 64 * 64, -1);
            std::copy(order.begin(), order.end(), tid.begin());
            drec.assign((static_cast<size_t>(steps) + 4) * 64, 0u);   // 4 steps are loaded ahead
        }
    }
    std::vector<int32_t> col(Tp), xhead(2 * static_cast<size_t>(Tp));
    for (size_t c = 0; c < tid.size(); ++c)
        if (tid[c] >= 0) col[tid[c]] = static_cast<int32_t>(c);
    std::vector<uint32_t> head(tid.size() * 4, 0u), sector[W];
    for (int32_t t = 0; t < Tp; ++t) {
        for (auto& v : sector) v.clear();
        uint32_t* h = &head[static_cast<size_t>(col[t]) * 4];
        xhead[2 * static_cast<size_t>(t)] = static_cast<int32_t>(xrec.size() / 2);
        h[0] = static_cast<uint32_t>(wrec.size() / kUnit);
        double wsum = 0.0;
        int cnt = 0;
        each_record(t, [&](uint32_t row, uint32_t k, uint32_t bits) {
            float wt;
            std::memcpy(&wt, &bits, 4);
            xrec.push_back(static_cast<uint32_t>(rows[row]) << 20 | row << 10 | k);
            xrec.push_back(bits);
            sector[k / w].push_back((row * w + k % w) |
                                    static_cast<uint32_t>(f16_up(std::ldexp(wt, kWeightExp))) << 16);
            wsum += wt;
            ++cnt;
        });
        while (xrec.size() / 2 % kExactPad) { xrec.push_back(0u); xrec.push_back(0u); }
        xhead[2 * static_cast<size_t>(t) + 1] =
            static_cast<int32_t>(xrec.size() / 2) - xhead[2 * static_cast<size_t>(t)];
        if (L->sr_all) {
            const uint32_t* ch = &chunk[static_cast<size_t>(col[t] / 64) * 4];
            uint32_t step = ch[0];
            for (int q = 0; q < W; ++q) {
                for (size_t i = 0; i < sector[q].size(); ++i)
                    drec[(static_cast<size_t>(step) + i) * 64 + col[t] % 64] = sector[q][i];
                step += (ch[2 + q / 4] >> (8 * (q % 4))) & 255u;
            }
        }
        for (int q = 0; q < W; ++q) {
            while (sector[q].size() % kUnit) sector[q].push_back(0u);
            const size_t units = sector[q].size() / kUnit;
            if (units > 255) { L->sr_all = false; return TM_OK; }
            h[2 + q / 4] |= static_cast<uint32_t>(units) << (8 * (q % 4));
            wrec.insert(wrec.end(), sector[q].begin(), sector[q].end());
        }
        // margin: gamma times the weights' sum, its roundings (this one, the
        // product with A, the first sum) covered by the last factor
        const float cf = static_cast<float>(std::ldexp(gamma32(cnt) * wsum, kWeightExp) * (1.0 + 0x1p-18));
        std::memcpy(&h[1], &cf, 4);
        if (xrec.size() / 2 > static_cast<size_t>(INT32_MAX) / 2 || wrec.size() > static_cast<size_t>(INT32_MAX) / 2) {
            L->sr_all = false;
            return TM_OK;
        }
    }
    if (wrec.empty()) wrec.assign(kUnit, 0u);
    if (xrec.empty()) xrec.assign(2, 0u);
    auto up = [&](auto** dst, const auto& v) -> int {
        using T = std::remove_reference_t<decltype(v[0])>;
        const size_t nb = std::max<size_t>(v.size(), 1) * sizeof(T);
        hipError_t e = hipMalloc(reinterpret_cast<void**>(dst), nb);
        if (e != hipSuccess) {
            *dst = nullptr;
            tmlib::set_error("hipMalloc(%zu) failed: %s", nb, hipGetErrorString(e));
            return TM_ENOMEM;
        }
        bytes += nb;
        TM_HIP(hipMemcpyAsync(*dst, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, s));
        return TM_OK;
    };
    if (int r = up(&L->d_sr_recs, wrec)) return r;
    if (int r = up(&L->d_sr_head, head)) return r;
    if (int r = up(&L->d_sr_xrecs, xrec)) return r;
    if (int r = up(&L->d_sr_xhead, xhead)) return r;
    if (int r = up(&L->d_sr_tid, tid)) return r;
    if (int r = up(&L->d_sr_col, col)) return r;
    if (L->sr_all) {
        if (int r = up(&L->d_sr_drecs, drec)) return r;
        if (int r = up(&L->d_sr_chunk, chunk)) return r;
    }
    TM_HIP(hipStreamSynchronize(s));          // the host arrays end here
    L->search = true;
    return TM_OK;
}

void tmlib::search_release(tm_library* L) {
    void** all[] = {reinterpret_cast<void**>(&L->d_sr_recs), reinterpret_cast<void**>(&L->d_sr_head),
                    reinterpret_cast<void**>(&L->d_sr_xrecs), reinterpret_cast<void**>(&L->d_sr_xhead),
                    reinterpret_cast<void**>(&L->d_sr_tid), reinterpret_cast<void**>(&L->d_sr_col),
                    reinterpret_cast<void**>(&L->d_sr_drecs), reinterpret_cast<void**>(&L->d_sr_chunk)};
    for (void** p : all) {
        (void)hipFree(*p);
        *p = nullptr;
    }
    L->search = false;
}

// ------------------------------------------------------------ launches

namespace {

// Launches a search with the bounds of a; ub_items: bounds kept in LDS per
// workgroup when there is one part (0: none).
int run_search(const tm_library* lib, Kind kind, SearchArgs a, int32_t B, size_t ub_items,
               int32_t* top_template, int32_t* top_angle, float* top_score, hipStream_t s) {
    a.n = lib->n_theta;
    a.n_rows = lib->n_rows;
    a.w = window_width(a.n);
    a.wlen = window_reach(a.n);
    a.scr = static_cast<int>(scratch_halves(a.n));
    a.recs = reinterpret_cast<const uint4*>(lib->d_sr_recs);
    a.head = reinterpret_cast<const uint4*>(lib->d_sr_head);
    a.xrecs = reinterpret_cast<const uint2*>(lib->d_sr_xrecs);
    a.xhead = reinterpret_cast<const int2*>(lib->d_sr_xhead);
    a.tid = lib->d_sr_tid;
    a.col = lib->d_sr_col;
    a.dfac = lib->bnd_dfac;
    a.drecs = lib->d_sr_drecs;
    a.dchunk = reinterpret_cast<const uint4*>(lib->d_sr_chunk);
    a.n_chunks = (lib->Tp + 63) / 64;
    a.Tp = lib->Tp;
    // few patterns: several workgroups per pattern, each with its share of
    // the columns, their lists merged
    const int columns = kind == kItems ? a.n_items : lib->Tp;
    int parts = 1;
    while (parts < kMaxParts && 2 * static_cast<int64_t>(parts) * B <= kSplitGrid &&
           2 * parts * kPartColumns <= columns)
        parts *= 2;
    a.parts = parts;
    a.top_t = top_template;
    a.top_s = top_angle;
    a.top_q = top_score;
    // A plain scan takes about records x (1 + group x slots) wave
    // instructions, a window of a candidate kWindowCost per record and
    // kWindowMore: a part gives up when it has spent half of its share of
    // the scan, at the latest after kMaxGive windows (a batch waits for its
    // last workgroup: a large one, or one with long scans, less so).
    const double mean = static_cast<double>(lib->n_spots) / lib->Tp;
    const double window = kWindowCost * mean + kWindowMore;
    const int slots = tmlib::slots_for(a.n);
    const double scan = kind == kItems ? a.n_items * mean * (2 + 2 * slots)
                                       : static_cast<double>(lib->n_records) * (1 + lib->group * slots);
    const double most = std::max<double>({kMaxGive, B / 8.0, scan / (64 * window)});
    a.give_up = static_cast<int>(std::min(most, std::max<double>(kMinGive, scan / (2 * window * parts))));
    // scratch: the parts' lists, flags of given-up parts and patterns
    const size_t ne = static_cast<size_t>(B) * parts * a.N;
    int32_t* full;
    tmlib::Scratch mem;
    mem.add(full, B);
    if (parts > 1) {
        mem.add(a.top_t, ne);
        mem.add(a.top_s, ne);
        mem.add(a.top_q, ne);
        mem.add(a.give, static_cast<size_t>(B) * parts);
    }
    if (int e = mem.allocate(s)) return e;
    if (parts == 1) a.give = full;
    const size_t ub = ub_items ? ((ub_items / 64 + parts) / parts + 1) * 64 * sizeof(uint16_t) : 0;
    // the intensities of few rows stay in LDS as well, two turns each
    const size_t lrows = static_cast<size_t>(a.n_rows) * 2 * a.n * sizeof(float);
    auto launch = [&](auto kind_c, auto rows_c) -> int {
        constexpr Kind KIND = static_cast<Kind>(decltype(kind_c)::value);
        constexpr bool LROWS = decltype(rows_c)::value;
        const size_t more = ub + (LROWS ? lrows : 0);
        const size_t l8 = lds_bytes<KIND, 8>(lib), l16 = lds_bytes<KIND, 16>(lib);
        // 16 waves where LDS allows two workgroups per CU at most, or where
        // the workgroups do not fill the chip
        const bool large = l8 + more > kThreePerCu || static_cast<int64_t>(B) * parts <= kFillGrid;
        const size_t lds = (large ? l16 : l8) + more;
        a.lists_end = static_cast<int>((large ? l16 : l8) / sizeof(uint4));
        a.pitch = LROWS ? 2 * a.n : 0;
        auto go = [&](auto kern, int nw) -> int {
            TM_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
            hipLaunchKernelGGL(kern, dim3(B, parts), dim3(nw * 64), lds, s, a);
            TM_HIP(hipGetLastError());
            return TM_OK;
        };
        if (a.n <= 384)
            return large ? go(search_kernel<KIND, 16, 6, LROWS>, 16) : go(search_kernel<KIND, 8, 6, LROWS>, 8);
        return large ? go(search_kernel<KIND, 16, kMaxCols, LROWS>, 16)
                     : go(search_kernel<KIND, 8, kMaxCols, LROWS>, 8);
    };
    int r;
    if (kind == kQc) {
        r = launch(std::integral_constant<int, kQc>{}, std::false_type{});
    } else if (kind == kItems) {
        r = launch(std::integral_constant<int, kItems>{}, std::false_type{});
    } else {
        const auto all = std::integral_constant<int, kAll>{};
        r = lds_bytes<kAll, 16>(lib) + ub + lrows <= kTwoPerCu ? launch(all, std::true_type{})
                                                               : launch(all, std::false_type{});
    }
    if (parts > 1 && !r) {
        hipLaunchKernelGGL(merge_parts, dim3((B + 3) / 4), dim3(256), 0, s, a.norms, B, parts, a.N,
                           a.top_t, a.top_s, a.top_q, a.give, full, top_template, top_angle, top_score);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) r = tmlib::hip_fail(e, "merge_parts launch");
    }
    // patterns given up: their items scored one and all
    if (!r)
        r = tmlib::full_scans(lib, a.polar, a.norms, B, a.N, full, top_template, top_angle, top_score,
                              !a.rows, s, kind == kItems ? a.items : nullptr, a.n_items);
    return mem.release(s, r);
}

SearchArgs pattern_args(const tm_library* lib, const float* polar, const double* norms, int32_t N,
                        bool compact) {
    SearchArgs a{};
    a.polar = polar;
    a.norms = norms;
    a.rows = compact ? nullptr : lib->d_rows;
    a.Rs = compact ? lib->n_rows : lib->R;
    a.N = N;
    return a;
}

}  // namespace

int tmlib::merge_lists(const double* norms, int32_t B, int32_t parts, int32_t N, const int32_t* part_t,
                       const int32_t* part_s, const float* part_q, int32_t* top_template,
                       int32_t* top_angle, float* top_score, hipStream_t s) {
    hipLaunchKernelGGL(merge_parts, dim3((B + 3) / 4), dim3(256), 0, s, norms, B, parts, N, part_t, part_s,
                       part_q, nullptr, nullptr, top_template, top_angle, top_score);
    TM_HIP(hipGetLastError());
    return TM_OK;
}

int tmlib::refine_search(const tm_library* lib, const float* polar, const double* norms, int32_t B,
                         int32_t N, const float* amax, const float* Qc, int32_t n_cs,
                         const float* lane_q, const int32_t* lane_c, int32_t n_list,
                         int32_t* top_template, int32_t* top_angle, float* top_score, bool compact,
                         hipStream_t s) {
    SearchArgs a = pattern_args(lib, polar, norms, N, compact);
    a.amax = amax;
    a.Qc = Qc;
    a.n_cs = n_cs;
    a.n_valid = std::min(n_cs, lib->Tp);
    a.lq = lane_q;
    a.lc = lane_c;
    a.n_list = n_list;
    return run_search(lib, kQc, a, B, 0, top_template, top_angle, top_score, s);
}

int tmlib::search_all(const tm_library* lib, const float* polar, const double* norms, int32_t B,
                      int32_t N, int32_t* top_template, int32_t* top_angle, float* top_score,
                      bool compact, hipStream_t s) {
    const SearchArgs a = pattern_args(lib, polar, norms, N, compact);
    return run_search(lib, kAll, a, B, static_cast<size_t>(lib->Tp + 63) / 64 * 64, top_template,
                      top_angle, top_score, s);
}

// By the work of the scan of a list that the search replaces. Measured (scan,
// search; us): FCC 84 000 at 256 patterns 467, 519 and at 2048 1562, 1502,
// 168 000 at 256 818, 713; HCP 62 400 279, 421, 124 800 454, 502, 249 600 at 64
// 801, 589; orthorhombic 456 000 1290, 1303, 1.0e6 at 64 1313, 538.
bool tmlib::search_items_pays(const tm_library* lib, int32_t n_items) {
    const bool sparse = static_cast<double>(lib->n_spots) <= kSparse * lib->Tp;
    const double work = static_cast<double>(lib->n_spots) / lib->Tp * n_items * tmlib::slots_for(lib->n_theta);
    return lib->search && work >= (sparse ? kItemsSparse : kItemsDense) && n_items <= kAllTemplates &&
           lds_bytes<kItems, 16>(lib) + 2 * static_cast<size_t>(n_items) + 256 <= kMaxLds;
}

int tmlib::search_items(const tm_library* lib, const float* polar, const double* norms, int32_t B,
                        int32_t N, const int32_t* items, int32_t n_items, int32_t* top_template,
                        int32_t* top_angle, float* top_score, bool compact, hipStream_t s) {
    SearchArgs a = pattern_args(lib, polar, norms, N, compact);
    a.items = items;
    a.n_items = n_items;
    return run_search(lib, kItems, a, B, n_items, top_template, top_angle, top_score, s);
}
