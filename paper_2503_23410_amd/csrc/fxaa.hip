// FXAA-style edge anti-aliasing inside the VaFR LP buffer (Sec. 3.4: the
// LP buffer is anti-aliased before the inverse map, because in the
// periphery one texel covers many display pixels).
//
// The method of Lottes (FXAA, 2009) is applied on the ragged polar grid:
// along the angle a texel's neighbours are the adjacent rows of its column
// (cyclic); along the radius they are the inner and outer columns sampled at
// the texel's angle, linear in the row coordinate.  Per texel: a luma
// contrast test, the edge normal from second differences, the side of the
// edge with the larger luma step, a search for the two ends of the edge
// along it, a sub-texel term, and a blend toward the neighbour across the
// edge.  The constants and the operation order (FP32, no fused multiply-add;
// built with -ffp-contract=off) are part of the library's contract with its
// test oracle.
//
// A workgroup takes a tile of kFxaaCols columns by one of the K equal sectors
// that give each of those columns at most 64 rows, one column per wave, and
// first copies the tile with the column on either side and three more rows at
// either end into LDS.  Most texels compare within that window (an edge search
// mostly ends after a step or two); what lies outside is read from the LP
// buffer.  Straight from the LP buffer (one thread per texel, up to 24
// dependent rounds of 16-byte gathers) the vector L1's return path was 70%
// busy at three resident waves per SIMD.  The paper's layout (1.06M texels),
// calls back to back, without -> with the window: 4.52M terrain (nearly every
// texel an edge) 46 -> 31 us, 1.13M terrain 49 -> 32, 4,096-triangle soup 28 ->
// 22, noise 63 -> 41, a buffer without edges 12.5 -> 12.2.  What bounds it now
// is the search: a wave walks on until the last of its 64 searches has ended.
// Windows of 2 to 16 columns on either side and 4 to 10 rows, and tiles of 8,
// 12 or 16 columns, measured 34-44 us on the 4.52M terrain.
//
// A layout of fewer than kFxaaDirect texels does not fill the chip, and what
// counts is how long one workgroup takes: it is faster without the window, one
// thread per texel (14,164 texels: soup 9.8 -> 8.5 us, 1.13M terrain 11.5 -> 11.2,
// noise 10.8 -> 11.6; 75,833: 11.6 -> 9.7, 11.5 -> 12.0, 10.7 -> 11.8; 282,968: 13.2
// -> 12.2, 12.9 -> 13.1, 15.4 -> 19.6; 1,063,314: 21.9 -> 26.9, 32.3 -> 41.7).
#include <type_traits>

#include "vafr_internal.h"

namespace vafr {
namespace {

constexpr float kEdgeRel = 0.125f;   // contrast threshold relative to the local luma maximum
constexpr float kEdgeMin = 0.0625f;  // absolute contrast threshold
constexpr float kSubpix = 0.75f;     // weight of the sub-texel term
constexpr int kSteps = 6;
__constant__ float kStepAt[kSteps] = {1.0f, 2.0f, 3.0f, 4.0f, 6.0f, 8.0f};   // end-search offsets

constexpr int kWindowCols = kFxaaCols + 16;       // the tile's columns and eight on either side
constexpr int kHalo = 3;                           // rows staged past the tile's at either end
constexpr int kWindowTexels = (kFxaaCols + 2) * (kFxaaRows + 2 * kHalo);

struct FxaaView {
    const int2* col;     // (rows, first texel) per column
    const int4* tile;    // staged form: (first column, sector, sectors, narrow) per workgroup
    const int32_t* blk_col;   // direct form: column of the first texel of each workgroup
    int32_t n_cols;
    int64_t n_texels;
    const float4* in;
    float4* out;
};

// A column of the window: rows lo .. lo + pairs (cyclic: row j is row j mod
// n) are at LDS texels base .. base + pairs; pairs = 0: none staged.
struct WinCol {
    int n, off, lo, base, pairs;
};

// The same record for every lane of the wave, in scalar registers.
__device__ __forceinline__ WinCol uniform(const WinCol& w) {
    return WinCol{__builtin_amdgcn_readfirstlane(w.n), __builtin_amdgcn_readfirstlane(w.off),
                  __builtin_amdgcn_readfirstlane(w.lo), __builtin_amdgcn_readfirstlane(w.base),
                  __builtin_amdgcn_readfirstlane(w.pairs)};
}

struct Window {
    float4 tex[kWindowTexels];
    WinCol col[kWindowCols];
};

// Row j (any integer, cyclic) of a column in the LP buffer; the modulo is
// only taken when j leaves [0, rows).
__device__ __forceinline__ float4 texel_of(const FxaaView& v, const WinCol& w, int j) {
    int r = j;
    if ((unsigned)r >= (unsigned)w.n) {
        r = j % w.n;
        r = r < 0 ? r + w.n : r;
    }
    return v.in[(int64_t)w.off + r];
}

// Rows j and j + 1 of a column (kStaged: from the window where they are there).
template <bool kStaged>
__device__ __forceinline__ void texel_pair(const FxaaView& v, const Window& win, const WinCol& w, int j, float4& a,
                                           float4& b) {
    const int rel = j - w.lo;
    if (kStaged && (unsigned)rel < (unsigned)w.pairs) {
        a = win.tex[w.base + rel];
        b = win.tex[w.base + rel + 1];
    } else {
        a = texel_of(v, w, j);
        b = texel_of(v, w, j + 1);
    }
}

// The column at angle t turns, linear between rows.
template <bool kStaged>
__device__ __forceinline__ float4 column_of(const FxaaView& v, const Window& win, const WinCol& cn, float t) {
    const float s = t * (float)cn.n - 0.5f;
    const float fs = floorf(s);
    const float w = s - fs;
    float4 a, b;
    texel_pair<kStaged>(v, win, cn, (int)fs, a, b);
    return make_float4(a.x + w * (b.x - a.x), a.y + w * (b.y - a.y), a.z + w * (b.z - a.z), a.w + w * (b.w - a.w));
}

__device__ __forceinline__ float luma(float4 p) { return (0.299f * p.x + 0.587f * p.y) + 0.114f * p.z; }

// |second difference| of three lumas along a line.
__device__ __forceinline__ float curvature(float a, float m, float b) { return fabsf((a - m) + (b - m)); }

// Texel (i, j); first: the column of window entry 0.
template <bool kStaged>
__device__ __forceinline__ float4 fxaa_texel(const FxaaView& v, const Window& win, int first, int i, int j) {
    auto window = [&](int c) -> std::conditional_t<kStaged, const WinCol&, WinCol> {
        c = c < 0 ? 0 : (c >= v.n_cols ? v.n_cols - 1 : c);
        if constexpr (kStaged) {
            return win.col[c - first];
        } else {
            const int2 cc = v.col[c];
            return WinCol{cc.x, cc.y, 0, 0, 0};
        }
    };
    // records of the texel's column and of its outer and inner neighbours
    const WinCol ci = kStaged ? uniform(window(i)) : window(i), co = kStaged ? uniform(window(i + 1)) : window(i + 1);
    const WinCol cn = kStaged ? uniform(window(i - 1)) : window(i - 1);
    const int n = ci.n;
    const float t = ((float)j + 0.5f) / (float)n;
    const float dt = 1.0f / (float)n;
    // (rows j - 1 .. j + 1 of a texel's own column are staged)
    const float4* own = win.tex + (kStaged ? ci.base + (j - ci.lo) : 0);
    const float4 M = kStaged ? own[0] : texel_of(v, ci, j);
    const float lM = luma(M);
    const float lU = luma(kStaged ? own[1] : texel_of(v, ci, j + 1));
    const float lD = luma(kStaged ? own[-1] : texel_of(v, ci, j - 1));
    const float lO = luma(column_of<kStaged>(v, win, co, t)), lI = luma(column_of<kStaged>(v, win, cn, t));
    const float lmax = fmaxf(fmaxf(fmaxf(lM, lU), fmaxf(lD, lO)), lI);
    const float lmin = fminf(fminf(fminf(lM, lU), fminf(lD, lO)), lI);
    const float range = lmax - lmin;
    if (range < fmaxf(kEdgeMin, lmax * kEdgeRel)) return M;
    const float lOU = luma(column_of<kStaged>(v, win, co, t + dt)), lOD = luma(column_of<kStaged>(v, win, co, t - dt));
    const float lIU = luma(column_of<kStaged>(v, win, cn, t + dt)), lID = luma(column_of<kStaged>(v, win, cn, t - dt));
    // luma curvature across the radius (three angles) and across the angle
    // (three radii), centre line weighted twice
    const float across_r = (curvature(lID, lD, lOD) + 2.0f * curvature(lI, lM, lO)) + curvature(lIU, lU, lOU);
    const float across_a = (curvature(lID, lI, lIU) + 2.0f * curvature(lD, lM, lU)) + curvature(lOD, lO, lOU);
    const bool radial = across_r >= across_a;   // the normal of the edge points along the radius
    const float lNeg = radial ? lI : lD, lPos = radial ? lO : lU;
    const float gNeg = fabsf(lNeg - lM), gPos = fabsf(lPos - lM);
    const int side = gPos >= gNeg ? 1 : -1;
    const float lSide = side > 0 ? lPos : lNeg;
    const float lLine = 0.5f * (lM + lSide);
    const float gScaled = 0.25f * fmaxf(gNeg, gPos);
    // End search: step p (in the edge's direction) compares the mean luma of
    // two samples with that of the edge's own two sides.  Along the angle
    // they are (column i, its side's column) at angle t + p dt; along the
    // radius, column i + p at angles t and t + side dt.  One form for both,
    // chosen by selects: a wave holds edges of either kind.
    float dist[2], lEnd[2];
    const int across = radial ? (side > 0 ? i + 1 : i - 1) : i;
    const float t_side = radial ? t : t + (float)side * dt;
#pragma unroll
    for (int dir = 0; dir < 2; ++dir) {
        const float sgn = dir == 0 ? -1.0f : 1.0f;
        dist[dir] = kStepAt[kSteps - 1] + 1.0f;
        lEnd[dir] = lLine;
        for (int k = 0; k < kSteps; ++k) {
            const float p = sgn * kStepAt[k];
            const float tt = t + p * dt;
            const int c = (int)p;
            const float la = luma(column_of<kStaged>(v, win, window(radial ? i : i + c), radial ? tt : t));
            const float lb = luma(column_of<kStaged>(v, win, window(radial ? across : i + c), radial ? tt : t_side));
            const float l = 0.5f * (la + lb);
            if (fabsf(l - lLine) >= gScaled) {
                dist[dir] = kStepAt[k];
                lEnd[dir] = l;
                break;
            }
        }
    }
    const int near = dist[0] <= dist[1] ? 0 : 1;
    const bool centre_below = lM - lLine < 0.0f, end_below = lEnd[near] - lLine < 0.0f;
    const float edge = centre_below != end_below ? 0.5f - dist[near] / (dist[0] + dist[1]) : 0.0f;
    const float lAvg = (2.0f * ((lU + lD) + (lI + lO)) + ((lIU + lID) + (lOU + lOD))) / 12.0f;
    const float s1 = fminf(fmaxf(fabsf(lAvg - lM) / range, 0.0f), 1.0f);
    const float s2 = (-2.0f * s1 + 3.0f) * (s1 * s1);
    const float off = fmaxf(edge, (s2 * s2) * kSubpix);
    const float4 S = radial ? column_of<kStaged>(v, win, side > 0 ? co : cn, t)
                            : kStaged ? own[side] : texel_of(v, ci, j + side);
    return make_float4(M.x + off * (S.x - M.x), M.y + off * (S.y - M.y), M.z + off * (S.z - M.z),
                       M.w + off * (S.w - M.w));
}

// First row of sector k of K in a column of n rows: the least j with
// (j + 1/2) / n >= k / K.
// (kNarrow: 2 n K + K fits 32 bits.)
template <bool kNarrow>
__device__ __forceinline__ int sector_row(int n, int k, int K) {
    if (kNarrow) return (int)((2u * (uint32_t)n * (uint32_t)k + (uint32_t)K - 1u) / (2u * (uint32_t)K));
    return (int)((2 * (int64_t)n * k + K - 1) / (2 * K));
}

__global__ __launch_bounds__(kFxaaThreads) void k_fxaa(const FxaaView v) {
    __shared__ Window win;
    const int4 tile = v.tile[blockIdx.x];
    const int i0 = tile.x, k = tile.y, K = tile.z;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int i1 = min(i0 + kFxaaCols, v.n_cols);      // past the tile's last column
    const int first = max(i0 - 8, 0), last = min(i1 + 8, v.n_cols);
    if (wave == 0) {
        WinCol w{1, 0, 0, 0, 0};
        int cnt = 0;
        if (lane < last - first) {
            const int c = first + lane;
            const int2 cn = v.col[c];
            int r0, r1;
            if (tile.w) {
                r0 = sector_row<true>(cn.x, k, K);
                r1 = sector_row<true>(cn.x, k + 1, K);
            } else {
                r0 = sector_row<false>(cn.x, k, K);
                r1 = sector_row<false>(cn.x, k + 1, K);
            }
            w.n = cn.x;
            w.off = cn.y;
            w.lo = r0 - kHalo;
            // columns outside the tile can hold more rows of the sector than
            // the tile's own: the rest of them is not staged
            if (c >= i0 - 1 && c <= i1) cnt = min(r1 - r0, kFxaaRows) + 2 * kHalo;
            w.pairs = cnt > 0 ? cnt - 1 : 0;
        }
        // exclusive prefix sum of the counts (at most 32 columns)
        int incl = cnt;
#pragma unroll
        for (int d = 1; d < 32; d <<= 1) {
            const int o = __shfl_up(incl, d, 64);
            if (lane >= d) incl += o;
        }
        w.base = incl - cnt;
        if (lane < last - first) win.col[lane] = w;
    }
    __syncthreads();
    // a wave copies a column at a time, all of its loads before the first write
    constexpr int kWaves = kFxaaThreads / 64, kMine = (kFxaaCols + 2 + kWaves - 1) / kWaves;
    static_assert(kFxaaRows + 2 * kHalo <= 128, "two rows per lane");
    const int s0 = max(i0 - 1, 0) - first, s1 = min(i1 + 1, v.n_cols) - first;
    float4 t[kMine][2];
#pragma unroll
    for (int q = 0; q < kMine; ++q) {
        const int c = s0 + wave + q * kWaves;
        if (c < s1) {
            const WinCol w = uniform(win.col[c]);
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (lane + 64 * h <= w.pairs) t[q][h] = texel_of(v, w, w.lo + lane + 64 * h);
        }
    }
#pragma unroll
    for (int q = 0; q < kMine; ++q) {
        const int c = s0 + wave + q * kWaves;
        if (c < s1) {
            const WinCol w = uniform(win.col[c]);
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (lane + 64 * h <= w.pairs) win.tex[w.base + lane + 64 * h] = t[q][h];
        }
    }
    __syncthreads();
    for (int i = i0 + wave; i < i1; i += kWaves) {
        const WinCol w = uniform(win.col[i - first]);
        const int r0 = w.lo + kHalo, rows = w.pairs + 1 - 2 * kHalo;
        if (lane < rows) v.out[(int64_t)w.off + r0 + lane] = fxaa_texel<true>(v, win, first, i, r0 + lane);
    }
}

// The direct form: one thread per texel, everything from the LP buffer.  The
// column of texel k: from the workgroup's first column, walk forward (a
// workgroup spans several columns only near the centre of the grid).
__global__ __launch_bounds__(kTexelBlock) void k_fxaa_direct(const FxaaView v) {
    const int64_t k = (int64_t)blockIdx.x * kTexelBlock + threadIdx.x;
    if (k >= v.n_texels) return;
    int c = v.blk_col[blockIdx.x];
    while (c + 1 < v.n_cols && (int64_t)v.col[c + 1].y <= k) ++c;
    __shared__ Window win;   // only named: the direct form does not read it, and no LDS is taken
    v.out[k] = fxaa_texel<false>(v, win, 0, c, (int)(k - v.col[c].y));
}

}  // namespace

int launch_fxaa(const LayoutDev& ld, int32_t n_cols, int64_t n_texels, const float* in, float* out,
                hipStream_t stream) {
    if (n_texels <= 0) return VAFR_OK;
    FxaaView v{ld.col, ld.fxaa_tile, ld.blk_col, n_cols, n_texels, reinterpret_cast<const float4*>(in),
               reinterpret_cast<float4*>(out)};
    if (n_texels < kFxaaDirect)
        hipLaunchKernelGGL(k_fxaa_direct, dim3((unsigned)((n_texels + kTexelBlock - 1) / kTexelBlock)),
                           dim3(kTexelBlock), 0, stream, v);
    else
        hipLaunchKernelGGL(k_fxaa, dim3((unsigned)ld.n_fxaa_tiles), dim3(kFxaaThreads), 0, stream, v);
    VAFR_HIP(hipGetLastError());
    return VAFR_OK;
}

}  // namespace vafr
