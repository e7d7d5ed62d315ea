// Inverse mapping of an LP buffer onto the display (Sec. 3.2.3,
// Eqs. (10)-(11)).
//
// A workgroup of 4 waves covers a tile of 64 x 4P display pixels; each wave
// writes P rows of 64 consecutive pixels, so the 16-byte RGBA stores of a
// wave form one contiguous 1 KiB segment per row; they are non-temporal
// because the image is written once and not read back here.
//
// VaFR tiles stage their LP texels in LDS first.  Wave 0 bounds the tile's
// footprint in the LP buffer -- the columns between the smallest and the
// largest film radius of the tile and, in each column, the rows between the
// smallest and the largest polar angle, with one texel of margin -- and the
// workgroup copies those texels with row-contiguous loads; the four texels
// of each pixel are then read from LDS.  In nearly every tile of a large
// display the staged rows do not cross the seam: such tiles take sample_rows,
// the others sample_vafr (178 VALU instructions per pixel), with the same
// arithmetic.  A texel outside the staged region (not expected, but the bound
// is computed in floating point) is read from the LP buffer instead, so the
// result never depends on the bound.  Tiles whose footprint exceeds the LDS budget -- those within a few
// degrees of the gaze point, where one display pixel maps to about one texel
// or the tile surrounds the gaze -- read every texel from the LP buffer.
//
// What bounds it is the store rate: binocular pairs at 8K run at 6.8 - 6.9 TB/s,
// where a fill reaches 6.86 on this card.  Measured, all tiles in the general
// sampler -> now: one view 7680x4320 134 -> 88 us, 3840x2160 42 -> 33 us,
// 1921x1083 20 -> 14 us; binocular pairs at 8K 174 -> 160 us; 16 mixed views
// (unpaired) 1.21 -> 0.83 ms.
//
// A view may carry a second LP buffer and image with the same layout, gaze
// and display (the other eye of a binocular frame): every pixel then reads
// the same four texel positions with the same weights in both buffers, so
// the tile stages both (half of the LDS budget each) and maps each pixel
// once for both images.
//
// Tiles are taken in row-major order of the workgroup id, so the eight XCDs
// (which receive consecutive ids in turn) write neighbouring tiles of the
// same tile row at the same time.  Giving each XCD a contiguous band of rows
// instead keeps each XCD's LP reads in its own L2, but makes the stores --
// 97% of the kernel's traffic -- slower: a store-only probe of 64 x 32 tiles
// drops from 6.2 to 5.6 TB/s, and the kernel took 217 instead of 213 us per
// binocular 8K frame when its tiles were of that size.
#include "vafr_internal.h"

namespace vafr {
namespace {

constexpr int kTileW = 64;
constexpr int kWaves = kReconThreads / 64;
// LDS budget of one tile: staged texels and staged columns (one per lane of
// the wave that builds the column table).
constexpr int kStageTexels = 1024;
constexpr int kStageCols = 64;

// Workgroup id (within one view) -> tile, row-major.
__device__ __forceinline__ void tile_of(int id, int nbx, int& bx, int& by) {
    by = id / nbx;
    bx = id - by * nbx;
}

// Buffer-resource access: 32-bit byte offsets from a uniform base keep the
// per-pixel address arithmetic out of 64-bit VALU operations.  Word 3 of the
// descriptor is the raw-buffer format of gfx9-family GPUs.
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
constexpr int kRsrcWord3 = 0x00020000;
constexpr int kNonTemporal = 2;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, kRsrcWord3);
}

__device__ __forceinline__ float4 ld4(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    const v4u v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}

__device__ __forceinline__ v2u ld2(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
}

// Streaming 16-byte store of one pixel.
__device__ __forceinline__ void store_px(__amdgpu_buffer_rsrc_t r, uint32_t off, float4 c) {
    const v4u v = {__float_as_uint(c.x), __float_as_uint(c.y), __float_as_uint(c.z), __float_as_uint(c.w)};
    __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, kNonTemporal);
}

// Polar angle of (dx, dy) in turns, [0, 1], measured from +x toward +y.
// atan on [0, 1] is a degree-15 odd minimax polynomial (coefficients fitted
// for this kernel; FP32 error below 1.4e-7 rad), extended by the octant
// symmetries.
__device__ __forceinline__ float angle_turns(float dx, float dy) {
    const float ax = fabsf(dx), ay = fabsf(dy);
    const float mx = fmaxf(ax, ay), mn = fminf(ax, ay);
    const float a = mx > 0.0f ? mn * __builtin_amdgcn_rcpf(mx) : 0.0f;
    const float z = a * a;
    float p = -0.00405457f;
    p = fmaf(p, z, 0.02186295f);
    p = fmaf(p, z, -0.05591232f);
    p = fmaf(p, z, 0.09642197f);
    p = fmaf(p, z, -0.13908629f);
    p = fmaf(p, z, 0.19946566f);
    p = fmaf(p, z, -0.33329861f);
    p = fmaf(p, z, 0.99999934f);
    float r = p * a * 0.15915494309189535f;                   // [0, 1/8]
    r = ay > ax ? 0.25f - r : r;
    r = dx < 0.0f ? 0.5f - r : r;
    r = dy < 0.0f ? 1.0f - r : r;
    return r;
}

// Row floor(s) and weight t of angular interpolation in a column of n rows,
// for turns in [0, 1]: s = turns n - 0.5 lies in [-0.5, n - 0.5].
__device__ __forceinline__ int column_row(float n, float turns, float& t) {
    const float s = fmaf(turns, n, -0.5f);
    const float fs = floorf(s);
    t = s - fs;
    return (int)fs;
}

// Rows j0, j1 = j0 + 1 (mod n): floor(s) is in [-1, n - 1], only -1 wraps.
__device__ __forceinline__ void column_rows(int n, float turns, int& j0, int& j1, float& t) {
    j0 = column_row((float)n, turns, t);
    j0 = j0 < 0 ? j0 + n : j0;
    j1 = j0 + 1 == n ? 0 : j0 + 1;
}

// Weights of the four texels of a pixel between two columns (w) and between
// the two rows of each (t0, t1), every rounding stated: both samplers of a
// tile give the same image whichever tiles take which.
struct Weights {
    float a, b, c, d;
};
__device__ __forceinline__ Weights tap_weights(float w, float t0, float t1) {
    const float w0 = 1.0f - w;
    return Weights{fmaf(-w0, t0, w0), w0 * t0, fmaf(-w, t1, w), w * t1};
}

// Weighted sum of four texels.
__device__ __forceinline__ float4 blend4(float4 a, float wa, float4 b, float wb, float4 c, float wc, float4 d,
                                         float wd) {
    return make_float4(fmaf(wd, d.x, fmaf(wc, c.x, fmaf(wb, b.x, wa * a.x))),
                       fmaf(wd, d.y, fmaf(wc, c.y, fmaf(wb, b.y, wa * a.y))),
                       fmaf(wd, d.z, fmaf(wc, c.z, fmaf(wb, b.z, wa * a.z))),
                       fmaf(wd, d.w, fmaf(wc, c.w, fmaf(wb, b.w, wa * a.w))));
}

// Column coordinate a = u(e(rho)) - 0.5 (Eqs. (3), (5), (12)) from the
// FP64-built radial table, already clamped to the first and last column
// centres.
__device__ __forceinline__ float column_coord(const ReconView& v, __amdgpu_buffer_rsrc_t ut, float rho) {
    const float tq = fminf(rho * v.rho_scale, (float)kURhoN);
    const int k = (int)tq;
    const v2u uk = ld2(ut, (uint32_t)k * 8u);
    return fmaf(tq - (float)k, __uint_as_float(uk.y), __uint_as_float(uk.x)) - 0.5f;
}

// One staged column: LP offset and row count of the column, staged rows
// j_start .. j_start + cnt - 1 (mod n) at LDS texels base .. base + cnt - 1.
struct StageCol {
    uint32_t off;
    uint32_t n_cnt;     // n | cnt << 16
    uint32_t js_base;   // j_start | base << 16
};

// A staged column as sample_rows reads it: row j of its n rows, for js <= j
// <= js + last + 1, at LDS byte at + 16 j.
struct alignas(16) StageRow {
    float n;
    int at, js, last;
};

struct Stage {
    float4 tex[kStageTexels];
    StageCol col[kStageCols];
    StageRow row[kStageCols + 1];   // the last column of the buffer is followed by itself
    int i_lo, n_cols;       // staged columns i_lo .. i_lo + n_cols - 1 (n_cols = 0: nothing staged)
    int n_rows;             // entries of row[] (0: the tile takes the general sampler)
};

// Where texel j of the column described by (off, n, j_start, cnt, base)
// is: its LDS index when staged (else -1), and its LP byte offset.
struct Tap {
    int lds;
    uint32_t src;
};

__device__ __forceinline__ Tap tap_of(uint32_t off, int n, int js, int cnt, int base, int j) {
    int rel = j - js;
    rel = rel < 0 ? rel + n : rel;
    return Tap{rel < cnt ? base + rel : -1, (off + (uint32_t)j) * 16u};
}

// The texel of tap t in the LP buffer whose staged copy starts at LDS
// texel `half` (0, or kStageTexels / 2 for the second buffer of a pair).
__device__ __forceinline__ float4 texel(const Stage& st, __amdgpu_buffer_rsrc_t lp, int half, const Tap& t) {
    if (t.lds >= 0) return st.tex[half + t.lds];
    return ld4(lp, t.src);
}

// Column i's (offset, rows, staged range): staged columns from LDS, others
// from the column table with an empty staged range.
__device__ __forceinline__ void column_of(const Stage& st, __amdgpu_buffer_rsrc_t ct, int i, uint32_t& off, int& n,
                                          int& js, int& cnt, int& base) {
    const int c = i - st.i_lo;
    if ((unsigned)c < (unsigned)st.n_cols) {
        const StageCol sc = st.col[c];
        off = sc.off;
        n = (int)(sc.n_cnt & 0xffffu);
        cnt = (int)(sc.n_cnt >> 16);
        js = (int)(sc.js_base & 0xffffu);
        base = (int)(sc.js_base >> 16);
    } else {
        const v2u c2 = ld2(ct, (uint32_t)i * 8u);
        n = (int)c2.x;
        off = c2.y;
        js = 0;
        cnt = 0;
        base = 0;
    }
}

// Pixel at film offset (dx, dy) from the gaze point whose column coordinate
// a = u - 0.5 is already known: c from the LP buffer lp and, with kPair, c2
// from the paired buffer lp2 (same positions and weights).
template <bool kPair>
__device__ __forceinline__ void sample_vafr(const ReconView& v, const Stage& st, __amdgpu_buffer_rsrc_t lp,
                                            __amdgpu_buffer_rsrc_t lp2, __amdgpu_buffer_rsrc_t ct, float dx,
                                            float dy, float a, float4& c, float4& c2) {
    int i0 = (int)a;
    i0 = i0 > v.n_cols - 1 ? v.n_cols - 1 : (i0 < 0 ? 0 : i0);
    const int i1 = i0 + 1 < v.n_cols ? i0 + 1 : v.n_cols - 1;
    const float w = a - (float)i0;
    const float turns = angle_turns(dx, dy);
    uint32_t off0, off1;
    int n0, js0, cnt0, base0, n1, js1, cnt1, base1;
    column_of(st, ct, i0, off0, n0, js0, cnt0, base0);
    column_of(st, ct, i1, off1, n1, js1, cnt1, base1);
    int j00, j01, j10, j11;
    float t0, t1;
    column_rows(n0, turns, j00, j01, t0);
    column_rows(n1, turns, j10, j11, t1);
    const Tap ta = tap_of(off0, n0, js0, cnt0, base0, j00), tb = tap_of(off0, n0, js0, cnt0, base0, j01);
    const Tap tc = tap_of(off1, n1, js1, cnt1, base1, j10), td = tap_of(off1, n1, js1, cnt1, base1, j11);
    const Weights q = tap_weights(w, t0, t1);
    c = blend4(texel(st, lp, 0, ta), q.a, texel(st, lp, 0, tb), q.b, texel(st, lp, 0, tc), q.c, texel(st, lp, 0, td),
               q.d);
    if (kPair) {
        constexpr int h = kStageTexels / 2;
        c2 = blend4(texel(st, lp2, h, ta), q.a, texel(st, lp2, h, tb), q.b, texel(st, lp2, h, tc), q.c,
                    texel(st, lp2, h, td), q.d);
    }
}

// u / w of the LaFR kernel (Sec. 4.1 Eq. (15)) at log ratio z in [0, 1] of
// a pixel at squared distance r2 (FP64) from the gaze point.
//  - z <= Z_ef: (z (1 - Fa))^(1/Fa).
//  - z > Z_ef: Eq. (15)'s arccos piece, ((2 acos Za - pi) / pi)^(beta/0.7)
//    (1 - U_ef) + U_ef with Za = (1/z - 1/Z_ef) / (1/Z_ef - 1).  Next to the
//    farthest screen corner Za tends to -1, where acos has an unbounded
//    slope, so it is evaluated through eps = 1 + Za = (1 - z) / (z k),
//    k = 1/Z_ef - 1, and acos(eps - 1) = pi - 2 asin(sqrt(eps / 2)):
//    s = 1 - (4 / pi) asin(sqrt(eps / 2)).  1 - z = -ln q / (2 ln L) with
//    q = r2 / R2 and R the farthest corner's distance (ln R = ln L), q formed
//    in FP64: ln q is log1p(q - 1) for q > 1/2, so it keeps its relative
//    precision as r approaches R, and log(q) below (where q - 1 rounded to
//    FP32 would lose the small q's digits).
// kOne: one pixel at a time.  Its two logarithms are branches (3840x2160 in a
// batch of one row per thread: both and a select 73 us, LMFR 51; branches 42
// and 42); two pixels at a time overlap both logarithms of each better than
// they branch (640x361, 8 rows: 13.7 us, branches 14.2).  The difference from 1
// is formed by one FMA either way.
template <bool kOne>
__device__ __forceinline__ float lafr_u(const ReconView& v, float z, double r2) {
    if (z <= v.lf_zef) return powf(z * v.lf_fa1, v.lf_inv_fa);
    const double q = r2 * v.lf_inv_r2;
    float lq;
    if (!kOne) {
        lq = q > 0.5 ? log1pf((float)fma(r2, v.lf_inv_r2, -1.0)) : logf((float)q);
    } else if (q > 0.5) {
        float qm = (float)fma(r2, v.lf_inv_r2, -1.0);
        __asm__ volatile("" : "+v"(qm));
        lq = log1pf(qm);
    } else {
        float ql = (float)q;
        __asm__ volatile("" : "+v"(ql));
        lq = logf(ql);
    }
    const float omz = fmaxf(-lq * v.lf_half_inv_lnl, 0.0f);
    const float eps = fminf(omz / ((1.0f - omz) * v.lf_k), 1.0f);
    const float s = fmaf(-4.0f * (float)M_1_PI, asinf(__builtin_amdgcn_sqrtf(0.5f * eps)), 1.0f);
    return (v.lf_bexp == 1.0f ? s : powf(s, v.lf_bexp)) * (1.0f - v.lf_uef) + v.lf_uef;
}

// Texel offsets (bytes) and weights of a pixel of an LMFR / LaFR view.
struct DenseTaps {
    uint32_t o00, o01, o10, o11;
    float w, t;
};

// Pixel (x, y) of an LMFR / LaFR view: the offset from the gaze point is
// formed in FP64 (the gaze is a continuous FP64 position), then rounded.
template <bool kOne>
__device__ __forceinline__ DenseTaps dense_taps(const ReconView& v, int x, int y) {
    const double dxd = (double)x + v.lm_cx, dyd = (double)y + v.lm_cy;
    const float dx = (float)dxd, dy = (float)dyd;
    const double r2 = dxd * dxd + dyd * dyd;
    const float r = fmaxf(__builtin_amdgcn_sqrtf((float)r2), 1.0f);
    const float z = __log2f(r) * v.inv_L;                     // Eq. (1); inv_L = ln 2 / L
    float u = (v.lf_on ? lafr_u<kOne>(v, z, r2)                                      // Eq. (15)
                       : v.alpha == 4.0f ? (z * z) * (z * z) : __powf(z, v.alpha)) * (float)v.n_cols;   // Eq. (14)
    u = fminf(fmaxf(u, 0.5f), (float)v.n_cols - 0.5f);
    const float a = u - 0.5f;
    int i0 = (int)a;
    i0 = i0 > v.n_cols - 1 ? v.n_cols - 1 : i0;
    const int i1 = i0 + 1 < v.n_cols ? i0 + 1 : v.n_cols - 1;
    int j0, j1;
    float t;
    column_rows(v.lm_h, angle_turns(dx, dy), j0, j1, t);
    const uint32_t o0 = (uint32_t)(i0 * v.lm_h), o1 = (uint32_t)(i1 * v.lm_h);
    return DenseTaps{(o0 + j0) * 16u, (o0 + j1) * 16u, (o1 + j0) * 16u, (o1 + j1) * 16u, a - (float)i0, t};
}

// Wave 0: the staged columns of the tile whose pixel centres span film
// offsets [xl, xh] x [yl, yh] from the gaze point, written to st.col, and
// st.i_lo / st.n_cols (n_cols = 0 when the footprint does not fit).
__device__ void build_stage(const ReconView& v, Stage& st, __amdgpu_buffer_rsrc_t ut, __amdgpu_buffer_rsrc_t ct,
                            float xl, float xh, float yl, float yh, int budget) {
    const int lane = threadIdx.x;
    int n_cols = 0, i_lo = 0, n_rows = 0;
    const bool around_gaze = xl <= 0.0f && xh >= 0.0f && yl <= 0.0f && yh >= 0.0f;
    if (!around_gaze) {
        // radius range: nearest point of the rectangle and farthest corner
        const float qx = fminf(fmaxf(0.0f, xl), xh), qy = fminf(fmaxf(0.0f, yl), yh);
        const float fx = fmaxf(fabsf(xl), fabsf(xh)), fy = fmaxf(fabsf(yl), fabsf(yh));
        const float r_lo = __builtin_amdgcn_sqrtf(fmaf(qx, qx, qy * qy));
        const float r_hi = __builtin_amdgcn_sqrtf(fmaf(fx, fx, fy * fy));
        const int c_lo = (int)column_coord(v, ut, r_lo) - 1;
        const int c_hi = (int)column_coord(v, ut, r_hi) + 2;
        i_lo = c_lo < 0 ? 0 : c_lo;
        const int i_hi = c_hi > v.n_cols - 1 ? v.n_cols - 1 : c_hi;
        n_cols = i_hi - i_lo + 1;
        // angle range: the rectangle does not hold the gaze point, so the
        // extreme angles are those of its corners (taken about the centre
        // direction, which keeps the range unwrapped)
        // Each lane takes one corner's angle from the centre's (the angle of
        // (dot, cross), in [-1/2, 1/2] turns); groups of four lanes share
        // the extremes.
        const float rx = 0.5f * (xl + xh), ry = 0.5f * (yl + yh);
        const float ref = angle_turns(rx, ry);
        const float cx = lane & 1 ? xh : xl, cy = lane & 2 ? yh : yl;
        float d = angle_turns(fmaf(cx, rx, cy * ry), fmaf(cy, rx, -(cx * ry)));
        d = d >= 0.5f ? d - 1.0f : d;
        float lo = fminf(d, 0.0f), hi = fmaxf(d, 0.0f);
        lo = fminf(lo, __shfl_xor(lo, 1, 64));
        hi = fmaxf(hi, __shfl_xor(hi, 1, 64));
        lo = fminf(lo, __shfl_xor(lo, 2, 64));
        hi = fmaxf(hi, __shfl_xor(hi, 2, 64));
        lo += ref;
        hi += ref;
        if (n_cols > kStageCols) n_cols = 0;
        int cnt = 0, js = 0, n = 0, j_first = 0;
        uint32_t off = 0;
        if (lane < n_cols) {
            const v2u c2 = ld2(ct, (uint32_t)(i_lo + lane) * 8u);
            n = (int)c2.x;
            off = c2.y;
            if (n > 0xffff) n_cols = 0;   // the packed column record holds 16-bit row counts
            const int j_lo = (int)floorf(fmaf(lo, (float)n, -0.5f)) - 1;
            const int j_hi = (int)floorf(fmaf(hi, (float)n, -0.5f)) + 2;
            cnt = j_hi - j_lo + 1;
            j_first = j_lo;
            if (cnt >= n) {
                cnt = n;
                js = 0;
            } else {
                js = j_lo % n;
                js = js < 0 ? js + n : js;
            }
        }
        // inclusive prefix sum of the counts over the wave, by row shifts
        // within 16 lanes and broadcasts of lane 15 and lane 31
        int incl = cnt;
        incl += __builtin_amdgcn_update_dpp(0, incl, 0x111, 0xf, 0xf, true);    // row_shr:1
        incl += __builtin_amdgcn_update_dpp(0, incl, 0x112, 0xf, 0xf, true);    // row_shr:2
        incl += __builtin_amdgcn_update_dpp(0, incl, 0x114, 0xf, 0xf, true);    // row_shr:4
        incl += __builtin_amdgcn_update_dpp(0, incl, 0x118, 0xf, 0xf, true);    // row_shr:8
        incl += __builtin_amdgcn_update_dpp(0, incl, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
        incl += __builtin_amdgcn_update_dpp(0, incl, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
        const int total = __builtin_amdgcn_readlane(incl, 63);
        if (total > budget || __ballot(n_cols == 0) != 0) n_cols = 0;
        // a tile whose rows would wrap round the seam takes the general sampler
        const bool wraps = lane < n_cols && (j_first < 0 || j_first + cnt > n);
        if (n_cols > 0 && __ballot(wraps) == 0) n_rows = n_cols;
        if (lane < n_cols) {
            StageCol sc;
            sc.off = off;
            sc.n_cnt = (uint32_t)n | ((uint32_t)cnt << 16);
            sc.js_base = (uint32_t)js | ((uint32_t)(incl - cnt) << 16);
            st.col[lane] = sc;
            StageRow sr;
            sr.n = (float)n;
            sr.at = (incl - cnt - js) * 16;
            sr.js = js;
            sr.last = cnt - 2;
            st.row[lane] = sr;
            if (lane == n_cols - 1 && i_lo + n_cols == v.n_cols) st.row[n_cols] = sr;
        }
        if (n_rows > 0 && i_lo + n_cols == v.n_cols) ++n_rows;
    }
    if (lane == 0) {
        st.i_lo = i_lo;
        st.n_cols = n_cols;
        st.n_rows = n_rows;
    }
}

// Half a wave copies one column at a time (a peripheral tile of an 8K display
// has about ten columns of fourteen rows), its loads of up to four columns
// issued before the first LDS write.  With kPair the same texels of lp2 go
// to the upper half.
template <bool kPair>
__device__ __forceinline__ void fill_stage(Stage& st, __amdgpu_buffer_rsrc_t lp, __amdgpu_buffer_rsrc_t lp2) {
    constexpr int kHalves = kReconThreads / 32, kAhead = kPair ? 2 : 4;
    constexpr int h = kStageTexels / 2;
    const int half = threadIdx.x >> 5, r = threadIdx.x & 31;
    const int n_cols = st.n_cols;
    for (int c0 = half; c0 < n_cols; c0 += kHalves * kAhead) {
        float4 t[kAhead], t2[kPair ? kAhead : 1];
        int to[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const int c = c0 + q * kHalves;
            to[q] = -1;
            if (c < n_cols) {
                const StageCol sc = st.col[c];
                const int n = (int)(sc.n_cnt & 0xffffu), cnt = (int)(sc.n_cnt >> 16);
                const int js = (int)(sc.js_base & 0xffffu), base = (int)(sc.js_base >> 16);
                if (r < cnt) {
                    int j = js + r;
                    j = j >= n ? j - n : j;
                    const uint32_t src = (sc.off + (uint32_t)j) * 16u;
                    to[q] = base + r;
                    t[q] = ld4(lp, src);
                    if (kPair) t2[q] = ld4(lp2, src);
                }
                // longer columns (near the gaze) finish here
                for (int k = r + 32; k < cnt; k += 32) {
                    int j = js + k;
                    j = j >= n ? j - n : j;
                    const uint32_t src = (sc.off + (uint32_t)j) * 16u;
                    st.tex[base + k] = ld4(lp, src);
                    if (kPair) st.tex[h + base + k] = ld4(lp2, src);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < kAhead; ++q)
            if (to[q] >= 0) {
                st.tex[to[q]] = t[q];
                if (kPair) st.tex[h + to[q]] = t2[q];
            }
    }
}

// sample_vafr for a tile with StageRow records: the same coordinates and
// weights, but the two rows of each column are neighbours in LDS, so a pixel
// needs two addresses for its four texels and no wrap, clamp or fallback.
// Returns false if a texel is not staged (not expected: the bound has a texel
// of margin), for the caller to take the general sampler instead.
template <bool kPair>
__device__ __forceinline__ bool sample_rows(const Stage& st, int i_lo, int n_rows, float dx, float dy, float a,
                                            float4& c, float4& c2) {
    const int i0 = (int)a;
    const float w = a - (float)i0;
    const float turns = angle_turns(dx, dy);
    const int k = i0 - i_lo;
    bool staged = (unsigned)k < (unsigned)(n_rows - 1);
    const StageRow* rec = st.row + (staged ? k : 0);
    const StageRow s0 = rec[0], s1 = rec[1];
    float t0, t1;
    const int j0 = column_row(s0.n, turns, t0), j1 = column_row(s1.n, turns, t1);
    staged = staged && (unsigned)(j0 - s0.js) <= (unsigned)s0.last && (unsigned)(j1 - s1.js) <= (unsigned)s1.last;
    const char* base = reinterpret_cast<const char*>(st.tex);
    const float4* p0 = reinterpret_cast<const float4*>(base + (staged ? s0.at + j0 * 16 : 0));
    const float4* p1 = reinterpret_cast<const float4*>(base + (staged ? s1.at + j1 * 16 : 0));
    const Weights q = tap_weights(w, t0, t1);
    c = blend4(p0[0], q.a, p0[1], q.b, p1[0], q.c, p1[1], q.d);
    if (kPair) {
        constexpr int h = kStageTexels / 2;
        c2 = blend4(p0[h], q.a, p0[h + 1], q.b, p1[h], q.c, p1[h + 1], q.d);
    }
    return staged;
}

// Tile `id` of view v: 64 x 4P pixels, P rows per wave.  M is the mapping
// (kModeVafr / kModeLmfr) or -1 to read it from the view.  kPair: a VaFR
// view with a paired buffer (v.lp2, v.img2), written in the same pass.
template <int P, int M, bool kPair = false>
__device__ __forceinline__ void recon_tile(const ReconView& v, int id, Stage& st) {
    constexpr int kTileH = kWaves * P;
    const int nbx = (v.width + kTileW - 1) / kTileW;
    int bx, by;
    tile_of(id, nbx, bx, by);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int x = bx * kTileW + lane;
    const int y0 = by * kTileH;
    const int mode = M >= 0 ? M : v.mode;
    const __amdgpu_buffer_rsrc_t lp = rsrc(v.lp, v.lp_bytes);
    // the tile's rows start at a uniform base; offsets stay 32-bit
    const int rows = v.height - y0 < kTileH ? v.height - y0 : kTileH;
    const __amdgpu_buffer_rsrc_t img = rsrc(v.img + (size_t)y0 * v.width, (uint32_t)(rows * v.width) * 16u);
    if (mode == kModeVafr) {
        const __amdgpu_buffer_rsrc_t ut = rsrc(v.u_of_rho, (kURhoN + 1) * 8);
        const __amdgpu_buffer_rsrc_t ct = rsrc(v.col, (uint32_t)v.n_cols * 8);
        if (wave == 0) {
            const int x_hi = bx * kTileW + kTileW - 1 < v.width - 1 ? bx * kTileW + kTileW - 1 : v.width - 1;
            build_stage(v, st, ut, ct, fmaf((float)(bx * kTileW), v.sx, v.cx), fmaf((float)x_hi, v.sx, v.cx),
                        fmaf((float)y0, v.sy, v.cy), fmaf((float)(y0 + rows - 1), v.sy, v.cy),
                        kPair ? kStageTexels / 2 : kStageTexels);
        }
        const __amdgpu_buffer_rsrc_t lp2 = rsrc(kPair ? v.lp2 : v.lp, v.lp_bytes);
        const __amdgpu_buffer_rsrc_t img2 =
            rsrc((kPair ? v.img2 : v.img) + (size_t)y0 * v.width, (uint32_t)(rows * v.width) * 16u);
        __syncthreads();
        fill_stage<kPair>(st, lp, lp2);
        __syncthreads();
        if (x >= v.width) return;
        const float dx = fmaf((float)x, v.sx, v.cx);
        const int i_lo = st.i_lo, n_rows = st.n_rows;
        // the radial table entries of all P pixels are loaded before the
        // first store, so their latencies overlap
        float tq[P];
        v2u uk[P];
#pragma unroll
        for (int r = 0; r < P; ++r) {
            const float dy = fmaf((float)(y0 + wave * P + r), v.sy, v.cy);
            tq[r] = fminf(__builtin_amdgcn_sqrtf(fmaf(dx, dx, dy * dy)) * v.rho_scale, (float)kURhoN);
            uk[r] = ld2(ut, (uint32_t)(int)tq[r] * 8u);
        }
#pragma unroll
        for (int r = 0; r < P; ++r) {
            const int ty = wave * P + r;
            if (ty < rows) {
                const float dy = fmaf((float)(y0 + ty), v.sy, v.cy);
                const float k = (float)(int)tq[r];
                const float a = fmaf(tq[r] - k, __uint_as_float(uk[r].y), __uint_as_float(uk[r].x)) - 0.5f;
                float4 c, c2;
                bool done = false;
                if (n_rows > 0) done = sample_rows<kPair>(st, i_lo, n_rows, dx, dy, a, c, c2);
                if (!done) sample_vafr<kPair>(v, st, lp, lp2, ct, dx, dy, a, c, c2);
                store_px(img, (uint32_t)(ty * v.width + x) * 16u, c);
                if (kPair) store_px(img2, (uint32_t)(ty * v.width + x) * 16u, c2);
            }
        }
    } else {
        if (x >= v.width) return;
        // two rows at a time: all eight loads are issued before the first use
        constexpr int kRows = P < 2 ? 1 : 2;
        for (int r = 0; r < P; r += kRows) {
            const int ty = wave * P + r;
            DenseTaps t[kRows];
            float4 c[kRows][4];
#pragma unroll
            for (int q = 0; q < kRows; ++q) {
                t[q] = dense_taps<kRows == 1>(v, x, y0 + ty + q);
                c[q][0] = ld4(lp, t[q].o00);
                c[q][1] = ld4(lp, t[q].o01);
                c[q][2] = ld4(lp, t[q].o10);
                c[q][3] = ld4(lp, t[q].o11);
            }
#pragma unroll
            for (int q = 0; q < kRows; ++q) {
                const float w = t[q].w, s = t[q].t, w0 = 1.0f - w;
                if (ty + q < rows)
                    store_px(img, (uint32_t)((ty + q) * v.width + x) * 16u,
                             blend4(c[q][0], w0 - w0 * s, c[q][1], w0 * s, c[q][2], w - w * s, c[q][3], w * s));
            }
        }
    }
}

template <int P, int M>
__global__ __launch_bounds__(kReconThreads) void k_recon(const ReconView v) {
    __shared__ Stage st;
    recon_tile<P, M>(v, blockIdx.x, st);
}

// Batched launch over several views (block_end: running tile counts).  The
// view of workgroup b, and b's number within it.
__device__ __forceinline__ const ReconView& batch_view(const ReconView* __restrict__ views,
                                                       const int32_t* __restrict__ block_end, int32_t n_views,
                                                       int& b) {
    int vid = 0;
    while (vid + 1 < n_views && b >= block_end[vid]) ++vid;
    b -= vid ? block_end[vid - 1] : 0;
    return views[vid];
}

// Every view with P rows per thread (pairs take 1, 2 or 8, see recon_rows_of).
template <int P>
__global__ __launch_bounds__(kReconThreads) void k_recon_batch(const ReconView* __restrict__ views,
                                                             const int32_t* __restrict__ block_end, int32_t n_views) {
    __shared__ Stage st;
    int b = blockIdx.x;
    const ReconView& v = batch_view(views, block_end, n_views, b);
    if (P != 4 && v.lp2) recon_tile<P, kModeVafr, true>(v, b, st);
    else recon_tile<P, -1>(v, b, st);
}

// Views of different rows: pairs with 2, single VaFR views of large displays
// with 8, all others with 4.
__global__ __launch_bounds__(kReconThreads) void k_recon_mixed(const ReconView* __restrict__ views,
                                                               const int32_t* __restrict__ block_end,
                                                               int32_t n_views) {
    __shared__ Stage st;
    int b = blockIdx.x;
    const ReconView& v = batch_view(views, block_end, n_views, b);
    if (v.lp2) recon_tile<2, kModeVafr, true>(v, b, st);
    else if (v.rows == 8) recon_tile<8, kModeVafr>(v, b, st);
    else recon_tile<4, -1>(v, b, st);
}

}  // namespace

bool recon_rows_ok(int rows) { return rows == 1 || rows == 2 || rows == 4 || rows == 8; }

int64_t recon_blocks_of(const ReconView& v, int rows) {
    const int tile_h = kWaves * rows;
    return (int64_t)((v.width + kTileW - 1) / kTileW) * ((v.height + tile_h - 1) / tile_h);
}

int launch_reconstruct(const ReconView& v, hipStream_t stream) {
    const int64_t pixels = (int64_t)v.width * v.height;
    const int rows = v.mode != kModeVafr ? kReconRowsDense : pixels < kShortPixels ? 2 : pixels < kTallPixels ? 4 : 8;
    const int64_t blocks = recon_blocks_of(v, rows);
    if (blocks > 0x7fffffff) return fail(VAFR_E_UNSUPPORTED, "display too large");
    const dim3 g((unsigned)blocks), t(kReconThreads);
    if (v.mode != kModeVafr) hipLaunchKernelGGL((k_recon<kReconRowsDense, kModeLmfr>), g, t, 0, stream, v);
    else if (rows == 2) hipLaunchKernelGGL((k_recon<2, kModeVafr>), g, t, 0, stream, v);
    else if (rows == 4) hipLaunchKernelGGL((k_recon<4, kModeVafr>), g, t, 0, stream, v);
    else hipLaunchKernelGGL((k_recon<8, kModeVafr>), g, t, 0, stream, v);
    VAFR_HIP(hipGetLastError());
    return VAFR_OK;
}

const void* recon_batch_kernel(int rows) {
    switch (rows) {
        case 1: return reinterpret_cast<const void*>(&k_recon_batch<1>);
        case 2: return reinterpret_cast<const void*>(&k_recon_batch<2>);
        case 4: return reinterpret_cast<const void*>(&k_recon_batch<4>);
        case 8: return reinterpret_cast<const void*>(&k_recon_batch<8>);
        case kReconRowsMixed: return reinterpret_cast<const void*>(&k_recon_mixed);
        default: return nullptr;
    }
}

int launch_reconstruct_batch(const ReconView* views_dev, const int32_t* block_end_dev, int32_t n_views,
                             int32_t blocks, int rows, hipStream_t stream) {
    if (blocks <= 0) return VAFR_OK;
    if (rows != kReconRowsMixed && !recon_rows_ok(rows))
        return fail(VAFR_E_ARG, "reconstruction rows per thread must be 1, 2, 4 or 8");
    const dim3 g((unsigned)blocks), t(kReconThreads);
    switch (rows) {
        case kReconRowsMixed: hipLaunchKernelGGL(k_recon_mixed, g, t, 0, stream, views_dev, block_end_dev, n_views); break;
        case 1: hipLaunchKernelGGL(k_recon_batch<1>, g, t, 0, stream, views_dev, block_end_dev, n_views); break;
        case 2: hipLaunchKernelGGL(k_recon_batch<2>, g, t, 0, stream, views_dev, block_end_dev, n_views); break;
        case 4: hipLaunchKernelGGL(k_recon_batch<4>, g, t, 0, stream, views_dev, block_end_dev, n_views); break;
        default: hipLaunchKernelGGL(k_recon_batch<8>, g, t, 0, stream, views_dev, block_end_dev, n_views); break;
    }
    VAFR_HIP(hipGetLastError());
    return VAFR_OK;
}

}  // namespace vafr
