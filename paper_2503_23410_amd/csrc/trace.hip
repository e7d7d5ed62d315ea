// Ray generation, BVH traversal, watertight closest hit and shading for the
// LP buffer (Sec. 6.1: one ray per LP texel, closest-hit shading, miss
// shader), the LMFR / LaFR buffers and the full-resolution comparison.
//
// Build with -ffp-contract=off: the ray set-up and the triangle test below
// are written operation by operation so that every rounding is stated, and
// no multiply-add may be fused unless fmaf() says so.
#include <type_traits>

#include "vafr_internal.h"

namespace vafr {
namespace {

// Conservative slab test of the general form (Ize, "Robust BVH Ray
// Traversal", JCGT 2013): the exit distance is scaled by 1 + 2 gamma_3
// before the overlap test.  The fast form needs no scale: its roundings are
// covered by the boxes' padding (see node_slabs).
constexpr float kExitScale = 1.0000004f;
// Boxes are tested up to the current hit distance scaled by this factor,
// which covers the rounding of a triangle's t relative to its box.
constexpr float kHitSlack = 1.00001f;
constexpr float kTiny = 1e-30f;
// The fast slab form works on distances scaled by 2^-100 (see node_slabs).
// It takes rays whose largest direction component lies in [kFastDirLo,
// kFastDirHi], and raises components below kFastTiny (2^-57) to it: over the
// distances it admits, that moves a ray by less than 2^-27 of the padding.
constexpr float kDistScale = 0x1p-100f;
constexpr float kCodeScale = 0x1p49f;    // 2^149 kDistScale: a code read as the bits of a float is code x 2^-149
constexpr float kFastDirLo = 0x1p-10f, kFastDirHi = 0x1p20f;

// Scene arrays are read through global-address-space pointers: the loads
// become global (not flat) loads, which wait on the vector-memory counter
// only and do not serialise with the LDS stack traffic.
typedef float NFloat4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 ldg4(const float4* p, size_t i) {
    const NFloat4 v = ((const __attribute__((address_space(1))) NFloat4*)p)[i];
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint4 ldg_u4(const void* p) {
    const float4 v = ldg4(reinterpret_cast<const float4*>(p), 0);
    return make_uint4(__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w));
}
__device__ __forceinline__ int4 ldg_i4(const void* p) {
    const float4 v = ldg4(reinterpret_cast<const float4*>(p), 0);
    return make_int4(__float_as_int(v.x), __float_as_int(v.y), __float_as_int(v.z), __float_as_int(v.w));
}

// Node i (uniform over the wave) through the scalar cache.
typedef uint32_t SWord4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ BvhNode scalar_node(const BvhNode* nodes, int i) {
    const auto* p = (const __attribute__((address_space(4))) SWord4*)(nodes + i);
    const SWord4 a = p[0], b = p[1], c = p[2], d = p[3];
    BvhNode n;
    n.org = make_float4(__uint_as_float(a.x), __uint_as_float(a.y), __uint_as_float(a.z), __uint_as_float(a.w));
    n.q0 = make_uint4(b.x, b.y, b.z, b.w);
    n.q1 = make_uint4(c.x, c.y, c.z, c.w);
    n.ref = make_int4((int)d.x, (int)d.y, (int)d.z, (int)d.w);
    return n;
}

struct RayPre {
    float ox, oy, oz;
    float dx, dy, dz;
    float ix, iy, iz;       // 1/d with components below kFastTiny replaced by +-kFastTiny
    float oix, oiy, oiz;    // o * (1/d), rounded once, times kDistScale
    uint32_t mx, my, mz;    // ~0 where 1/d is negative (the box's high plane is entered first), else 0
    int kx, ky, kz;
    float Sx, Sy, Sz;
    bool valid;
};

__device__ __forceinline__ float sel3(int k, float a, float b, float c) { return k == 0 ? a : (k == 1 ? b : c); }

__device__ __forceinline__ void ray_setup(float ox, float oy, float oz, float dx, float dy, float dz, RayPre& r) {
    r.ox = ox; r.oy = oy; r.oz = oz;
    r.dx = dx; r.dy = dy; r.dz = dz;
    r.ix = 1.0f / (fabsf(dx) < kFastTiny ? copysignf(kFastTiny, dx) : dx);
    r.iy = 1.0f / (fabsf(dy) < kFastTiny ? copysignf(kFastTiny, dy) : dy);
    r.iz = 1.0f / (fabsf(dz) < kFastTiny ? copysignf(kFastTiny, dz) : dz);
    r.oix = ox * r.ix * kDistScale;
    r.oiy = oy * r.iy * kDistScale;
    r.oiz = oz * r.iz * kDistScale;
    r.mx = (uint32_t)((int)__float_as_uint(r.ix) >> 31);
    r.my = (uint32_t)((int)__float_as_uint(r.iy) >> 31);
    r.mz = (uint32_t)((int)__float_as_uint(r.iz) >> 31);
    // Watertight set-up: the axis of largest |d| becomes z (first on ties);
    // x, y follow cyclically and swap when d_z < 0.
    int kz = 0;
    float m = fabsf(dx);
    if (fabsf(dy) > m) { kz = 1; m = fabsf(dy); }
    if (fabsf(dz) > m) { kz = 2; }
    int kx = kz == 2 ? 0 : kz + 1;
    int ky = kx == 2 ? 0 : kx + 1;
    const float dkz = sel3(kz, dx, dy, dz);
    if (dkz < 0.0f) { const int t = kx; kx = ky; ky = t; }
    r.kx = kx; r.ky = ky; r.kz = kz;
    r.valid = dkz != 0.0f;
    const float dkx = sel3(kx, dx, dy, dz), dky = sel3(ky, dx, dy, dz);
    r.Sx = dkx / dkz;
    r.Sy = dky / dkz;
    r.Sz = 1.0f / dkz;
}

// The view's shadow ray from o: ray_setup along the light direction, whose
// part that does not depend on the origin the host prepared (six divisions,
// about 1% of a wave's issue cycles).
__device__ __forceinline__ void light_ray(const TraceView& v, const float3 o, RayPre& r) {
    r.ox = o.x; r.oy = o.y; r.oz = o.z;
    r.dx = v.light_dir[0]; r.dy = v.light_dir[1]; r.dz = v.light_dir[2];
    r.ix = v.light_inv[0]; r.iy = v.light_inv[1]; r.iz = v.light_inv[2];
    r.oix = o.x * r.ix * kDistScale;
    r.oiy = o.y * r.iy * kDistScale;
    r.oiz = o.z * r.iz * kDistScale;
    r.mx = (uint32_t)((int)__float_as_uint(r.ix) >> 31);
    r.my = (uint32_t)((int)__float_as_uint(r.iy) >> 31);
    r.mz = (uint32_t)((int)__float_as_uint(r.iz) >> 31);
    r.kx = v.light_axes & 3; r.ky = (v.light_axes >> 2) & 3; r.kz = v.light_axes >> 4;
    r.Sx = v.light_shear[0]; r.Sy = v.light_shear[1]; r.Sz = v.light_shear[2];
    r.valid = true;
    // Kept in vector registers: with a scalar operand a 2-cycle instruction
    // takes 4 (v_fma 0.36 against 0.22 per SIMD and clock).  Left as scalars
    // these constants made one eye on the 4.52M terrain 270 instead of 263 us
    // and LMFR(1.8) at 8K 1.27 instead of 1.22 ms.
    __asm__("" : "+v"(r.ix), "+v"(r.iy), "+v"(r.iz), "+v"(r.Sx), "+v"(r.Sy), "+v"(r.Sz));
    __asm__("" : "+v"(r.mx), "+v"(r.my), "+v"(r.mz), "+v"(r.kx), "+v"(r.ky), "+v"(r.kz));
}

// Component of (a0, a1, a2) on axis K when K is fixed at compile time, else
// on the lane's axis k.
template <int K>
__device__ __forceinline__ float comp(int k, float a0, float a1, float a2) {
    if constexpr (K == 0) return a0;
    else if constexpr (K == 1) return a1;
    else if constexpr (K == 2) return a2;
    else return sel3(k, a0, a1, a2);
}

// Axis permutation (kx, ky, kz) of the watertight set-up as one number,
// kz * 3 + kx (ky is the remaining axis).
constexpr int perm_code(int kx, int kz) { return kz * 3 + kx; }

// FP32 watertight ray/triangle test (Woop, Benthin, Wald, JCGT 2013).
// Returns true on a hit with t > 0 and writes t = T / det.  KX, KY, KZ fix
// the ray's axis permutation when every lane of the wave shares it, which
// turns the per-lane component selects into plain register choices; -1
// reads it from the ray.  Either way the same operations run on the same
// values.
template <int KX = -1, int KY = -1, int KZ = -1>
__device__ __forceinline__ bool tri_hit(const RayPre& r, float4 v0, float4 v1, float4 v2, float& t_out) {
    const float A0 = v0.x - r.ox, A1 = v0.y - r.oy, A2 = v0.z - r.oz;
    const float B0 = v1.x - r.ox, B1 = v1.y - r.oy, B2 = v1.z - r.oz;
    const float C0 = v2.x - r.ox, C1 = v2.y - r.oy, C2 = v2.z - r.oz;
    const float Akz = comp<KZ>(r.kz, A0, A1, A2), Bkz = comp<KZ>(r.kz, B0, B1, B2);
    const float Ckz = comp<KZ>(r.kz, C0, C1, C2);
    const float Ax = fmaf(-r.Sx, Akz, comp<KX>(r.kx, A0, A1, A2));
    const float Ay = fmaf(-r.Sy, Akz, comp<KY>(r.ky, A0, A1, A2));
    const float Bx = fmaf(-r.Sx, Bkz, comp<KX>(r.kx, B0, B1, B2));
    const float By = fmaf(-r.Sy, Bkz, comp<KY>(r.ky, B0, B1, B2));
    const float Cx = fmaf(-r.Sx, Ckz, comp<KX>(r.kx, C0, C1, C2));
    const float Cy = fmaf(-r.Sy, Ckz, comp<KY>(r.ky, C0, C1, C2));
    // Edge functions with plain products (a shared edge gets exactly
    // negated values in its two triangles).
    float U = Cx * By - Cy * Bx;
    float V = Ax * Cy - Ay * Cx;
    float W = Bx * Ay - By * Ax;
    if (U == 0.0f || V == 0.0f || W == 0.0f) {
        U = (float)((double)Cx * (double)By - (double)Cy * (double)Bx);
        V = (float)((double)Ax * (double)Cy - (double)Ay * (double)Cx);
        W = (float)((double)Bx * (double)Ay - (double)By * (double)Ax);
    }
    if ((U < 0.0f || V < 0.0f || W < 0.0f) && (U > 0.0f || V > 0.0f || W > 0.0f)) return false;
    const float det = (U + V) + W;
    if (det == 0.0f || !r.valid) return false;
    const float Az = r.Sz * Akz, Bz = r.Sz * Bkz, Cz = r.Sz * Ckz;
    const float T = (U * Az + V * Bz) + W * Cz;
    const float t = T / det;
    t_out = t;
    return t > 0.0f;
}

// Bitwise select (m ? a : b, bit by bit) and three-way or in one full-rate
// instruction each.  A wave64 v_fma / v_add / v_mul / v_sub, 32-bit add, and,
// or, xor, right shift, move or v_bitop3 issues in 2 cycles on gfx950; a
// compare, v_cndmask, min, max, byte conversion, left shift or any 64-bit
// operation takes 4 (measured with eight independent chains per lane: 0.38 -
// 0.44 against 0.22 - 0.24 instructions per SIMD and clock).  The node step
// below is written in the 2-cycle set where it can be.
__device__ __forceinline__ uint32_t bit_select(uint32_t m, uint32_t a, uint32_t b) {
    uint32_t r;
    __asm__("v_bitop3_b32 %0, %1, %2, %3 bitop3:0xca" : "=v"(r) : "v"(m), "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ uint32_t bit_or3(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    __asm__("v_bitop3_b32 %0, %1, %2, %3 bitop3:0xfe" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Orders two (distance bits << 32 | reference) pairs with one FP64 minimum
// and maximum: as doubles they compare by distance, then by reference.  No
// distance or +inf in the high word reads as an FP64 infinity or NaN (their
// exponents stay below 0x7ff), and the inline form keeps the compiler from
// canonicalising the operands first.  8 cycles against 20 for a compare and
// four selects.
__device__ __forceinline__ void pair_swap(double& a, double& b) {
    double lo, hi;
    __asm__("v_min_f64 %0, %1, %2" : "=v"(lo) : "v"(a), "v"(b));
    __asm__("v_max_f64 %0, %1, %2" : "=v"(hi) : "v"(a), "v"(b));
    a = lo;
    b = hi;
}

// Bits of code c of a plane word, as a float that is the code times
// 2^-149 2^(8 c) (c = 0, 1, 2) or times 2^-149 (c = 3): the bits of an FP32
// number below 2^24 are its value in units of 2^-149, subnormal or not.
template <int c>
__device__ __forceinline__ float code_bits(uint32_t w) {
    return __uint_as_float(c == 3 ? w >> 24 : w & (0xffu << (8 * c)));
}

// Byte c of a code word as a float (general form).
__device__ __forceinline__ float code(uint32_t w, int c) { return (float)((w >> (8 * c)) & 0xffu); }

// Slab distances of a node's quantised child boxes: miss[c] has its sign bit
// set unless child box c meets the ray over [0, tlim], tn[c] is the entry
// distance.  Per axis the node gives origin g and scale s = 2^k; a plane
// with code q lies at g + q s.  Along an axis with 1/d >= 0 the low plane is
// the entry plane, otherwise the high one: the distance is monotone in the
// code for either form below (every rounding is monotone), so choosing the
// plane words by the sign of 1/d gives exactly the min / max of the two
// distances.
//
// Fast form: distance = fma(q, s/d, fma(g, 1/d, -o/d)), everything scaled by
// kDistScale so that a code masked out of its word needs no conversion: read
// as a float it is q 2^-149, and the node holds s kCodeScale and g
// kDistScale (k_node_format).  Against the exact distance to the stored plane
// this is the distance to a plane moved by at most 2^-24 (|o| + |g - o| +
// 2 |plane - o|) (the roundings of 1/d, o/d and the two FMAs), at most an
// eighth of the padding of every stored box while every |o| component is at
// most TraceView::fma_origin_limit; results below 2^-126 lose at most 2^-49
// in distance.  So it needs no exit scale either.  An empty slot's codes are
// 255 / 0, a box turned inside out by at least 2 pad per axis, sixteen times
// those errors: never met (its reference is not looked at).
// Callers check the origin limit and the direction's range per wave.
// Against byte conversions, compares and selects on unscaled distances, this
// form and the stack's and loop's bookkeeping below measured: one eye on the
// 4.52M terrain 299 / 273 / 290 -> 267 / 242 / 253 us (three gazes), the
// binocular 8K batch 413 / 363 / 393 -> 372 / 330 / 355 us, 16 views 2.81 ->
// 2.53 ms, path-traced frames 1.48 -> 1.34 ms.
//
// General form (any finite origin and direction): each plane is decoded as
// fmaf(q, s, g), which the builder checked lies outside the child's padded
// box (up to the 2^-49 that an origin below 2^-26 loses in the device format,
// a billionth of the padding), and tested in the subtract-multiply form with
// unscaled distances; empty slots are skipped by their reference.
//
// kSeg: the ray is followed over [t_lo, tlim] only (distances as the form
// scales them), and may have narrowed tlim beforehand also as an any-hit ray.
template <bool kFast, bool kAny, bool kSeg>
__device__ __forceinline__ void node_slabs(const RayPre& r, const float4 org, const uint4 q0, const uint4 q1,
                                           const int4 ref, float tlim, float t_lo, float tn[4], uint32_t miss[4]) {
    const float sx = __uint_as_float(q1.z), sy = __uint_as_float(q1.w), sz = org.w;
    const uint32_t ex = bit_select(r.mx, q0.y, q0.x), xx = bit_select(r.mx, q0.x, q0.y);   // entry / exit codes
    const uint32_t ey = bit_select(r.my, q0.w, q0.z), xy = bit_select(r.my, q0.z, q0.w);
    const uint32_t ez = bit_select(r.mz, q1.y, q1.x), xz = bit_select(r.mz, q1.x, q1.y);
    if (kFast) {
        const float bx = fmaf(org.x, r.ix, -r.oix), by = fmaf(org.y, r.iy, -r.oiy), bz = fmaf(org.z, r.iz, -r.oiz);
        const float tx[3] = {sx * r.ix, sx * r.ix * 0x1p-8f, sx * r.ix * 0x1p-16f};
        const float ty[3] = {sy * r.iy, sy * r.iy * 0x1p-8f, sy * r.iy * 0x1p-16f};
        const float tz[3] = {sz * r.iz, sz * r.iz * 0x1p-8f, sz * r.iz * 0x1p-16f};
        auto child = [&](auto cc) {
            constexpr int c = decltype(cc)::value, m = c == 3 ? 0 : c;
            const float n = fmaxf(fmaxf(fmaf(code_bits<c>(ex), tx[m], bx), fmaf(code_bits<c>(ey), ty[m], by)),
                                  fmaf(code_bits<c>(ez), tz[m], bz));
            const float f = fminf(fminf(fmaf(code_bits<c>(xx), tx[m], bx), fmaf(code_bits<c>(xy), ty[m], by)),
                                  fmaf(code_bits<c>(xz), tz[m], bz));
            tn[c] = n;
            // met: entry <= exit, entry <= tlim, exit >= 0
            // (tlim stays +inf for an any-hit ray followed to its end)
            const float past = kSeg ? f - t_lo : f;
            miss[c] = kAny && !kSeg ? __float_as_uint(f - n) | __float_as_uint(past)
                                    : bit_or3(__float_as_uint(f - n), __float_as_uint(tlim - n), __float_as_uint(past));
        };
        child(std::integral_constant<int, 0>{});
        child(std::integral_constant<int, 1>{});
        child(std::integral_constant<int, 2>{});
        child(std::integral_constant<int, 3>{});
    } else {
        // the node's device format scaled back (powers of two)
        const float gx = org.x * 0x1p100f, gy = org.y * 0x1p100f, gz = org.z * 0x1p100f;
        const float ux = sx * 0x1p-49f, uy = sy * 0x1p-49f, uz = sz * 0x1p-49f;
        const int rf[4] = {ref.x, ref.y, ref.z, ref.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float nx = (fmaf(code(ex, c), ux, gx) - r.ox) * r.ix, fx = (fmaf(code(xx, c), ux, gx) - r.ox) * r.ix;
            const float ny = (fmaf(code(ey, c), uy, gy) - r.oy) * r.iy, fy = (fmaf(code(xy, c), uy, gy) - r.oy) * r.iy;
            const float nz = (fmaf(code(ez, c), uz, gz) - r.oz) * r.iz, fz = (fmaf(code(xz, c), uz, gz) - r.oz) * r.iz;
            tn[c] = fminf(fmaxf(fmaxf(nx, ny), fmaxf(nz, 0.0f)), 3.4e38f);   // +inf marks a miss
            const float tf = fminf(fminf(fx, fy), fminf(fz, tlim));
            const bool met = tn[c] <= tf * kExitScale && rf[c] != kEmptyRef &&
                             (!kSeg || fminf(fminf(fx, fy), fz) * kExitScale >= t_lo);
            miss[c] = met ? 0u : ~0u;
        }
    }
}

// Device format of the nodes, in place: origins times kDistScale, scales
// times kCodeScale (powers of two), empty slots' codes 255 / 0 (low / high).
__global__ __launch_bounds__(256) void k_node_format(BvhNode* nodes, int64_t n) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    BvhNode b = nodes[k];
    b.org = make_float4(b.org.x * kDistScale, b.org.y * kDistScale, b.org.z * kDistScale, b.org.w * kCodeScale);
    const uint32_t e = (b.ref.x == kEmptyRef ? 0xffu : 0u) | (b.ref.y == kEmptyRef ? 0xff00u : 0u) |
                       (b.ref.z == kEmptyRef ? 0xff0000u : 0u) | (b.ref.w == kEmptyRef ? 0xff000000u : 0u);
    b.q0 = make_uint4(b.q0.x | e, b.q0.y & ~e, b.q0.z | e, b.q0.w & ~e);
    b.q1 = make_uint4(b.q1.x | e, b.q1.y & ~e, __float_as_uint(__uint_as_float(b.q1.z) * kCodeScale),
                      __float_as_uint(__uint_as_float(b.q1.w) * kCodeScale));
    nodes[k] = b;
}

// Per-lane work counters of the diagnostic pass (node visits, each a test
// of a node's four child boxes; triangle tests).
struct WorkCount {
    uint32_t nodes = 0, tris = 0;
};

// Traversal loop shared by closest-hit and any-hit queries.
//
// Each step of the loop is wave-uniform: either a node step (lanes standing
// on an internal node test its four child boxes, continue with the nearest
// hit child and push the other hit children) or a triangle step (lanes
// holding a parked leaf test its triangles).  A lane parks the first leaf it
// reaches and keeps descending from its stack; the wave switches to the
// triangle step once kParkNum/kParkDen of its live lanes hold a parked leaf,
// or when no lane can take a node step.  This speculative order (Aila and
// Laine, "Understanding the efficiency of ray traversal on GPUs", HPG 2009)
// keeps more of the 64 lanes busy in both steps than descending and testing
// leaves in lock step.  Node steps taken before a parked leaf is tested use
// a hit distance that is not yet the smallest, so they only ever visit more
// boxes; the result is the same (t, id) minimum or the same any-hit bit.
constexpr int kParkNum = 5, kParkDen = 8;

// LDS entries per lane of stack class S (the rest of the stack is scratch).
constexpr int lds_entries(int s) { return s < kStackLds ? s : kStackLds; }

// Triangle step of one lane: the `count` triangles from `first` against the
// ray (axis permutation fixed by KX, KY, KZ, or -1 for the lane's own).
// Closest hit keeps the smallest (t, id) and narrows tlim; any hit stops at
// the first hit (slot_best = 1, ref = kEmptyRef).
template <int KX, int KY, int KZ, bool kAny, bool kFast>
__device__ __forceinline__ void leaf_test(const TraceView& sc, const RayPre& r, int first, int count, float& t_best,
                                          int& id_best, int& slot_best, float& tlim, int& ref) {
    const float4* tp = sc.tris + 3 * (size_t)first;
    for (int q = 0; q < count; ++q) {
        const float4 v0 = ldg4(tp, 3 * q), v1 = ldg4(tp, 3 * q + 1), v2 = ldg4(tp, 3 * q + 2);
        float t;
        if (tri_hit<KX, KY, KZ>(r, v0, v1, v2, t)) {
            if (kAny) {
                slot_best = 1;
                ref = kEmptyRef;
                break;
            }
            const int id = __float_as_int(v0.w);
            if (t < t_best || (t == t_best && id < id_best)) {
                t_best = t;
                id_best = id;
                slot_best = first + q;
                tlim = t * (kFast ? kHitSlack * kDistScale : kHitSlack);
            }
        }
    }
}

// Triangle step with the axis permutation fixed when perm names one (a
// wave-uniform value, so the choice is a scalar branch).
template <bool kAny, bool kPerm, bool kFast>
__device__ __forceinline__ void leaf_step(int perm, const TraceView& sc, const RayPre& r, int first, int count,
                                          float& tb, int& ib, int& sb, float& tl, int& ref) {
    if (kPerm) {
        if (perm == perm_code(1, 0)) return leaf_test<1, 2, 0, kAny, kFast>(sc, r, first, count, tb, ib, sb, tl, ref);
        if (perm == perm_code(2, 0)) return leaf_test<2, 1, 0, kAny, kFast>(sc, r, first, count, tb, ib, sb, tl, ref);
        if (perm == perm_code(2, 1)) return leaf_test<2, 0, 1, kAny, kFast>(sc, r, first, count, tb, ib, sb, tl, ref);
        if (perm == perm_code(0, 1)) return leaf_test<0, 2, 1, kAny, kFast>(sc, r, first, count, tb, ib, sb, tl, ref);
        if (perm == perm_code(0, 2)) return leaf_test<0, 1, 2, kAny, kFast>(sc, r, first, count, tb, ib, sb, tl, ref);
        if (perm == perm_code(1, 2)) return leaf_test<1, 0, 2, kAny, kFast>(sc, r, first, count, tb, ib, sb, tl, ref);
    }
    leaf_test<-1, -1, -1, kAny, kFast>(sc, r, first, count, tb, ib, sb, tl, ref);
}

// stk points at the block's LDS stack: entry e of thread x at stk[e B + x].
// Closest hit (kAny = false): smallest (t, triangle id); returns the stored
// slot or -1.  Any hit with t > 0 (kAny = true): returns 1 or -1.  With
// kPerm, perm is the rays' axis permutation (perm_code) when every lane of
// the wave shares it, else -1.  With kSeg the ray is followed over distances
// [seg.x, seg.y] only: every box that meets that range is visited, so a hit
// within it is found; hits outside it may be.  The first kBase entries of
// each lane's LDS column are left alone (they hold what waits for the result).
template <int B, int S, bool kAny, bool kCount, bool kFast, bool kPerm, bool kSeg, int kBase, bool kUni>
__device__ int traverse_loop(const TraceView& sc, const RayPre& r, int* stk, float& t_best, int& id_best,
                             WorkCount& wc, int perm, float2 seg) {
    t_best = INFINITY;
    id_best = -1;
    // Entries 0 .. kLds-1 in the lane's LDS column, the rest in scratch (the
    // two kept in separate branches and address spaces, so that the common
    // case stays an LDS access and the rare one a scratch access, neither a
    // generic one; volatile keeps the spill area in memory instead of in
    // registers).  The position is kept as the LDS byte offset of the next
    // free entry; the first holds kEmptyRef, so a pop needs no empty check.
    // Whether any lane is near the end of its LDS column is checked once per
    // node step, for the whole wave.
    constexpr int kLds = lds_entries(S);
    constexpr uint32_t kStep = 4u * B, kLdsEnd = kStep * kLds;
    int spill_mem[S + kStackSpill - kLds + kBase + 1];
    volatile __attribute__((address_space(5))) int* spill =
        (volatile __attribute__((address_space(5))) int*)spill_mem;
    auto lds = [&](uint32_t o) -> __attribute__((address_space(3))) int& {
        return *(__attribute__((address_space(3))) int*)((__attribute__((address_space(3))) char*)(stk) + o);
    };
    uint32_t sp = 4u * threadIdx.x + kBase * kStep;
    auto push = [&](bool checked, int v) {
        if (!checked || sp < kLdsEnd) lds(sp) = v;
        else spill[(sp - kLdsEnd) / kStep] = v;
        sp += kStep;
    };
    auto pop = [&]() {
        sp -= kStep;
        int v;
        if (sp < kLdsEnd) v = lds(sp);
        else v = spill[(sp - kLdsEnd) / kStep];
        return v;
    };
    push(false, kEmptyRef);
    if (kFast && kSeg) seg = make_float2(seg.x * kDistScale, seg.y * kDistScale);
    // boxes are tested over [0, t_best * kHitSlack] (times kDistScale in the
    // fast form), or over the segment
    float tlim = kSeg ? seg.y : INFINITY;
    int slot_best = -1;
    int ref = sc.root;   // kEmptyRef: nothing left to visit
    int parked = 0;      // parked leaf reference (< 0); 0 = none
    for (;;) {
        if (ref < 0 && ref != kEmptyRef && parked == 0) {
            parked = ref;
            ref = pop();
        }
        // a lane on a leaf reference holds a parked leaf as well
        const uint64_t at_node = __ballot(ref >= 0);
        const uint64_t holding = __ballot(parked != 0);
        const uint64_t live = at_node | holding;
        if (live == 0) break;
        if (at_node != 0 && kParkDen * __popcll(holding) < kParkNum * __popcll(live)) {
            if (ref >= 0) {
                if (kCount) ++wc.nodes;
                float tn[4];
                uint32_t miss[4];
                int4 rf;
                // kUni: a node that every active lane visits (35-46% of the
                // node steps of coherent rays) comes through the scalar
                // cache, which spares the vector path four 16-byte loads per
                // lane.  That pays where many waves keep the vector path
                // full: 2.60 -> 2.53 ms for a batch of 16 views on the 4.52M
                // terrain, 1.38 -> 1.34 ms per path-traced binocular frame.
                // A per-view launch waits for its longest waves instead, and
                // a scalar load is a wave's longer wait: without it 83 -> 80
                // us (283 thousand rays on the 1.13M terrain), 202 -> 198 us
                // (1.06M), 256 -> 250 us (LMFR, 2561x1441), 1.027 -> 1.010 ms
                // (LMFR(1.8), 8K), and 1% either way on the soup.
                const int ref0 = __builtin_amdgcn_readfirstlane(ref);
                if (kUni && __ballot(ref != ref0) == 0) {
                    const BvhNode n = scalar_node(sc.nodes, ref0);
                    rf = n.ref;
                    node_slabs<kFast, kAny, kSeg>(r, n.org, n.q0, n.q1, rf, tlim, seg.x, tn, miss);
                } else {
                    const float4* p = reinterpret_cast<const float4*>(sc.nodes + ref);
                    const float4 org = ldg4(p, 0);
                    const uint4 q0 = ldg_u4(p + 1), q1 = ldg_u4(p + 2);
                    rf = ldg_i4(p + 3);
                    node_slabs<kFast, kAny, kSeg>(r, org, q0, q1, rf, tlim, seg.x, tn, miss);
                }
                const bool near_end = __ballot(sp >= kLdsEnd - 3 * kStep) != 0;
                auto rest = [&](auto chk) {
                    constexpr bool checked = decltype(chk)::value;
                    if (kAny) {
                        // any hit needs no order: the last hit child next,
                        // the other hit children pushed
                        int nr = kEmptyRef;
                        if ((int)miss[0] >= 0) nr = rf.x;
                        if ((int)miss[1] >= 0) {
                            if (nr != kEmptyRef) push(checked, nr);
                            nr = rf.y;
                        }
                        if ((int)miss[2] >= 0) {
                            if (nr != kEmptyRef) push(checked, nr);
                            nr = rf.z;
                        }
                        if ((int)miss[3] >= 0) {
                            if (nr != kEmptyRef) push(checked, nr);
                            nr = rf.w;
                        }
                        ref = nr;
                    } else {
                        // nearest hit child next; the others pushed far first
                        const int kInf = 0x7f800000;
                        auto key = [&](int c, int rr) {
                            const uint32_t m = (uint32_t)((int)miss[c] >> 31);
                            return __hiloint2double((int)bit_select(m, kInf, __float_as_uint(tn[c])), rr);
                        };
                        double k0 = key(0, rf.x), k1 = key(1, rf.y), k2 = key(2, rf.z), k3 = key(3, rf.w);
                        pair_swap(k0, k1);
                        pair_swap(k2, k3);
                        pair_swap(k0, k2);
                        pair_swap(k1, k3);
                        pair_swap(k1, k2);
                        if (__double2hiint(k3) != kInf) push(checked, __double2loint(k3));
                        if (__double2hiint(k2) != kInf) push(checked, __double2loint(k2));
                        if (__double2hiint(k1) != kInf) push(checked, __double2loint(k1));
                        ref = __double2hiint(k0) != kInf ? __double2loint(k0) : kEmptyRef;
                    }
                };
                if (near_end) rest(std::true_type{});
                else rest(std::false_type{});
                if (ref == kEmptyRef) ref = pop();
            }
            continue;
        }
        if (parked != 0) {
            const int x = ~parked;
            parked = 0;
            const int first = x >> 3, count = (x & 7) + 1;
            if (kCount) wc.tris += count;
            leaf_step<kAny, kPerm, kFast>(perm, sc, r, first, count, t_best, id_best, slot_best, tlim, ref);
        }
    }
    return slot_best;
}

// The fast slab form is taken when every lane's origin and direction lie
// within its range (wave-uniform choice, so both loops run without
// divergence).
// kPerm: the triangle test's axis permutation is fixed for the whole
// traversal when every active lane shares it -- always for shadow rays (one
// light direction), and for most waves of primary rays (a wave covers a
// small screen patch).  The phased path kernels take it for their shadow
// rays only: bounce rays rarely share a permutation, and fixing it for
// every traversal there cost more in registers than it saved.
template <int B, int S, bool kAny, bool kCount, bool kPerm, bool kSeg = false, int kBase = 0, bool kUni = true>
__device__ __forceinline__ int traverse(const TraceView& sc, const RayPre& r, int* stk, float& t_best, int& id_best,
                                        WorkCount& wc, float2 seg = make_float2(0.0f, INFINITY)) {
    const float om = fmaxf(fmaxf(fabsf(r.ox), fabsf(r.oy)), fabsf(r.oz));
    const float dm = fmaxf(fmaxf(fabsf(r.dx), fabsf(r.dy)), fabsf(r.dz));
    const bool fast = om <= sc.fma_origin_limit && dm >= kFastDirLo && dm <= kFastDirHi;
    int perm = -1;
    if (kPerm) {
        const int pc = perm_code(r.kx, r.kz);
        const int p0 = __builtin_amdgcn_readfirstlane(pc);
        perm = __ballot(pc != p0) == 0 ? p0 : -1;
    }
    if (__ballot(!fast) == 0)
        return traverse_loop<B, S, kAny, kCount, true, kPerm, kSeg, kBase, kUni>(sc, r, stk, t_best, id_best, wc, perm,
                                                                                 seg);
    RayPre g = r;
    g.ix = 1.0f / (r.dx == 0.0f ? copysignf(kTiny, r.dx) : r.dx);
    g.iy = 1.0f / (r.dy == 0.0f ? copysignf(kTiny, r.dy) : r.dy);
    g.iz = 1.0f / (r.dz == 0.0f ? copysignf(kTiny, r.dz) : r.dz);
    return traverse_loop<B, S, kAny, kCount, false, kPerm, kSeg, kBase, kUni>(sc, g, stk, t_best, id_best, wc, perm, seg);
}

template <int B, int S, bool kCount, bool kPerm = false, int kBase = 0, bool kUni = true>
__device__ __forceinline__ int closest_hit(const TraceView& sc, const RayPre& r, int* stk, float& t_best,
                                           int& id_best, WorkCount& wc) {
    return traverse<B, S, false, kCount, kPerm, false, kBase, kUni>(sc, r, stk, t_best, id_best, wc);
}

template <int B, int S, bool kCount, bool kPerm = false, bool kUni = true>
__device__ __forceinline__ bool any_hit(const TraceView& sc, const RayPre& r, int* stk, WorkCount& wc) {
    float t;
    int id;
    return traverse<B, S, true, kCount, kPerm, false, 0, kUni>(sc, r, stk, t, id, wc) >= 0;
}

// 32-bit hash of Jarzynski and Olano, "Hash Functions for GPU Rendering",
// JCGT 9(3), 2020 (PCG output permutation of one LCG step).
__device__ __forceinline__ uint32_t pcg_hash(uint32_t v) {
    const uint32_t state = v * 747796405u + 2891336453u;
    const uint32_t word = ((state >> ((state >> 28u) + 4u)) ^ state) * 277803737u;
    return (word >> 22u) ^ word;
}

__device__ __forceinline__ float3 albedo_of(int id) {
    const uint32_t h = pcg_hash((uint32_t)id);
    return make_float3(0.2f + 0.7f * (float)(h & 255u) / 255.0f, 0.2f + 0.7f * (float)((h >> 8) & 255u) / 255.0f,
                       0.2f + 0.7f * (float)((h >> 16) & 255u) / 255.0f);
}

// Geometric normal facing the ray and the offset origin of the next ray.
__device__ __forceinline__ void hit_frame(const float4 v0, const float4 v1, const float4 v2, const RayPre& r, float t,
                                          float3& n, float3& os) {
    const float e1x = v1.x - v0.x, e1y = v1.y - v0.y, e1z = v1.z - v0.z;
    const float e2x = v2.x - v0.x, e2y = v2.y - v0.y, e2z = v2.z - v0.z;
    float nx = e1y * e2z - e1z * e2y;
    float ny = e1z * e2x - e1x * e2z;
    float nz = e1x * e2y - e1y * e2x;
    const float l2 = (nx * nx + ny * ny) + nz * nz;
    const float len = sqrtf(l2);
    if (len > 0.0f) { nx = nx / len; ny = ny / len; nz = nz / len; }
    const float nd = (nx * r.dx + ny * r.dy) + nz * r.dz;
    if (nd > 0.0f) { nx = -nx; ny = -ny; nz = -nz; }
    const float px = fmaf(t, r.dx, r.ox), py = fmaf(t, r.dy, r.oy), pz = fmaf(t, r.dz, r.oz);
    const float mx = fmaxf(fmaxf(fabsf(px), fabsf(py)), fabsf(pz));
    const float eps = 1e-4f * (1.0f + mx);
    n = make_float3(nx, ny, nz);
    os = make_float3(fmaf(eps, nx, px), fmaf(eps, ny, py), fmaf(eps, nz, pz));
}

__device__ __forceinline__ float rng01(const TraceView& v, uint32_t texel, uint32_t slot) {
    uint32_t h = pcg_hash(v.seed_lo);
    h = pcg_hash(h ^ v.seed_hi);
    h = pcg_hash(h ^ v.frame);
    h = pcg_hash(h ^ v.view);
    h = pcg_hash(h ^ texel);
    h = pcg_hash(h ^ slot);
    return (float)(h >> 8) * (1.0f / 16777216.0f);
}

// Cosine-weighted direction about n: rejection-sampled disk point (up to 8
// tries) lifted to the hemisphere, in the frame of Duff et al. (JCGT 2017).
__device__ __forceinline__ float3 cosine_dir(const TraceView& v, float3 n, uint32_t texel, uint32_t bounce) {
    float x = 0.0f, y = 0.0f;
    for (uint32_t tr = 0; tr < 8; ++tr) {
        const float r0 = rng01(v, texel, bounce * 32u + 2u * tr);
        const float r1 = rng01(v, texel, bounce * 32u + 2u * tr + 1u);
        const float xx = 2.0f * r0 - 1.0f, yy = 2.0f * r1 - 1.0f;
        if (xx * xx + yy * yy < 1.0f) { x = xx; y = yy; break; }
    }
    const float zz = (1.0f - x * x) - y * y;
    const float z = sqrtf(zz > 0.0f ? zz : 0.0f);
    const float s = copysignf(1.0f, n.z);
    const float a = -1.0f / (s + n.z);
    const float b = n.x * n.y * a;
    const float t1x = 1.0f + s * n.x * n.x * a, t1y = s * b, t1z = -s * n.x;
    const float t2x = b, t2y = s + n.y * n.y * a, t2z = -n.y;
    return make_float3((x * t1x + y * t2x) + z * n.x, (x * t1y + y * t2y) + z * n.y, (x * t1z + y * t2z) + z * n.z);
}

// Primary ray direction through film point (Px, Py): (Px R - Py U) + F,
// formed in FP64 operation by operation and rounded to FP32 once.
__device__ __forceinline__ void film_ray(const TraceView& v, double Px, double Py, RayPre& r) {
    float d[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double a = Px * (double)v.right[k];
        const double b = Py * (double)v.up[k];
        const double s = a - b;
        d[k] = (float)(s + (double)v.fwd[k]);
    }
    ray_setup(v.eye[0], v.eye[1], v.eye[2], d[0], d[1], d[2], r);
    __asm__("" : "+v"(r.ox), "+v"(r.oy), "+v"(r.oz));   // not as scalar operands, see light_ray
}

// LaFR (Sec. 4.1 Eq. (15)) column -> log ratio z, inverting the kernel piece
// that holds the column's abscissa t = (i + 1/2)/w; FP64 like the LMFR table.
// Out of line and with scalar arguments, so that it adds neither registers
// nor a private copy of the view to the traversal kernels.
__device__ __noinline__ double lafr_column_z(double t, double fa, double uef, double sexp, double zef_inv,
                                             double k) {
    if (t <= uef) return pow(t, fa) / (1.0 - fa);
    const double s = pow((t - uef) / (1.0 - uef), sexp);
    return 1.0 / (zef_inv - sin(0.5 * M_PI * s) * k);
}

// Item -> (ray, output slot).  Returns false for padding items.
__device__ __forceinline__ bool make_item_ray(const TraceView& v, int64_t k, RayPre& r, int64_t& out) {
    if (v.mode == kModeVafr) {
        // trace order: compact screen patches per wave
        const float2 o = v.dxy[k];
        film_ray(v, v.gx + (double)o.x, v.gy + (double)o.y, r);
        out = v.ord[k];
        return true;
    }
    if (v.mode == kModeLmfr) {
        // 8 x 8 tiles of (column, row) of the dense LMFR buffer
        const int tiles_j = (v.lm_h + 7) >> 3;
        const int64_t tile = k >> 6;
        const int w = (int)(k & 63);
        const int64_t i = (tile / tiles_j) * 8 + (w >> 3);
        const int64_t j = (tile % tiles_j) * 8 + (w & 7);
        if (i >= v.lm_w || j >= v.lm_h) return false;
        const double z = v.lf_on ? lafr_column_z(((double)i + 0.5) / (double)v.lm_w, v.lf_fa, v.lf_uef, v.lf_sexp,
                                                 v.lf_zef_inv, v.lf_k)
                                 : v.lm_z[i];
        const double rad = exp(v.lm_L * z);
        const double2 cs = v.lm_cs[j];
        film_ray(v, v.gx + (rad * cs.x) * v.px, v.gy + (rad * cs.y) * v.py, r);
        out = i * v.lm_h + j;
        return true;
    }
    // full resolution, 8 x 8 pixel tiles for coherent waves
    const int tiles_x = (v.width + 7) >> 3;
    const int64_t tile = k >> 6;
    const int w = (int)(k & 63);
    const int x = (int)(tile % tiles_x) * 8 + (w & 7);
    const int y = (int)(tile / tiles_x) * 8 + (w >> 3);
    if (x >= v.width || y >= v.height) return false;
    film_ray(v, ((double)x + 0.5 - 0.5 * (double)v.width) * v.px, ((double)y + 0.5 - 0.5 * (double)v.height) * v.py,
             r);
    out = (int64_t)y * v.width + x;
    return true;
}

// While the primary ray is traced its direction and output slot (below 2^32:
// no buffer has more than 65536 x 65536 items) wait outside the registers,
// which lets the Lambert-only kernels run eight waves per SIMD.  kSolo
// (per-view launches): in four entries at the bottom of the lane's LDS
// column, found again from the lane's number.  In scratch, where batches keep
// them, each wave pays a trip to memory that only a launch of many waves
// hides: 4,347 rays on the 17,664-triangle terrain took 15.8 us (12.9 with
// everything in registers at seven waves) and take 13.0, a 1280x720 view that
// sees nothing 16.8 (12.1) and 14.2, one eye of 1.06M rays on the 1.13M
// terrain 206 and 202, LMFR(1.8) at 8K 1.057 and 1.027 ms.  In LDS the
// batched kernel spills six registers inside its loop (binocular frame on the
// 4.52M terrain 346 -> 360 us).
template <int B, int S, bool kCount, bool kPerm, bool kSolo>
__device__ float4 shade_lambert(const TraceView& v, RayPre& r, int64_t& out, int* stk, int& id_out, WorkCount& wc,
                                uint32_t& n_shadow, float4& p_out) {
    const TraceView& sc = v;
    float t;
    int id, slot;
    if constexpr (kSolo) {
        static_assert(B == 64, "one wave: a lane's column is its number");
        volatile __attribute__((address_space(3))) int* keep = (volatile __attribute__((address_space(3))) int*)stk;
        const uint32_t at = threadIdx.x;
        keep[at] = __float_as_int(r.dx);
        keep[at + B] = __float_as_int(r.dy);
        keep[at + 2 * B] = __float_as_int(r.dz);
        keep[at + 3 * B] = (int)(uint32_t)out;
        slot = closest_hit<B, S, kCount, kPerm, 4, false>(sc, r, stk, t, id, wc);
        uint32_t lane;   // (formed here, not kept from above)
        __asm__ volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
        r.dx = __int_as_float(keep[lane]);
        r.dy = __int_as_float(keep[lane + B]);
        r.dz = __int_as_float(keep[lane + 2 * B]);
        out = (uint32_t)keep[lane + 3 * B];
    } else {
        int keep_mem[5];
        volatile __attribute__((address_space(5))) int* keep = (volatile __attribute__((address_space(5))) int*)keep_mem;
        keep[0] = __float_as_int(r.dx);
        keep[1] = __float_as_int(r.dy);
        keep[2] = __float_as_int(r.dz);
        keep[3] = (int)(uint32_t)out;
        keep[4] = (int)(out >> 32);
        slot = closest_hit<B, S, kCount, kPerm>(sc, r, stk, t, id, wc);
        r.dx = __int_as_float(keep[0]);
        r.dy = __int_as_float(keep[1]);
        r.dz = __int_as_float(keep[2]);
        out = (int64_t)keep[4] << 32 | (uint32_t)keep[3];
    }
    id_out = id;
    p_out = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (slot < 0) return make_float4(v.background[0], v.background[1], v.background[2], 1.0f);
    p_out = make_float4(fmaf(t, r.dx, r.ox), fmaf(t, r.dy, r.oy), fmaf(t, r.dz, r.oz), 1.0f);
    const float4* tp = sc.tris + 3 * (size_t)slot;
    float3 n, os;
    hit_frame(ldg4(tp, 0), ldg4(tp, 1), ldg4(tp, 2), r, t, n, os);
    const float ndl = (n.x * v.light_dir[0] + n.y * v.light_dir[1]) + n.z * v.light_dir[2];
    float vis = 1.0f;
    if (ndl > 0.0f && v.shadow) {
        RayPre s;
        light_ray(v, os, s);
        ++n_shadow;
        if (any_hit<B, S, kCount, kPerm, !kSolo>(sc, s, stk, wc)) vis = 0.0f;
    }
    const float lam = ndl > 0.0f ? ndl : 0.0f;
    const float3 a = albedo_of(id);
    return make_float4(a.x * (v.ambient[0] + v.light_rgb[0] * lam * vis),
                       a.y * (v.ambient[1] + v.light_rgb[1] * lam * vis),
                       a.z * (v.ambient[2] + v.light_rgb[2] * lam * vis), 1.0f);
}

// Path from bounce b0 (ray r, throughput thr, radiance L so far): returns
// true when the path has ended (L final), false when it stopped after
// bounce b_last with r set to the next ray.  Bounce 0 reports the primary
// hit id and point.
template <int B, int S, bool kCount>
__device__ bool path_segment(const TraceView& v, RayPre& r, uint32_t texel, int* stk, float3& thr, float3& L,
                             int b0, int b_last, int& id_out, float4& p_out, WorkCount& wc, uint32_t& n_shadow) {
    const TraceView& sc = v;
    for (int bnc = b0; bnc <= v.bounces; ++bnc) {
        float t;
        int id;
        const int slot = closest_hit<B, S, kCount>(sc, r, stk, t, id, wc);
        if (bnc == 0) {
            id_out = id;
            if (slot >= 0) p_out = make_float4(fmaf(t, r.dx, r.ox), fmaf(t, r.dy, r.oy), fmaf(t, r.dz, r.oz), 1.0f);
        }
        if (slot < 0) {
            L.x += thr.x * v.background[0];
            L.y += thr.y * v.background[1];
            L.z += thr.z * v.background[2];
            return true;
        }
        const float4* tp = sc.tris + 3 * (size_t)slot;
        float3 n, os;
        hit_frame(ldg4(tp, 0), ldg4(tp, 1), ldg4(tp, 2), r, t, n, os);
        const float ndl = (n.x * v.light_dir[0] + n.y * v.light_dir[1]) + n.z * v.light_dir[2];
        float vis = 0.0f;
        if (ndl > 0.0f) {
            RayPre s;
            light_ray(v, os, s);
            ++n_shadow;
            vis = any_hit<B, S, kCount>(sc, s, stk, wc) ? 0.0f : 1.0f;
        }
        const float3 a = albedo_of(id);
        thr = make_float3(thr.x * a.x, thr.y * a.y, thr.z * a.z);
        L.x += thr.x * (v.ambient[0] + v.light_rgb[0] * ndl * vis);
        L.y += thr.y * (v.ambient[1] + v.light_rgb[1] * ndl * vis);
        L.z += thr.z * (v.ambient[2] + v.light_rgb[2] * ndl * vis);
        if (bnc == v.bounces) return true;
        const float3 w = cosine_dir(v, n, texel, (uint32_t)bnc);
        ray_setup(os.x, os.y, os.z, w.x, w.y, w.z, r);
        if (bnc == b_last) return false;
    }
    return true;
}

template <int B, int S, bool kCount>
__device__ float4 shade_path(const TraceView& v, RayPre r, uint32_t texel, int* stk, int& id_out, WorkCount& wc,
                             uint32_t& n_shadow, float4& p_out) {
    float3 thr = make_float3(1.0f, 1.0f, 1.0f);
    float3 L = make_float3(0.0f, 0.0f, 0.0f);
    id_out = -1;
    p_out = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    path_segment<B, S, kCount>(v, r, texel, stk, thr, L, 0, 0x7fffffff, id_out, p_out, wc, n_shadow);
    return make_float4(L.x, L.y, L.z, 1.0f);
}

// Compiler-level memory fence: memory written before it is stored before
// it, and memory read after it is loaded again, so that the path state of a
// phased path-mode bounce lives in memory, not in registers, while a
// traversal runs (no instruction is emitted).
__device__ __forceinline__ void state_fence() { __asm__ __volatile__("" ::: "memory"); }

// Bounce `bnc` of a phased path-mode view (batched launches): path p (its
// trace item) with ray r and output index `out`; its throughput and
// radiance so far are (1, 1, 1) and 0 on bounce 0 and come from the path's
// state on later bounces.  The same operations as path_segment, in the
// same order: closest hit; a miss adds thr x background and ends the path;
// a hit multiplies thr by the albedo, and when bounces remain writes the
// next ray (cosine-weighted about the face-forwarded normal, keyed by
// (texel, bnc)) to the path's state and, with `list`, lists p for bounce
// bnc + 1 (one atomic per wave); then the shadow ray toward the light when
// n.l > 0, and L += thr (ambient + light n.l vis), the final radiance on
// the last bounce.  Returns whether the path continues (its next ray is in
// the state).
// Throughput and radiance are read from the state after the closest-hit
// traversal, and throughput, n.l and radiance go through it across the
// shadow ray, so none of them is live during a traversal.  Bounce 0
// reports the primary hit id and point.
template <int B, int S>
__device__ bool path_bounce(const TraceView& v, RayPre& r, int32_t p, int32_t out, int bnc, int* stk, bool list) {
    WorkCount wc;
    float t;
    int id;
    const int slot = closest_hit<B, S, false>(v, r, stk, t, id, wc);
    if (bnc == 0) {
        if (v.out_id) v.out_id[out] = id;
        if (v.out_p)
            v.out_p[out] = slot >= 0 ? make_float4(fmaf(t, r.dx, r.ox), fmaf(t, r.dy, r.oy), fmaf(t, r.dz, r.oz), 1.0f)
                                     : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    float4* st = v.pt_state + 4 * (size_t)p;
    state_fence();
    float3 thr = make_float3(1.0f, 1.0f, 1.0f), L = make_float3(0.0f, 0.0f, 0.0f);
    if (bnc > 0) {
        const float4 th = st[2], lr = st[3];
        thr = make_float3(th.x, th.y, th.z);
        L = make_float3(lr.x, lr.y, lr.z);
    }
    if (slot < 0) {
        L.x += thr.x * v.background[0];
        L.y += thr.y * v.background[1];
        L.z += thr.z * v.background[2];
        v.out_rgba[out] = make_float4(L.x, L.y, L.z, 1.0f);
        return false;
    }
    const float4* tp = v.tris + 3 * (size_t)slot;
    float3 n, os;
    hit_frame(ldg4(tp, 0), ldg4(tp, 1), ldg4(tp, 2), r, t, n, os);
    const float ndl = (n.x * v.light_dir[0] + n.y * v.light_dir[1]) + n.z * v.light_dir[2];
    const float3 a = albedo_of(id);
    thr = make_float3(thr.x * a.x, thr.y * a.y, thr.z * a.z);
    const bool more = bnc < v.bounces;
    if (more) {
        const float3 w = cosine_dir(v, n, (uint32_t)out, (uint32_t)bnc);
        st[0] = make_float4(os.x, os.y, os.z, __int_as_float(out));
        st[1] = make_float4(w.x, w.y, w.z, 0.0f);
        if (list) {
            const uint64_t m = __ballot(1);
            const int lane = (int)__lane_id();
            const int leader = __builtin_ctzll(m);
            uint32_t base = 0;
            if (lane == leader) base = atomicAdd(v.pt_count + bnc + 1, (uint32_t)__popcll(m));
            base = __shfl(base, leader, 64);
            v.pt_list[((bnc + 1) & 1) * v.n_items + base + __popcll(m & ((1ull << lane) - 1ull))] = p;
        }
    }
    st[2] = make_float4(thr.x, thr.y, thr.z, ndl);
    st[3] = make_float4(L.x, L.y, L.z, 0.0f);
    float vis = 0.0f;
    state_fence();
    if (ndl > 0.0f) {
        RayPre s;
        light_ray(v, os, s);
        vis = any_hit<B, S, false, true>(v, s, stk, wc) ? 0.0f : 1.0f;
    }
    state_fence();
    const float4 th = st[2], lr = st[3];
    const float4 c = make_float4(lr.x + th.x * (v.ambient[0] + v.light_rgb[0] * th.w * vis),
                                 lr.y + th.y * (v.ambient[1] + v.light_rgb[1] * th.w * vis),
                                 lr.z + th.z * (v.ambient[2] + v.light_rgb[2] * th.w * vis), more ? 0.0f : 1.0f);
    if (more) st[3] = c;
    else v.out_rgba[out] = c;
    return more;
}

// One ray per thread: item `k` of view `v`.  kCount: diagnostic pass that
// counts work into counters[0..3] = primary rays, shadow rays, node visits,
// triangle tests, and writes no image.  kPhased: path-mode views of the
// launch run their bounce 0 as the first phase of path_bounce (batched
// launches only).  kLambert: every view of the launch is Lambert-shaded, so
// the path-tracing code is left out of the kernel.  kSolo: the launch has one
// view.
template <int B, int S, bool kCount, bool kPhased = false, bool kLambert = false, bool kSolo = false>
__device__ __forceinline__ void trace_item(const TraceView& v, int64_t k, int* stack, unsigned long long* counters) {
    RayPre r;
    int64_t out;
    if (k >= v.n_items || !make_item_ray(v, k, r, out)) return;
    int* stk = stack;
    if (kPhased && v.pt_phased) {
        // bounces 0 .. kPathFuse by this thread (few paths end before then,
        // and this launch's blocks are XCD-aware and planned); a path still
        // alive after bounce kPathFuse is listed for the queue launches
        const float4* st = v.pt_state + 4 * (size_t)k;
        for (int bnc = 0;; ++bnc) {
            if (!path_bounce<B, S>(v, r, (int32_t)k, (int32_t)out, bnc, stk, bnc >= kPathFuse) || bnc >= kPathFuse)
                break;
            const float4 e0 = st[0], e1 = st[1];
            ray_setup(e0.x, e0.y, e0.z, e1.x, e1.y, e1.z, r);
        }
        return;
    }
    int id;
    float4 c, p;
    WorkCount wc;
    uint32_t n_shadow = 0;
    if (!kLambert && !kPhased && v.shade_mode == VAFR_SHADE_PATH)
        c = shade_path<B, S, kCount>(v, r, (uint32_t)out, stk, id, wc, n_shadow, p);
    else
        c = shade_lambert<B, S, kCount, kLambert, kSolo>(v, r, out, stk, id, wc, n_shadow, p);
    if (kCount) {
        atomicAdd(counters + 0, 1ull);
        atomicAdd(counters + 1, (unsigned long long)n_shadow);
        atomicAdd(counters + 2, (unsigned long long)wc.nodes);
        atomicAdd(counters + 3, (unsigned long long)wc.tris);
        return;
    }
    v.out_rgba[out] = c;
    if (v.out_id) v.out_id[out] = id;
    if (v.out_p) v.out_p[out] = p;
}

// Register budget of the traversal kernels, in waves per SIMD (512 VGPRs per
// lane over that many waves, in allocation steps of 8).  Kernels that trace
// whole paths in one pass (per view and over the reprojection's list) keep
// five waves (at most 96 VGPRs): below that their extra state spills.
// The Lambert-only kernels, which keep the primary ray's direction and
// output slot elsewhere while it is traced, and the phased path-mode
// kernels, which hold no path state across a traversal, take the eight-wave
// budget (64 VGPRs); at the 69 VGPRs the former take otherwise, an eye of
// 1.06M rays on the 1.13M terrain takes 210 us instead of 198 and LMFR(1.8) at
// 8K 1.08 ms instead of 1.01.  The Lambert-shaded list, which also holds the
// rays shared by four lanes, needs 69.
#define kTraceWaves(lambert) __attribute__((amdgpu_waves_per_eu((lambert) ? 8 : 5)))
#define kListWaves(lambert) __attribute__((amdgpu_waves_per_eu((lambert) ? 6 : 5)))
#define kBatchWaves(lambert, phased) __attribute__((amdgpu_waves_per_eu((phased) || (lambert) ? 8 : 5)))

// Workgroups are dispatched to the 8 XCDs round-robin (workgroup id b runs
// on XCD b % 8).  Work is dealt to the XCDs in chunks of kXcdChunk
// consecutive rays in trace order: chunk c goes to XCD c % 8.  A chunk is a
// compact screen patch whose rays share the BVH levels near the leaves in
// their XCD's L2, and every XCD gets chunks from all over the screen, so that
// none of them holds more than its share of the expensive rays.  One
// contiguous eighth of the rays per XCD left the XCD with the worst screen
// region running alone.  Measured, contiguous eighths -> chunks of 1024
// rays: one eye on the 4.52M terrain 304 / 295 / 315 -> 299 / 274 / 290 us
// (three gazes), binocular 8K batch 414 / 402 / 430 -> 416 / 366 / 396 us,
// LMFR(1.8) at 8K 1.68 -> 1.45 / 1.33 ms, 2560x1440 full resolution 0.62 ->
// 0.54 ms, the 4,096-triangle soup 5.35 -> 3.55 ms.  Chunks of 128 to 4096
// rays are within 2% of each other; 16384 is 3% slower on batches.
constexpr int kXcds = 8;
constexpr int kXcdChunk = 1024;

// Work block of the i-th workgroup on XCD x, of per = workgroups / 8 on each
// (a permutation of 0 .. 8 per - 1; the rest of a partial last chunk is
// shared out contiguously).
template <int B>
__device__ __forceinline__ int xcd_work(int x, int i, int per) {
    constexpr int kChunk = kXcdChunk / B;
    const int whole = per / kChunk * kChunk;
    if (i >= whole) return kXcds * whole + x * (per - whole) + (i - whole);
    return (i / kChunk * kXcds + x) * kChunk + i % kChunk;
}

// Work block of workgroup b of n; ids past the last multiple of 8 keep their
// place.
template <int B>
__device__ __forceinline__ int xcd_block(int b, int n) {
    const int per = n / kXcds;
    return b < per * kXcds ? xcd_work<B>(b % kXcds, b / kXcds, per) : b;
}

// S = stack entries per lane (the scene's stack class).
template <int B, int S, bool kCount, bool kLambert>
__global__ __launch_bounds__(B) kTraceWaves(kLambert) void k_trace(const TraceView v, unsigned long long* counters) {
    __shared__ int stack[lds_entries(S) * B];
    const int b = xcd_block<B>(blockIdx.x, gridDim.x);
    trace_item<B, S, kCount, false, kLambert, kLambert>(v, (int64_t)b * B + threadIdx.x, stack, counters);
}

// Bounce `bounce` > kPathFuse of the phased path-mode views (batched): workgroup b
// serves view vid with qblock_end[vid-1] <= b < qblock_end[vid]; its thread q
// traces path list[q] of the bounce while q < pt_count[bounce] (workgroups
// past the count exit at once).
template <int S>
__global__ __launch_bounds__(kQueueBlock) kBatchWaves(false, true) void k_trace_queue_batch(
    const TraceView* __restrict__ views, const int32_t* __restrict__ qblock_end, int32_t n_views, int32_t bounce) {
    __shared__ int stack[lds_entries(S) * kQueueBlock];
    const int b = blockIdx.x;
    int vid = 0;
    while (vid + 1 < n_views && b >= qblock_end[vid]) ++vid;
    const TraceView& v = views[vid];
    const int first = vid ? qblock_end[vid - 1] : 0;
    const int64_t q = (int64_t)(b - first) * kQueueBlock + threadIdx.x;
    if (!v.pt_phased || bounce > v.bounces || q >= (int64_t)v.pt_count[bounce]) return;
    const int32_t p = v.pt_list[(bounce & 1) * v.n_items + q];
    const float4* e = v.pt_state + 4 * (size_t)p;
    const float4 e0 = e[0], e1 = e[1];
    RayPre r;
    ray_setup(e0.x, e0.y, e0.z, e1.x, e1.y, e1.z, r);
    path_bounce<kQueueBlock, S>(v, r, p, __float_as_int(e0.w), bounce, stack, true);
}

// List mode: items item_list[0 .. *item_count), by a grid for the longest list
// (workgroups past the count exit at once).  A fixed grid of 8192 workgroups
// that took long lists in rounds left the last round to a few of them: all
// 1.06M texels of an eye on the 1.13M terrain 442 -> 342 us, path-traced 1328
// -> 1046 us.  Lambert and path shading have kernels of their own: in one
// kernel the two forms below and the path code spilled 88 registers (binocular
// frame with 92 thousand holes 521 -> 495 us).
//
// The texels that a left eye leaves uncovered are mostly the longest rays of
// a frame (they skim the surface), and a short list of them leaves most of
// the chip idle while the last of them walk their nodes one after the other:
// up to kSplitItems Lambert-shaded items, when they are at most one in
// kSplitShare of the view's, are therefore followed by kSplit lanes each, a
// part of the way per lane.  A longer list fills the chip with a lane each,
// and one that holds a larger share of the texels holds ordinary rays as
// well, which are too short to share.  Whole frames, one lane -> four: 1.06M
// texels on the 4.52M terrain, 28 thousand listed 523 -> 475 us, 86 thousand
// 535 -> 489, 145 thousand 563 -> 557, 188 thousand 900 -> 903, 346 thousand
// 949 -> 1036; 4.25M texels, 100 thousand 1205 -> 1137, 227 thousand 1206 ->
// 1188, 330 thousand 1232 -> 1250; 487 thousand texels on the 1.13M terrain, 66
// thousand 255 -> 251, 106 thousand 265 -> 279; 76 thousand texels, 66
// thousand listed 122 -> 124.  Eight lanes and more were slower (four / 8 / 16 /
// 32: 527 / 534 / 646 / 733 us).
constexpr int kSplit = 4;
constexpr int kSplitItems = 196608;
constexpr int kSplitShare = 5;
static_assert(kSplit <= kSplitShare, "one lane per item of the view is lanes enough");

// Segment c of the kSplit equal ones that cut the ray's way through the scene's
// box; the first reaches back to the origin and the last on to infinity, and
// each begins a little early (the rounding of a hit's distance, kHitSlack).
__device__ __forceinline__ float2 ray_segment(const TraceView& v, const RayPre& r, int c) {
    float t0 = 0.0f, t1 = INFINITY;
    const float o[3] = {r.ox, r.oy, r.oz}, i[3] = {r.ix, r.iy, r.iz};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float a = (v.lo[k] - o[k]) * i[k], b = (v.hi[k] - o[k]) * i[k];
        t0 = fmaxf(t0, fminf(a, b));
        t1 = fminf(t1, fmaxf(a, b));
    }
    const float step = fmaxf((1.0f / kSplit) * (t1 - t0), 0.0f);
    return make_float2(c == 0 ? 0.0f : (t0 + (float)c * step) * (2.0f - kHitSlack),
                       c == kSplit - 1 ? INFINITY : (t0 + (float)(c + 1) * step) * kHitSlack);
}

// shade_lambert of item k by kSplit lanes, each following its segment of the
// primary and of the shadow ray; lane c = 0 writes the outputs.
template <int B, int S>
__device__ void trace_item_split(const TraceView& v, int64_t k, int c, int* stk) {
    RayPre r;
    int64_t out;
    if (!make_item_ray(v, k, r, out)) return;
    WorkCount wc;
    float t;
    int id;
    int slot = traverse<B, S, false, false, false, true, 0, false>(v, r, stk, t, id, wc, ray_segment(v, r, c));
    // the group's least (t, id); lanes without a hit hold (+inf, -1)
    auto least = [&](float ot, int oi, int os) {
        if (ot < t || (ot == t && oi < id)) {
            t = ot;
            id = oi;
            slot = os;
        }
    };
#pragma unroll
    for (int m = 1; m < kSplit; m <<= 1) {
        const float ot = __shfl_xor(t, m, 64);
        const int oi = __shfl_xor(id, m, 64), os = __shfl_xor(slot, m, 64);
        least(ot, oi, os);
    }
    float4 rgba = make_float4(v.background[0], v.background[1], v.background[2], 1.0f);
    float4 p = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (slot >= 0) {
        p = make_float4(fmaf(t, r.dx, r.ox), fmaf(t, r.dy, r.oy), fmaf(t, r.dz, r.oz), 1.0f);
        const float4* tp = v.tris + 3 * (size_t)slot;
        float3 n, os;
        hit_frame(ldg4(tp, 0), ldg4(tp, 1), ldg4(tp, 2), r, t, n, os);
        const float ndl = (n.x * v.light_dir[0] + n.y * v.light_dir[1]) + n.z * v.light_dir[2];
        float vis = 1.0f;
        if (ndl > 0.0f && v.shadow) {
            RayPre s;
            light_ray(v, os, s);
            float ts;
            int ids;
            int any = traverse<B, S, true, false, true, true, 0, false>(v, s, stk, ts, ids, wc, ray_segment(v, s, c)) >= 0;
#pragma unroll
            for (int m = 1; m < kSplit; m <<= 1) any |= __shfl_xor(any, m, 64);
            if (any) vis = 0.0f;
        }
        const float lam = ndl > 0.0f ? ndl : 0.0f;
        const float3 a = albedo_of(id);
        rgba = make_float4(a.x * (v.ambient[0] + v.light_rgb[0] * lam * vis),
                           a.y * (v.ambient[1] + v.light_rgb[1] * lam * vis),
                           a.z * (v.ambient[2] + v.light_rgb[2] * lam * vis), 1.0f);
    }
    if (c != 0) return;
    v.out_rgba[out] = rgba;
    if (v.out_id) v.out_id[out] = id;
    if (v.out_p) v.out_p[out] = p;
}

// kLambert: the view is Lambert-shaded (69 VGPRs, seven waves per SIMD; a
// budget of eight spilled 14 registers, 494 -> 511 us), else path-traced.
template <int B, int S, bool kLambert>
__global__ __launch_bounds__(B) kListWaves(kLambert) void k_trace_list(const TraceView v) {
    __shared__ int stack[lds_entries(S) * B];
    const int64_t count = *v.item_count;
    const int64_t q = (int64_t)blockIdx.x * B + threadIdx.x;
    if (kLambert && count <= kSplitItems && kSplitShare * count <= v.n_items) {
        if (q < kSplit * count) trace_item_split<B, S>(v, v.item_list[q / kSplit], (int)(q % kSplit), stack);
    } else if (q < count) {
        trace_item<B, S, false, false, kLambert, kLambert>(v, v.item_list[q], stack, nullptr);
    }
}

// Batched launch: workgroup b serves view vid with block_end[vid-1] <= b <
// block_end[vid] (block_end is the running sum of per-view workgroups of B
// items each).  S covers the deepest scene of the batch.
// order (nullable): per XCD, the dispatch order of its blocks (see
// k_trace_plan); cost (nullable): each block's duration in 100 MHz ticks,
// the larger of its waves', kept by slot for the next frame's plan.
template <int B, int S, bool kCount, bool kPhased, bool kLambert>
__global__ __launch_bounds__(B) kBatchWaves(kLambert, kPhased) void k_trace_batch(const TraceView* __restrict__ views,
                                                   const int32_t* __restrict__ block_end, int32_t n_views,
                                                   unsigned long long* counters, const int32_t* __restrict__ order,
                                                   uint32_t* __restrict__ cost) {
    __shared__ int stack[lds_entries(S) * B];
    // Four bytes that place the traversal loops: the same code four bytes lower
    // took 338 instead of 335 us (binocular frame, 4.52M terrain), 2.509
    // instead of 2.494 ms (16 views); offsets 4 and 36 are the faster ones, 0,
    // 20 and 52 the slower.
    if (B > 64) __asm__ volatile("s_nop 0");
    const uint64_t t0 = cost ? wall_clock64() : 0;
    // XCD x runs `slot`s x per .. x per + per - 1 of the plan; slot s holds
    // the work block xcd_work(x, s - x per)
    const int per = gridDim.x / kXcds;
    int b = blockIdx.x, slot = blockIdx.x;
    if (b < per * kXcds) {
        const int x = b % kXcds;
        int i = b / kXcds;
        if (order) i = order[x * per + i];
        slot = x * per + i;
        b = xcd_work<B>(x, i, per);
    }
    int vid = 0;
    while (vid + 1 < n_views && b >= block_end[vid]) ++vid;
    const int first = vid ? block_end[vid - 1] : 0;
    trace_item<B, S, kCount, kPhased, kLambert>(views[vid], (int64_t)(b - first) * B + threadIdx.x, stack, counters);
    if (cost && (threadIdx.x & 63) == 0) {
        const uint64_t dt = wall_clock64() - t0;
        atomicMax(cost + slot, (uint32_t)(dt < 0xffffffffull ? dt : 0xffffffffull));
    }
}

// Longest-first dispatch order of a batched traversal launch, from the
// previous frame's block durations.  Workgroup x plans XCD x, which runs the
// slots x per .. x per + per - 1 (per = blocks / 8; the few blocks past
// 8 per keep their place): the blocks are ranked into 32 classes of
// duration (two per octave from 2.56 us up, longest first) by a counting
// sort, and order[x per + p] is the p-th block of that ranking, so the
// traversal starts the expensive screen regions first and the cheap ones
// fill in behind them.  Each duration is read once and then cleared for the
// frame being planned; the order is a permutation whatever the durations.
constexpr int kPlanThreads = 1024;
constexpr int kPlanMaxPer = 32768;
constexpr int kPlanClasses = 32;

__global__ __launch_bounds__(kPlanThreads) void k_trace_plan(uint32_t* __restrict__ cost, int32_t* __restrict__ order,
                                                             int32_t blocks) {
    __shared__ uint8_t cls[kPlanMaxPer];
    __shared__ int hist[kPlanClasses], base[kPlanClasses];
    const int per = blocks / kXcds;
    const int x = blockIdx.x;
    const int t = threadIdx.x;
    if (t < kPlanClasses) hist[t] = 0;
    __syncthreads();
    for (int i = t; i < per; i += kPlanThreads) {
        const uint32_t c = cost[x * per + i];
        cost[x * per + i] = 0u;
        // level = 2 log2(c) in half octaves from 2^8 ticks; longer is earlier
        const uint32_t bits = __float_as_uint((float)c);
        int lvl = c ? (int)(bits >> 22) - ((127 + 8) << 1) : 0;
        lvl = lvl < 0 ? 0 : (lvl > kPlanClasses - 1 ? kPlanClasses - 1 : lvl);
        const int k = kPlanClasses - 1 - lvl;
        cls[i] = (uint8_t)k;
        atomicAdd(&hist[k], 1);
    }
    __syncthreads();
    if (t == 0) {
        int acc = 0;
        for (int k = 0; k < kPlanClasses; ++k) {
            base[k] = acc;
            acc += hist[k];
        }
    }
    __syncthreads();
    for (int i = t; i < per; i += kPlanThreads) {
        const int pos = atomicAdd(&base[cls[i]], 1);
        order[x * per + pos] = i;
    }
}

template <int S>
void launch_single(const TraceView& v, int64_t blocks, hipStream_t stream, unsigned long long* counters) {
    constexpr int B = kTraceBlockSingle;
    if (v.item_list) {
        if (v.shade_mode == VAFR_SHADE_PATH)
            hipLaunchKernelGGL((k_trace_list<B, S, false>), dim3((unsigned)blocks), dim3(B), 0, stream, v);
        else
            hipLaunchKernelGGL((k_trace_list<B, S, true>), dim3((unsigned)blocks), dim3(B), 0, stream, v);
    } else if (counters)
        hipLaunchKernelGGL((k_trace<B, S, true, false>), dim3((unsigned)blocks), dim3(B), 0, stream, v, counters);
    else if (v.shade_mode == VAFR_SHADE_PATH)
        hipLaunchKernelGGL((k_trace<B, S, false, false>), dim3((unsigned)blocks), dim3(B), 0, stream, v, counters);
    else
        hipLaunchKernelGGL((k_trace<B, S, false, true>), dim3((unsigned)blocks), dim3(B), 0, stream, v, counters);
}

template <int B, int S>
void launch_batch(const TraceView* views, const int32_t* block_end, int32_t n_views, int32_t blocks, bool phased,
                  bool lambert, hipStream_t stream, unsigned long long* counters, const int32_t* order,
                  uint32_t* cost) {
    if (counters)
        hipLaunchKernelGGL((k_trace_batch<B, S, true, false, false>), dim3((unsigned)blocks), dim3(B), 0, stream,
                           views, block_end, n_views, counters, order, cost);
    else if (phased || !lambert)
        hipLaunchKernelGGL((k_trace_batch<B, S, false, true, false>), dim3((unsigned)blocks), dim3(B), 0, stream,
                           views, block_end, n_views, counters, order, cost);
    else
        hipLaunchKernelGGL((k_trace_batch<B, S, false, false, true>), dim3((unsigned)blocks), dim3(B), 0, stream,
                           views, block_end, n_views, counters, order, cost);
}

template <int S>
void launch_batch_s(const TraceView* views, const int32_t* block_end, int32_t n_views, int32_t blocks, int block,
                    bool phased, bool lambert, hipStream_t stream, unsigned long long* counters, const int32_t* order,
                    uint32_t* cost) {
    if (block == 64)
        launch_batch<64, S>(views, block_end, n_views, blocks, phased, lambert, stream, counters, order, cost);
    else if (block == 128)
        launch_batch<128, S>(views, block_end, n_views, blocks, phased, lambert, stream, counters, order, cost);
    else launch_batch<256, S>(views, block_end, n_views, blocks, phased, lambert, stream, counters, order, cost);
}

template <int S, bool kPhased, bool kLambert>
const void* batch_kernel_s(int block) {
    if (block == 64) return reinterpret_cast<const void*>(&k_trace_batch<64, S, false, kPhased, kLambert>);
    if (block == 128) return reinterpret_cast<const void*>(&k_trace_batch<128, S, false, kPhased, kLambert>);
    if (block == 256) return reinterpret_cast<const void*>(&k_trace_batch<256, S, false, kPhased, kLambert>);
    return nullptr;
}

template <int S>
const void* batch_kernel_any(int block, bool phased, bool lambert) {
    if (phased || !lambert) return batch_kernel_s<S, true, false>(block);
    return batch_kernel_s<S, false, true>(block);
}

bool stack_ok(int stack) { return stack == kStackShort || stack == kStackLong; }

}  // namespace

int format_nodes(BvhNode* nodes_dev, int64_t n, hipStream_t stream) {
    if (n <= 0) return VAFR_OK;
    hipLaunchKernelGGL(k_node_format, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, nodes_dev, n);
    VAFR_HIP(hipGetLastError());
    return VAFR_OK;
}

int64_t trace_items_of(const TraceView& v) {
    if (v.mode == kModeFull) return (int64_t)((v.width + 7) / 8) * ((v.height + 7) / 8) * 64;
    if (v.mode == kModeLmfr) return (int64_t)((v.lm_w + 7) / 8) * ((v.lm_h + 7) / 8) * 64;
    return v.n_items;
}

bool trace_block_ok(int block) { return block == 64 || block == 128 || block == 256; }

int launch_trace(const TraceView& v, hipStream_t stream, unsigned long long* counters) {
    if (v.n_items <= 0) return VAFR_OK;
    if (!stack_ok(v.stack)) return fail(VAFR_E_ARG, "unknown traversal stack class %d", v.stack);
    const int64_t blocks = (v.n_items + kTraceBlockSingle - 1) / kTraceBlockSingle;
    if (v.item_list && counters) return fail(VAFR_E_UNSUPPORTED, "work counting does not take an item list");
    if (blocks > 0x7fffffff) return fail(VAFR_E_UNSUPPORTED, "too many rays in one launch");
    if (v.stack == kStackShort) launch_single<kStackShort>(v, blocks, stream, counters);
    else launch_single<kStackLong>(v, blocks, stream, counters);
    VAFR_HIP(hipGetLastError());
    return VAFR_OK;
}

const void* trace_batch_kernel(int block, int stack, bool phased, bool lambert) {
    if (stack == kStackShort) return batch_kernel_any<kStackShort>(block, phased, lambert);
    if (stack == kStackLong) return batch_kernel_any<kStackLong>(block, phased, lambert);
    return nullptr;
}

int launch_trace_batch(const TraceView* views_dev, const int32_t* block_end_dev, int32_t n_views, int32_t blocks,
                       int block, int stack, bool phased, bool lambert, hipStream_t stream,
                       unsigned long long* counters, const int32_t* order, uint32_t* cost) {
    if (blocks <= 0) return VAFR_OK;
    if (!trace_block_ok(block)) return fail(VAFR_E_ARG, "trace workgroup size must be 64, 128 or 256");
    if (!stack_ok(stack)) return fail(VAFR_E_ARG, "unknown traversal stack class %d", stack);
    if (order && !trace_plan_ok(blocks)) return fail(VAFR_E_ARG, "too many blocks for a planned launch");
    if (stack == kStackShort)
        launch_batch_s<kStackShort>(views_dev, block_end_dev, n_views, blocks, block, phased, lambert, stream,
                                    counters, order, cost);
    else
        launch_batch_s<kStackLong>(views_dev, block_end_dev, n_views, blocks, block, phased, lambert, stream,
                                   counters, order, cost);
    VAFR_HIP(hipGetLastError());
    return VAFR_OK;
}

bool trace_plan_ok(int32_t blocks) { return blocks / kXcds <= kPlanMaxPer; }

const void* trace_queue_batch_kernel(int stack) {
    if (stack == kStackShort) return reinterpret_cast<const void*>(&k_trace_queue_batch<kStackShort>);
    if (stack == kStackLong) return reinterpret_cast<const void*>(&k_trace_queue_batch<kStackLong>);
    return nullptr;
}

int launch_trace_queue_batch(const TraceView* views_dev, const int32_t* qblock_end_dev, int32_t n_views,
                             int32_t blocks, int stack, int bounce, hipStream_t stream) {
    if (blocks <= 0) return VAFR_OK;
    if (!stack_ok(stack)) return fail(VAFR_E_ARG, "unknown traversal stack class %d", stack);
    if (bounce < 1 || bounce > kMaxBounces) return fail(VAFR_E_ARG, "bounce %d out of range", bounce);
    if (stack == kStackShort)
        hipLaunchKernelGGL((k_trace_queue_batch<kStackShort>), dim3((unsigned)blocks), dim3(kQueueBlock), 0, stream,
                           views_dev, qblock_end_dev, n_views, (int32_t)bounce);
    else
        hipLaunchKernelGGL((k_trace_queue_batch<kStackLong>), dim3((unsigned)blocks), dim3(kQueueBlock), 0, stream,
                           views_dev, qblock_end_dev, n_views, (int32_t)bounce);
    VAFR_HIP(hipGetLastError());
    return VAFR_OK;
}

const void* trace_plan_kernel() { return reinterpret_cast<const void*>(&k_trace_plan); }

int launch_trace_plan(uint32_t* cost, int32_t* order, int32_t blocks, hipStream_t stream) {
    if (blocks <= 0) return VAFR_OK;
    if (!trace_plan_ok(blocks)) return fail(VAFR_E_ARG, "too many blocks for a planned launch");
    hipLaunchKernelGGL(k_trace_plan, dim3(kXcds), dim3(kPlanThreads), 0, stream, cost, order, blocks);
    VAFR_HIP(hipGetLastError());
    return VAFR_OK;
}

}  // namespace vafr
