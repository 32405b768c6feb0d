// Device building blocks of the emission-absorption march, shared by the
// plain render (ea.hip) and the batched form (batched.hip).
//
// Per sample k of a ray (all float32):
//   t_k = (k + 0.5) * dt,   p_k = fma(t_k, dir, org),
//   rho_k = trilinear(volume, p_k) (clamp to edge; lerp x, then y, then z),
//   sigma_k = c * rho_k,
//   I   += exp(-tau) * (1 - exp(-sigma_k)) * rho_k,   tau += sigma_k.
// The opacity 1 - exp(-sigma) is taken as -expm1(-sigma) and both sums are
// compensated (Kahan) within a brick visit, so the float32 integral stays
// within a few ulps of the exact value over hundreds of samples.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "rafi.h"

namespace rafi {
namespace ea {

struct Item {
    int32_t ray;
    int32_t k;
    float tau;
    float I;  // forward: partial integral; backward: B, the integral behind sample k
};
static_assert(sizeof(Item) == RAFI_EA_ITEM_BYTES, "item layout");

struct Geo {
    int32_t n;
    int32_t g0, g1, g2;
    int32_t b0, b1, b2;  // brick edge per axis
};

__device__ inline Geo make_geo(int32_t n, const int32_t grid[3])
{
    return Geo{n, grid[0], grid[1], grid[2], n / grid[0], n / grid[1], n / grid[2]};
}

// Owning brick of p, or -1 outside [0, n)^3. Bricks are half-open.
__device__ inline int32_t owner_of(const float p[3], const Geo &g)
{
    const float fn = (float)g.n;
#pragma unroll
    for (int a = 0; a < 3; ++a)
        if (!(p[a] >= 0.0f) || !(p[a] < fn)) return -1;
    const int32_t bx = (int32_t)floorf(p[0]) / g.b0;
    const int32_t by = (int32_t)floorf(p[1]) / g.b1;
    const int32_t bz = (int32_t)floorf(p[2]) / g.b2;
    return bx + g.g0 * (by + g.g1 * bz);
}

// Brick bounds of domain d: a point is in d iff lo <= p < hi on every axis
// (the bounds are integers, so this equals owner_of(p) == d).
struct Box {
    float lo0, hi0, lo1, hi1, lo2, hi2;
    // the six compares combined without short-circuit branches
    __device__ bool contains(const float p[3]) const
    {
        return (p[0] >= lo0) & (p[0] < hi0) & (p[1] >= lo1) & (p[1] < hi1) & (p[2] >= lo2) & (p[2] < hi2);
    }
};

__device__ inline Box box_of(int32_t d, const Geo &g)
{
    const int32_t bx = d % g.g0, by = (d / g.g0) % g.g1, bz = d / (g.g0 * g.g1);
    return Box{(float)(bx * g.b0), (float)((bx + 1) * g.b0), (float)(by * g.b1), (float)((by + 1) * g.b1),
               (float)(bz * g.b2), (float)((bz + 1) * g.b2)};
}

// Ray `local` of a view (row-major pixels): origin, direction, sample count.
__device__ inline void ray_setup(const rafi_ortho_view &V, int32_t local, float org[3], float dir[3],
                                 int32_t *n_samples)
{
    const int32_t py = local / V.width;
    const int32_t px = local - py * V.width;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        org[a] = __fmaf_rn((float)py, V.dv[a], __fmaf_rn((float)px, V.du[a], V.org0[a]));
        dir[a] = V.dir[a];
    }
    *n_samples = V.n_samples;
}

__device__ inline void sample_pos(const float org[3], const float dir[3], float dt, int32_t k, float p[3])
{
    const float t = ((float)k + 0.5f) * dt;
#pragma unroll
    for (int a = 0; a < 3; ++a) p[a] = __fmaf_rn(t, dir[a], org[a]);
}

__device__ inline float lerpf(float a, float b, float t) { return __fmaf_rn(t, b - a, a); }

// Trilinear setup at p: corner (i0, j0, k0), its linear index and the
// fractional weights.
struct Tri {
    int64_t base;
    int32_t x, y, z;
    float f0, f1, f2;
};

__device__ inline Tri tri_setup(int32_t n, const float p[3])
{
    int32_t i0[3];
    float f[3];
    const float hi = (float)(n - 1);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float u = fminf(fmaxf(p[a] - 0.5f, 0.0f), hi);
        const int32_t i = min((int32_t)floorf(u), n - 2);
        i0[a] = i;
        f[a] = u - (float)i;
    }
    return Tri{i0[0] + (int64_t)n * (i0[1] + (int64_t)n * i0[2]), i0[0], i0[1], i0[2], f[0], f[1], f[2]};
}

// tri_setup for volumes of at most 1290^3 voxels (n^3 < 2^31, the caller's
// test): the same cell and weights, the clamp as one med3 (the clamp for any
// non-NaN value), the floor limited to n - 2 in float (exact: an integer
// below 2^24) and the corner's linear index from full-rate 24-bit
// multiplies (every factor below 2^24, the sum below 2^31).
constexpr int32_t kSmallN = 1290;

__device__ inline Tri tri_setup_small(int32_t n, const float p[3])
{
    const float hi = (float)(n - 1), top = (float)(n - 2);
    uint32_t i0[3];
    float f[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float u = __builtin_amdgcn_fmed3f(p[a] - 0.5f, 0.0f, hi);
        const float fl = __builtin_amdgcn_fmed3f(floorf(u), 0.0f, top);
        i0[a] = (uint32_t)fl;
        f[a] = u - fl;
    }
    const uint32_t nn = (uint32_t)n;
    const uint32_t base = i0[0] + __umul24(i0[1], nn) + __umul24(i0[2], nn * nn);
    return Tri{(int64_t)base, (int32_t)i0[0], (int32_t)i0[1], (int32_t)i0[2], f[0], f[1], f[2]};
}

// 1 - exp(-s). For |s| below 1/16, the Maclaurin series of the function to
// the s^6 term (Horner form; the truncated terms are below 1.2e-11 |s|):
// five fused multiply-adds and a product instead of the library's expm1.
// Larger |s|, or a NaN, take the library call.
__device__ inline float one_minus_exp_neg(float s)
{
    float q = __fmaf_rn(s, -1.0f / 720.0f, 1.0f / 120.0f);
    q = __fmaf_rn(s, q, -1.0f / 24.0f);
    q = __fmaf_rn(s, q, 1.0f / 6.0f);
    q = __fmaf_rn(s, q, -0.5f);
    q = __fmaf_rn(s, q, 1.0f);
    q = s * q;
    if (!(fabsf(s) < 0.0625f)) q = -expm1f(-s);
    return q;
}

// Trilinear density from the volume (voxel centres at i + 0.5).
__device__ inline float density(const float *__restrict__ vol, int32_t n, const Tri &t)
{
    const int64_t sx = 1, sy = n, sz = (int64_t)n * n;
    const float *b = vol + t.base;
    const float x00 = lerpf(b[0], b[sx], t.f0);
    const float x10 = lerpf(b[sy], b[sy + sx], t.f0);
    const float x01 = lerpf(b[sz], b[sz + sx], t.f0);
    const float x11 = lerpf(b[sz + sy], b[sz + sy + sx], t.f0);
    const float y0 = lerpf(x00, x10, t.f1);
    const float y1 = lerpf(x01, x11, t.f1);
    return lerpf(y0, y1, t.f2);
}

// The 8 voxels of the last sampled cell, kept in registers. Samples half a
// voxel apart along a ray often fall in the same cell, and then no memory is
// read: on the 64-view render the texture-address unit's work drops by about
// a third. The values and the interpolation are those of density(), so the
// result is bit-identical.
struct Corners {
    int64_t base = -1;  // linear index of the cached cell's corner; -1 = empty
    float v[8];
};

// density_cached in two halves: the loads of a new cell's corners (issued,
// not waited for), and the interpolation that uses them.
__device__ inline void fetch_corners(const float *__restrict__ vol, int32_t n, const Tri &t, Corners &cc)
{
    if (t.base != cc.base) {
        const int64_t sy = n, sz = (int64_t)n * n;
        const float *b = vol + t.base;
        cc.v[0] = b[0];
        cc.v[1] = b[1];
        cc.v[2] = b[sy];
        cc.v[3] = b[sy + 1];
        cc.v[4] = b[sz];
        cc.v[5] = b[sz + 1];
        cc.v[6] = b[sz + sy];
        cc.v[7] = b[sz + sy + 1];
        cc.base = t.base;
    }
}

__device__ inline float interp_corners(const Corners &cc, const Tri &t)
{
    const float x00 = lerpf(cc.v[0], cc.v[1], t.f0);
    const float x10 = lerpf(cc.v[2], cc.v[3], t.f0);
    const float x01 = lerpf(cc.v[4], cc.v[5], t.f0);
    const float x11 = lerpf(cc.v[6], cc.v[7], t.f0);
    const float y0 = lerpf(x00, x10, t.f1);
    const float y1 = lerpf(x01, x11, t.f1);
    return lerpf(y0, y1, t.f2);
}

__device__ inline float density_cached(const float *__restrict__ vol, int32_t n, const Tri &t, Corners &cc)
{
    fetch_corners(vol, n, t, cc);
    return interp_corners(cc, t);
}

// First k in [0, K] for which pred(k) flips from `from` to !from (K if never):
// the estimate or a neighbour of it, or else a binary search of what is left.
template <typename Pred>
__device__ inline int32_t first_flip(int32_t K, bool from, float estimate, Pred pred)
{
    int32_t lo = 0, hi = K;
    const int32_t k = min((int32_t)fminf(fmaxf(estimate, 0.0f), 2147483520.0f), K);
    if (k < K && pred(k) == from) {
        lo = k + 1;
        if (lo < K && pred(lo) != from) hi = lo;
    } else {
        hi = k;
        if (k > 0 && pred(k - 1) == from) lo = k;
    }
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (pred(mid) != from) hi = mid; else lo = mid + 1;
    }
    return lo;
}

// Ray generation: the first sample index inside [0, n)^3, or -1 if none.
// Every coordinate of p_k is monotone in k (the product and the fma are
// correctly rounded, hence monotone), so the inside samples form one interval
// of k: per face, the straight line's crossing estimates its end and the exact
// test settles it. *owner is the brick of the first sample.
__device__ inline int32_t first_inside(const Geo &g, const float org[3], const float dir[3], int32_t K, float dt,
                                       int32_t *owner)
{
    const float fn = (float)g.n, rdt = __builtin_amdgcn_rcpf(dt);
    int32_t k_lo = 0, k_hi = K;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        auto coord = [&](int32_t k) {
            const float t = ((float)k + 0.5f) * dt;
            return __fmaf_rn(t, dir[a], org[a]);
        };
        auto ge0 = [&](int32_t k) { return coord(k) >= 0.0f; };
        auto ltn = [&](int32_t k) { return coord(k) < fn; };
        const float r = __builtin_amdgcn_rcpf(dir[a]) * rdt;
        const float k0 = ceilf(-org[a] * r - 0.5f), kn = ceilf((fn - org[a]) * r - 0.5f);
        const bool moves = dir[a] > 0.0f || dir[a] < 0.0f;
        if (moves && (dir[a] > 0.0f) == (dt > 0.0f)) {  // the coordinate rises with k
            k_lo = max(k_lo, first_flip(K, false, k0, ge0));   // becomes true
            k_hi = min(k_hi, first_flip(K, true, kn, ltn));    // becomes false
        } else if (moves) {
            k_lo = max(k_lo, first_flip(K, false, kn, ltn));
            k_hi = min(k_hi, first_flip(K, true, k0, ge0));
        } else if (!(org[a] >= 0.0f && org[a] < fn)) {
            k_hi = 0;
        }
    }
    if (k_lo >= k_hi) return -1;
    float p[3];
    sample_pos(org, dir, dt, k_lo, p);
    *owner = owner_of(p, g);
    return k_lo;
}

// First sample index past the box along a straight line, to rounding.
__device__ inline float exit_estimate(const Box &box, const float org[3], const float dir[3], float dt)
{
    const float lo[3] = {box.lo0, box.lo1, box.lo2}, hi[3] = {box.hi0, box.hi1, box.hi2};
    float texit = 3.0e38f;
#pragma unroll
    for (int a = 0; a < 3; ++a)
        if (dir[a] != 0.0f)
            texit = fminf(texit, ((dir[a] > 0.0f ? hi[a] : lo[a]) - org[a]) * __builtin_amdgcn_rcpf(dir[a]));
    return ceilf(texit * __builtin_amdgcn_rcpf(dt) - 0.5f);
}

// First sample index >= k outside the box, or K. Every coordinate of p_k is
// monotone in k, so from a sample k inside the box the inside samples are
// [k, end): a straight-line estimate of `end`, corrected with the exact test
// (usually by nothing), gives the index a per-sample test would stop at.
// Per visit this costs about what three per-sample tests did (the 64-view
// render of 128^3: 2.46 -> 2.32 ms).
__device__ inline int32_t exit_sample(const Box &box, const float org[3], const float dir[3], float dt, int32_t k,
                                      int32_t K)
{
    auto inside = [&](int32_t j) {
        float p[3];
        sample_pos(org, dir, dt, j, p);
        return box.contains(p);
    };
    if (k >= K || !inside(k)) return k;
    const float est = exit_estimate(box, org, dir, dt);
    int32_t end = min(max((int32_t)fminf(fmaxf(est, 0.0f), 2147483520.0f), k + 1), K);
    while (end < K && inside(end)) ++end;
    while (end > k + 1 && !inside(end - 1)) --end;
    return end;
}

// First sample index of the run of inside samples that ends at k: the walk of
// the adjoint stops below it (k + 1 when k itself is outside). As exit_sample,
// in the other direction.
__device__ inline float entry_estimate(const Box &box, const float org[3], const float dir[3], float dt)
{
    const float lo[3] = {box.lo0, box.lo1, box.lo2}, hi[3] = {box.hi0, box.hi1, box.hi2};
    float tin = -3.0e38f;
#pragma unroll
    for (int a = 0; a < 3; ++a)
        if (dir[a] != 0.0f)
            tin = fmaxf(tin, ((dir[a] > 0.0f ? lo[a] : hi[a]) - org[a]) * __builtin_amdgcn_rcpf(dir[a]));
    return ceilf(tin * __builtin_amdgcn_rcpf(dt) - 0.5f);
}

__device__ inline int32_t entry_sample(const Box &box, const float org[3], const float dir[3], float dt, int32_t k)
{
    auto inside = [&](int32_t j) {
        float p[3];
        sample_pos(org, dir, dt, j, p);
        return box.contains(p);
    };
    if (k < 0 || !inside(k)) return k + 1;
    const float est = entry_estimate(box, org, dir, dt);
    int32_t first = min((int32_t)fminf(fmaxf(est, 0.0f), 2147483520.0f), k);
    while (first > 0 && inside(first - 1)) --first;
    while (first < k && !inside(first)) ++first;
    return first;
}

// The running integral and optical depth of a visit, both sums compensated
// (Kahan). The transmittance exp(-tau) is the hardware exponential (a base-2
// exponential of -tau log2(e)); its relative error, about 1e-6 for the
// optical depths of a ray, stays well inside the integrals' tolerance; the
// emission weight 1 - exp(-sigma) keeps full relative accuracy for small
// sigma (one_minus_exp_neg). kLib: the library's expf and expm1 instead, both
// within an ulp or two at every optical depth (contexts with large tiles,
// rafi_set_tile_items).
template <bool kLib>
struct Sums {
    float tau, I, ctau = 0.0f, cI = 0.0f;
    __device__ Sums(const Item &it) : tau(it.tau), I(it.I) {}
    __device__ void add(float rho, float c)
    {
        const float sigma = c * rho;
        const float w = kLib ? expf(-tau) * -expm1f(-sigma) : __expf(-tau) * one_minus_exp_neg(sigma);
        // compensated I += w * rho
        const float yI = w * rho - cI;
        const float tI = I + yI;
        cI = (tI - I) - yI;
        I = tI;
        // compensated tau += sigma
        const float yt = sigma - ctau;
        const float tt = tau + yt;
        ctau = (tt - tau) - yt;
        tau = tt;
    }
    __device__ void store(Item &it) const
    {
        it.tau = tau - ctau;
        it.I = I - cI;
    }
};

// Sample counts up to which k + 0.5 and its increments are exact in float.
constexpr int32_t kFloatK = 1 << 22;

// Where a march reads densities from: the volume in global memory ...
struct GlobalVol {
    const float *__restrict__ vol;
    int32_t n;
    __device__ const float *at(float x, float y, float z) const
    {
        return vol + ((uint32_t)x + __umul24((uint32_t)y, (uint32_t)n) + __umul24((uint32_t)z, (uint32_t)(n * n)));
    }
    __device__ uint32_t row() const { return (uint32_t)n; }
    __device__ uint32_t plane() const { return (uint32_t)(n * n); }
    __device__ int32_t z_first() const { return 0; }
    __device__ int32_t z_last() const { return n - 1; }
};

// ... or a brick's voxels plus a one-voxel rim, staged in LDS: region origin
// o = lo - 1 per axis, extent e = b + 2. Samples inside the brick only touch
// voxels [max(lo-1, 0), min(hi, n-1)], all inside the region.
struct Region {
    int32_t ox, oy, oz, ex, ey, ez;
};

__device__ inline Region region_of(const Box &box, const Geo &g)
{
    return Region{(int32_t)box.lo0 - 1, (int32_t)box.lo1 - 1, (int32_t)box.lo2 - 1, g.b0 + 2, g.b1 + 2, g.b2 + 2};
}

struct LdsVol {
    const float *origin;  // the LDS address voxel (0, 0, 0) would have
    Region r;
    __device__ LdsVol(const float *lds, const Region &reg)
        : origin(lds - (reg.ox + reg.ex * (reg.oy + reg.ey * reg.oz))), r(reg)
    {
    }
    // x, y, z: whole numbers. The index is computed in float, at full rate and
    // exactly: at most 8192 bricks of at most 160 KiB make n < 690, and with
    // three planes or more in a region the index stays below 2^24.
    __device__ const float *at(float x, float y, float z) const
    {
        return origin + (int32_t)__fmaf_rn(__fmaf_rn(z, (float)r.ey, y), (float)r.ex, x);
    }
    __device__ uint32_t row() const { return (uint32_t)r.ex; }
    __device__ uint32_t plane() const { return (uint32_t)(r.ex * r.ey); }
    __device__ int32_t z_first() const { return r.oz; }
    __device__ int32_t z_last() const { return r.oz + r.ez - 1; }
};

// Samples [k, end) of a ray along z (dir[0] = dir[1] = 0): its x and y cell
// and weights are fixed, so a voxel plane enters the interpolation as one
// bilinear value, kept while the ray moves to the next plane, and the plane
// after that is loaded one cell ahead. Per sample one lerp remains of seven,
// per cell two 8-byte loads of four, with the operations and rounding of
// interp_corners. Bound by VALU issue, 45 instructions a sample for 80: 256
// scenes of axis views (7.4 G samples) 18.5 -> 10.8 ms with a floor and two
// clamps a sample to find the cell, 10.4 ms without.
template <typename Vol, typename Sums>
__device__ __forceinline__ void march_z(const Vol &vol, int32_t n, const float org[3], float dirz, bool up, float dt,
                                        float c, int32_t k, int32_t end, Sums &s)
{
    const float at[3] = {org[0], org[1], 0.0f};
    const Tri t = tri_setup_small(n, at);
    const uint32_t row = vol.row(), plane = vol.plane();
    struct Raw {
        float a, b, c, d;
    };
    const float tx = (float)t.x, ty = (float)t.y;
    auto load = [&](const float *b) {
        const float *b1 = b + row;
        return Raw{b[0], b[1], b1[0], b1[1]};
    };
    auto blend = [&](const Raw &r) { return lerpf(lerpf(r.a, r.b, t.f0), lerpf(r.c, r.d, t.f0), t.f1); };
    // u lies in the cell [z, z + 1) when the bits of u - z, which is exact
    // there, are below those of 1: a negative difference has the sign bit.
    auto inside = [](float f) { return __float_as_uint(f) < 0x3f800000u; };
    const float hi = (float)(n - 1), top = (float)(n - 2);
    const float z_first = (float)vol.z_first(), z_last = (float)vol.z_last();
    float zc = 2.0f * hi, y0 = 0.0f, y1 = 0.0f, dy = 0.0f;  // the cell, the values of its planes, y1 - y0
    Raw ahead{};                                            // the plane after them in the ray's direction,
    const float *p = vol.at(tx, ty, z_first);               // and its place
    const float kend = (float)end + 0.5f;
    for (float kf = (float)k + 0.5f; kf < kend; kf += 1.0f) {
        const float u = __builtin_amdgcn_fmed3f(__fmaf_rn(kf * dt, dirz, org[2]) - 0.5f, 0.0f, hi);
        float f = u - zc;
        if (!inside(f)) {
            zc += up ? 1.0f : -1.0f;
            f = u - zc;
            if (inside(f) && zc < hi) {
                if (up) {
                    y0 = y1;
                    y1 = blend(ahead);
                } else {
                    y1 = y0;
                    y0 = blend(ahead);
                }
            } else {  // the first sample, a step of several cells, or u = hi, which cell n - 2 holds
                zc = __builtin_amdgcn_fmed3f(floorf(u), 0.0f, top);
                f = u - zc;
                p = vol.at(tx, ty, zc);
                const Raw r0 = load(p), r1 = load(p + plane);
                y0 = blend(r0);
                y1 = blend(r1);
                if (up) p += plane;
            }
            dy = y1 - y0;
            if (up ? zc + 2.0f <= z_last : zc - 1.0f >= z_first) {
                p = up ? p + plane : p - plane;
                ahead = load(p);
            }
        }
        s.add(__fmaf_rn(f, dy, y0), c);
    }
}

// Advance a ray through its brick (box) from sample it.k: accumulates tau and
// I and leaves it.k at the first sample not taken. Returns the brick that owns
// that sample, or -1 when the ray left the volume or ran out of samples.
// kSmall: the volume has at most kSmallN^3 voxels (tri_setup_small) and the
// ray at most kFloatK samples. kLib: see Sums.
template <bool kSmall, bool kLib>
__device__ inline int32_t march_through_n(const float *__restrict__ vol, const Geo &g, const Box &box,
                                          const float org[3], const float dir[3], int32_t K, float dt, float c,
                                          Item &it)
{
    const int32_t end = exit_sample(box, org, dir, dt, it.k, K);
    Sums<kLib> s(it);
    if (kSmall && dir[0] == 0.0f && dir[1] == 0.0f) {
        if (dir[2] * dt > 0.0f)
            march_z(GlobalVol{vol, g.n}, g.n, org, dir[2], true, dt, c, it.k, end, s);
        else
            march_z(GlobalVol{vol, g.n}, g.n, org, dir[2], false, dt, c, it.k, end, s);
    } else if (kSmall) {
        Corners cc;
        const float kend = (float)end + 0.5f;
        for (float kf = (float)it.k + 0.5f; kf < kend; kf += 1.0f) {
            const float t = kf * dt;
            const float p[3] = {__fmaf_rn(t, dir[0], org[0]), __fmaf_rn(t, dir[1], org[1]),
                                __fmaf_rn(t, dir[2], org[2])};
            s.add(density_cached(vol, g.n, tri_setup_small(g.n, p), cc), c);
        }
    } else {
        Corners cc;
        for (int32_t k = it.k; k < end; ++k) {
            float p[3];
            sample_pos(org, dir, dt, k, p);
            s.add(density_cached(vol, g.n, tri_setup(g.n, p), cc), c);
        }
    }
    s.store(it);
    it.k = max(it.k, end);
    if (end >= K) return -1;
    float p[3];
    sample_pos(org, dir, dt, end, p);
    return owner_of(p, g);
}

template <bool kLib = false>
__device__ inline int32_t march_through(const float *__restrict__ vol, const Geo &g, const Box &box,
                                        const float org[3], const float dir[3], int32_t K, float dt, float c,
                                        Item &it)
{
    return g.n <= kSmallN && K <= kFloatK ? march_through_n<true, kLib>(vol, g, box, org, dir, K, dt, c, it)
                                          : march_through_n<false, kLib>(vol, g, box, org, dir, K, dt, c, it);
}

// march_through with the brick's densities read from a staged region, for
// volumes of at most kSmallN^3 voxels and rays of at most kFloatK samples: the
// same values and operations. No cell is kept in registers here: eight LDS
// reads cost less than testing for a new cell and branching.
template <bool kLib>
__device__ inline int32_t march_through_lds(const LdsVol &vol, const Geo &g, const Box &box, const float org[3],
                                            const float dir[3], int32_t K, float dt, float c, Item &it)
{
    const int32_t end = exit_sample(box, org, dir, dt, it.k, K);
    Sums<kLib> s(it);
    if (dir[0] == 0.0f && dir[1] == 0.0f) {
        // one loop for both directions: wavefronts here hold rays of all views
        march_z(vol, g.n, org, dir[2], dir[2] * dt > 0.0f, dt, c, it.k, end, s);
    } else {
        const uint32_t row = vol.row(), plane = vol.plane();
        const float hi = (float)(g.n - 1), top = (float)(g.n - 2);
        const float kend = (float)end + 0.5f;
#pragma unroll 2
        for (float kf = (float)it.k + 0.5f; kf < kend; kf += 1.0f) {
            const float t = kf * dt;
            const float p[3] = {__fmaf_rn(t, dir[0], org[0]), __fmaf_rn(t, dir[1], org[1]),
                                __fmaf_rn(t, dir[2], org[2])};
            float fl[3], f[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float u = __builtin_amdgcn_fmed3f(p[a] - 0.5f, 0.0f, hi);
                fl[a] = __builtin_amdgcn_fmed3f(floorf(u), 0.0f, top);
                f[a] = u - fl[a];
            }
            const float *b0 = vol.at(fl[0], fl[1], fl[2]), *b1 = b0 + row, *b2 = b0 + plane, *b3 = b1 + plane;
            Corners cc;
            cc.v[0] = b0[0];
            cc.v[1] = b0[1];
            cc.v[2] = b1[0];
            cc.v[3] = b1[1];
            cc.v[4] = b2[0];
            cc.v[5] = b2[1];
            cc.v[6] = b3[0];
            cc.v[7] = b3[1];
            s.add(interp_corners(cc, Tri{0, 0, 0, 0, f[0], f[1], f[2]}), c);
        }
    }
    s.store(it);
    it.k = max(it.k, end);
    if (end >= K) return -1;
    float p[3];
    sample_pos(org, dir, dt, end, p);
    return owner_of(p, g);
}

// Position k of a region, as thread t of NT threads steps through it by NT:
// carries instead of divisions.
template <uint32_t NT>
struct RegionWalk {
    int32_t k, x, y, z, dx, dy, dz;
    __device__ RegionWalk(const Region &r)
    {
        const int32_t sxy = r.ex * r.ey;
        dz = (int32_t)NT / sxy;
        dy = ((int32_t)NT - dz * sxy) / r.ex;
        dx = (int32_t)NT - dz * sxy - dy * r.ex;
        k = (int32_t)threadIdx.x;
        z = k / sxy;
        y = (k - z * sxy) / r.ex;
        x = k - z * sxy - y * r.ex;
    }
    __device__ void step(const Region &r)
    {
        k += NT;
        x += dx;
        if (x >= r.ex) { x -= r.ex; ++y; }
        y += dy;
        if (y >= r.ey) { y -= r.ey; ++z; }
        z += dz;
    }
};

// The staged region of `vol`, loaded by the whole workgroup of NT threads
// (positions outside the volume take its nearest voxel and are never used),
// eight loads in flight per thread.
template <uint32_t NT>
__device__ inline void load_region(float *lds, const float *__restrict__ vol, int32_t n, const Region &r)
{
    constexpr int kU = 8;
    const int32_t total = r.ex * r.ey * r.ez;
    for (RegionWalk<NT> at(r); at.k < total;) {
        float v[kU];
        const int32_t k0 = at.k;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int32_t gx = min(max(r.ox + at.x, 0), n - 1), gy = min(max(r.oy + at.y, 0), n - 1),
                          gz = min(max(r.oz + at.z, 0), n - 1);
            v[u] = vol[gx + (int64_t)n * (gy + (int64_t)n * gz)];
            at.step(r);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u)
            if (k0 + u * (int32_t)NT < total) lds[k0 + u * (int32_t)NT] = v[u];
    }
}

__device__ inline int32_t find_domain(const uint64_t *__restrict__ off, int32_t D, uint64_t i)
{
    int32_t lo = 0, hi = D;  // last d with off[d] <= i
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (off[mid] <= i) lo = mid; else hi = mid;
    }
    return lo;
}

}  // namespace ea
}  // namespace rafi
