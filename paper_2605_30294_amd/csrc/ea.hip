// Emission-absorption ray march over bricked domains: ray generation (round
// 0), the brick kernel that advances rays through their current brick and
// forwards them at its boundary (the VoPaT / Lander pattern, Sec. 5.1-5.2:
// each forwarded ray carries its partial integration state), and the adjoint
// that replays every ray backwards through the same bricks. The per-sample
// arithmetic is in ea_device.h.
#include <algorithm>

#include "ea_device.h"
#include "internal.h"
#include "rafi_device.h"
#include "split_device.h"

namespace rafi {
namespace {

using ea::Box;
using ea::Geo;
using ea::Item;
using ea::Tri;

__device__ inline Geo job_geo(const rafi_ea_job &j) { return ea::make_geo(j.n, j.grid); }

__device__ inline void job_ray(const rafi_ea_job &j, int32_t ray, float org[3], float dir[3], int32_t *K)
{
    const int32_t per = j.width * j.height;
    const int32_t v = ray / per;
    ea::ray_setup(j.views[v], ray - v * per, org, dir, K);
}

__device__ inline void log_visit(const rafi_ea_job &j, int32_t ray, int32_t d)
{
    if (!j.visit_log) return;
    const int32_t c = j.visit_count[ray];
    if (c < j.visit_stride) j.visit_log[(int64_t)ray * j.visit_stride + c] = d;
    j.visit_count[ray] = c + 1;
}

// ------------------------------------------------------------- raygen ---
__global__ void __launch_bounds__(256)
raygen_kernel(rafi_device_view view, rafi_ea_job job, uint64_t n_rays)
{
    const uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    if (r >= n_rays) return;
    const Geo g = job_geo(job);
    float org[3], dir[3];
    int32_t K, owner = -1;
    job_ray(job, (int32_t)r, org, dir, &K);
    const int32_t k0 = ea::first_inside(g, org, dir, K, job.dt, &owner);
    if (job.visit_count) job.visit_count[r] = 0;
    if (k0 >= 0) {
        if (job.kfirst) job.kfirst[r] = k0;
        rafi_forward_t(view, r, Item{(int32_t)r, k0, 0.0f, 0.0f}, owner);
    } else {
        if (job.kfirst) job.kfirst[r] = 0;
        job.image[r] = 0.0f;
        if (job.tau) job.tau[r] = 0.0f;
        if (job.klast) job.klast[r] = 0;
        rafi_done(view, r);
    }
}

// Emission of a marched ray from input slot i: to its own output slot, or
// appended (rafi_open append mode, where every slot starts as RAFI_DONE).
__device__ inline void emit_item(const rafi_device_view &view, const rafi_ea_job &job, uint64_t i, const Item &it,
                                 int32_t dest)
{
    if (job.emit_mode == RAFI_SLOTS_APPEND) rafi_emit_t(view, it, dest);
    else rafi_forward_t(view, i, it, dest);
}

// A ray leaving brick d: forwarded to `dest`, or finished (dest < 0) with its
// integral, optical depth and end sample written out.
__device__ inline void emit_ray(const rafi_device_view &view, const rafi_ea_job &job, uint64_t i, const Item &it,
                                int32_t dest)
{
    if (dest >= 0) {
        emit_item(view, job, i, it, dest);
        return;
    }
    job.image[it.ray] = it.I;
    if (job.tau) job.tau[it.ray] = it.tau;
    if (job.klast) job.klast[it.ray] = it.k;
    if (job.emit_mode != RAFI_SLOTS_APPEND) rafi_done(view, i);
}

// ------------------------------------------------------------- march ----
// One lane per ray. A wave marches until the longest chord among its 64 rays
// ends, so each workgroup first orders its rays by the samples each has left
// in its brick (a counting sort through LDS), where chords can differ and
// unless they all fall in one bucket. Every ray is marched as if alone and
// written to its own output slot, so results do not depend on the lane.
template <bool kLib>
__global__ void __launch_bounds__(256)
march_kernel(rafi_device_view view, rafi_ea_job job, uint32_t n_rays)
{
    constexpr uint32_t kThreads = 256, kWaves = kThreads / 64, kBuckets = 16;
    __shared__ Item s_item[kThreads];
    __shared__ uint32_t s_slot[kThreads];
    __shared__ int32_t s_d[kThreads];
    __shared__ uint32_t s_cnt[kWaves][kBuckets];
    // the grid may be sized for an upper bound: number the live workgroups only
    const uint64_t n_in = rafi_queue_length(view);
    const uint32_t nb = (uint32_t)((n_in + kThreads - 1) / kThreads);
    if (blockIdx.x >= nb) return;
    const uint32_t t = threadIdx.x, w = t >> 6, lane = t & 63;
    const uint64_t base = rafi_xcd_block(blockIdx.x, nb) * (uint64_t)kThreads;
    const Geo g = job_geo(job);
    uint64_t slot = base + t;
    int32_t d = 0;
    Item it{};
    uint32_t key = kBuckets - 1;
    // Order the lanes only where chords can differ much: bricks whose chord
    // can exceed 64 samples, and rays not along an axis (the same decision in
    // every thread, taken from the workgroup's first ray; any choice gives the
    // same results).
    bool order = (float)(g.b0 + g.b1 + g.b2) >= 64.0f * job.dt;
    if (order) {
        const int32_t r0 = static_cast<const Item *>(view.in_items)[base].ray;
        if ((uint32_t)r0 < n_rays) {
            const float *dir0 = job.views[r0 / (job.width * job.height)].dir;
            order = (dir0[0] != 0.0f) + (dir0[1] != 0.0f) + (dir0[2] != 0.0f) > 1;
        }
    }
    if (!order) {
        if (slot >= n_in) return;
        d = ea::find_domain(view.in_offsets, view.n_domains, slot);
        it = static_cast<const Item *>(view.in_items)[slot];
        if ((uint32_t)it.ray >= n_rays) {  // never true for items this library emitted
            emit_item(view, job, slot, it, RAFI_POISON);
            return;
        }
        log_visit(job, it.ray, d);
        float org[3], dir[3];
        int32_t K;
        job_ray(job, it.ray, org, dir, &K);
        const int32_t dest =
            ea::march_through<kLib>(job.volume, g, ea::box_of(d, g), org, dir, K, job.dt, job.c, it);
        emit_ray(view, job, slot, it, dest);
        return;
    }
    if (slot < n_in) {
        d = ea::find_domain(view.in_offsets, view.n_domains, slot);
        it = static_cast<const Item *>(view.in_items)[slot];
        if ((uint32_t)it.ray >= n_rays) {  // never true for items this library emitted
            emit_item(view, job, slot, it, RAFI_POISON);
        } else {
            // samples left in the brick along a straight line (an estimate: it
            // only orders the lanes)
            float org[3], dir[3];
            int32_t K;
            job_ray(job, it.ray, org, dir, &K);
            const Box box = ea::box_of(d, g);
            const float span = (float)(g.b0 + g.b1 + g.b2) * __builtin_amdgcn_rcpf(job.dt);
            const float left = fminf(ea::exit_estimate(box, org, dir, job.dt), (float)K) - (float)it.k;
            key = (uint32_t)fminf(fmaxf(left * ((float)(kBuckets - 1) / span), 0.0f), (float)(kBuckets - 2));
        }
    }
    // Stable counting sort of the workgroup's lanes by key, through LDS: lanes
    // with a similar number of samples left share a wave.
    uint32_t rank = 0;
#pragma unroll
    for (uint32_t k = 0; k < kBuckets; ++k) {
        const uint64_t m = __ballot(key == k);
        if (lane == 0) s_cnt[w][k] = (uint32_t)__popcll(m);
        if (key == k) rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
    }
    __syncthreads();
    uint32_t pos = rank, n_live = 0, n_full = 0;
    for (uint32_t k = 0; k < kBuckets; ++k) {
        uint32_t tot = 0;
#pragma unroll
        for (uint32_t ww = 0; ww < kWaves; ++ww) {
            const uint32_t c = s_cnt[ww][k];
            pos += (k < key || (k == key && ww < w)) ? c : 0;
            tot += c;
        }
        n_live += k < kBuckets - 1 ? tot : 0;
        n_full += (k < kBuckets - 1 && tot > 0) ? 1 : 0;
    }
    // One bucket (or none) holds every live ray: the order stays (the same
    // decision in every thread, so the barrier below is met by all or none).
    if (n_full > 1) {
        s_item[pos] = it;
        s_slot[pos] = (uint32_t)(slot - base);
        s_d[pos] = d;
        __syncthreads();
        if (t >= n_live) return;  // no barrier follows
        it = s_item[t];
        slot = base + s_slot[t];
        d = s_d[t];
    } else if (key == kBuckets - 1) {
        return;
    }
    log_visit(job, it.ray, d);
    float org[3], dir[3];
    int32_t K;
    job_ray(job, it.ray, org, dir, &K);
    const int32_t dest =
        ea::march_through<kLib>(job.volume, g, ea::box_of(d, g), org, dir, K, job.dt, job.c, it);
    emit_ray(view, job, slot, it, dest);
}

// LDS-staged march: one workgroup per CU, each taking an equal contiguous
// slice of the queue and working through the brick segments it spans (usually
// one or two): it stages the brick's densities plus a one-voxel rim in LDS and
// marches the segment's rays against them. Gathers from global memory cost
// by the lane (about 26 address cycles per wave-wide gather, the address unit
// 74% busy), LDS reads a few cycles each. Rays go through in batches ordered
// by the samples they have left in the brick, longest first, and each wave
// takes the next 64 when it is done, so lanes and waves stay busy (94% of the
// issued lanes live, 66% with gathers). Every ray is marched as if alone and
// written to its own output slot, so results do not depend on the lane. Bound
// by VALU issue (62% of the slots, 83 instructions a live sample) and the brick
// loads (first launch of the 64-view render of 128^3: 243 us for 2.1 M rays,
// 90.1 M samples).
constexpr uint32_t kBrickThreads = 1024, kBrickBatch = 2 * kBrickThreads, kBrickKeys = 64;

struct BrickOrder {
    uint32_t cnt[kBrickKeys], next;
};

// Batch order of the brick kernels: s_idx[0, m) = the batch's items by
// descending `left(q)` (samples item q has left), 1 / per_key samples to a
// bucket; o.next = 0. Called by the whole workgroup; m <= kBrickBatch. Ends
// with a barrier. The order within a bucket varies from run to run.
template <typename Left>
__device__ inline void order_batch(BrickOrder &o, uint16_t *s_idx, uint32_t m, float per_key, Left left)
{
    const uint32_t t = threadIdx.x;
    if (t < kBrickKeys) o.cnt[t] = 0;
    if (t == 0) o.next = 0;
    __syncthreads();
    uint32_t key[2], rank[2];
#pragma unroll
    for (uint32_t j = 0; j < 2; ++j) {
        const uint32_t q = j * kBrickThreads + t;
        if (q >= m) continue;
        key[j] = kBrickKeys - 1 - (uint32_t)fminf(fmaxf(left(q) * per_key, 0.0f), (float)(kBrickKeys - 1));
        rank[j] = atomicAdd(&o.cnt[key[j]], 1u);
    }
    __syncthreads();
    if (t < kBrickKeys) {  // one wave
        const uint32_t c = o.cnt[t];
        o.cnt[t] = dev::wave_incl_scan(c) - c;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < 2; ++j)
        if (j * kBrickThreads + t < m) s_idx[o.cnt[key[j]] + rank[j]] = (uint16_t)(j * kBrickThreads + t);
    __syncthreads();
}
static_assert(kBrickKeys == 64, "one wave scans the buckets");

// This wave's next 64 places of the batch (the first of them).
__device__ inline uint32_t next_places(BrickOrder &o)
{
    uint32_t c = 0;
    if ((threadIdx.x & 63) == 0) c = atomicAdd(&o.next, 64u);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)c);
}

template <bool kLib>
__global__ void __launch_bounds__(kBrickThreads)
march_brick_kernel(rafi_device_view view, rafi_ea_job job, uint32_t n_rays)
{
    extern __shared__ float region[];  // the brick's region, then s_idx
    __shared__ BrickOrder s_order;
    const uint64_t n = rafi_queue_length(view);
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t w = rafi_xcd_block(blockIdx.x, gridDim.x);
    uint64_t i = n * w / gridDim.x;
    const uint64_t end = n * (w + 1) / gridDim.x;
    const Item *__restrict__ in = static_cast<const Item *>(view.in_items);
    const Geo g = job_geo(job);
    const float per_key = (float)kBrickKeys * job.dt / (float)(g.b0 + g.b1 + g.b2);
    while (i < end) {
        const int32_t d = ea::find_domain(view.in_offsets, view.n_domains, i);
        const uint64_t seg_end = min(end, view.in_offsets[d + 1]);
        const Box box = ea::box_of(d, g);
        const ea::LdsVol vol(region, ea::region_of(box, g));
        ea::load_region<kBrickThreads>(region, job.volume, g.n, vol.r);
        uint16_t *s_idx = reinterpret_cast<uint16_t *>(region + vol.r.ex * vol.r.ey * vol.r.ez);
        for (; i < seg_end; i += kBrickBatch) {
            const uint32_t m = (uint32_t)min((uint64_t)kBrickBatch, seg_end - i);
            order_batch(s_order, s_idx, m, per_key, [&](uint32_t q) {
                const Item it = in[i + q];
                if ((uint32_t)it.ray >= n_rays) return 0.0f;
                float org[3], dir[3];
                int32_t K;
                job_ray(job, it.ray, org, dir, &K);
                return fminf(ea::exit_estimate(box, org, dir, job.dt), (float)K) - (float)it.k;
            });
            for (uint32_t c; (c = next_places(s_order)) < m;) {
                if (c + lane >= m) continue;
                const uint64_t slot = i + s_idx[c + lane];
                Item it = in[slot];
                if ((uint32_t)it.ray >= n_rays) {  // never true for items this library emitted
                    emit_item(view, job, slot, it, RAFI_POISON);
                    continue;
                }
                log_visit(job, it.ray, d);
                float org[3], dir[3];
                int32_t K;
                job_ray(job, it.ray, org, dir, &K);
                const int32_t dest =
                    K <= ea::kFloatK ? ea::march_through_lds<kLib>(vol, g, box, org, dir, K, job.dt, job.c, it)
                                     : ea::march_through<kLib>(job.volume, g, box, org, dir, K, job.dt, job.c, it);
                emit_ray(view, job, slot, it, dest);
            }
            __syncthreads();  // the order and the region are reused
        }
        i = seg_end;
    }
}

// ----------------------------------------------------------- adjoint ----
// Round 0 of the backward pass: every ray that sampled the volume starts at
// its last inside sample, in that sample's brick, with tau = tau_N, B = 0.
__global__ void __launch_bounds__(256)
bwd_seed_kernel(rafi_device_view view, rafi_ea_job job, uint64_t n_rays)
{
    const uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    if (r >= n_rays) return;
    if (job.visit_count) job.visit_count[r] = 0;
    const int32_t kl = job.klast[r];
    if (kl <= 0) {
        rafi_done(view, r);
        return;
    }
    const Geo g = job_geo(job);
    float org[3], dir[3];
    int32_t K;
    job_ray(job, (int32_t)r, org, dir, &K);
    float p[3];
    ea::sample_pos(org, dir, job.dt, kl - 1, p);
    rafi_forward_t(view, r, Item{(int32_t)r, kl - 1, job.tau[r], 0.0f}, ea::owner_of(p, g));
}

__device__ inline void scatter8(float *__restrict__ grad, int32_t n, const Tri &t, float s)
{
    const int64_t sy = n, sz = (int64_t)n * n;
    const float gx0 = 1.0f - t.f0, gy0 = 1.0f - t.f1, gz0 = 1.0f - t.f2;
    const float a00 = s * gz0 * gy0, a01 = s * gz0 * t.f1, a10 = s * t.f2 * gy0, a11 = s * t.f2 * t.f1;
    float *b = grad + t.base;
    unsafeAtomicAdd(b, a00 * gx0);
    unsafeAtomicAdd(b + 1, a00 * t.f0);
    unsafeAtomicAdd(b + sy, a01 * gx0);
    unsafeAtomicAdd(b + sy + 1, a01 * t.f0);
    unsafeAtomicAdd(b + sz, a10 * gx0);
    unsafeAtomicAdd(b + sz + 1, a10 * t.f0);
    unsafeAtomicAdd(b + sz + sy, a11 * gx0);
    unsafeAtomicAdd(b + sz + sy + 1, a11 * t.f0);
}

// Walk the ray's samples backwards through its brick:
//   tau <- tau - sigma_k (now the depth in front of k), T = exp(-tau),
//   a = 1 - exp(-sigma_k), dI/drho_k = T (a + c (1 - a)(rho_k - B)),
//   scatter dL/dI * dI/drho_k to the 8 voxels, B <- a rho_k + (1 - a) B.
__global__ void __launch_bounds__(256)
bwd_march_kernel(rafi_device_view view, rafi_ea_job job, const float *__restrict__ grad_image,
                 float *__restrict__ grad, uint32_t n_rays)
{
    // the grid may be sized for an upper bound: number the live workgroups only
    const uint64_t n_in = rafi_queue_length(view);
    const uint32_t nb = (uint32_t)((n_in + blockDim.x - 1) / blockDim.x);
    if (blockIdx.x >= nb) return;
    const uint64_t i = rafi_xcd_block(blockIdx.x, nb) * (uint64_t)blockDim.x + threadIdx.x;
    if (i >= n_in) return;
    const Geo g = job_geo(job);
    const int32_t d = ea::find_domain(view.in_offsets, view.n_domains, i);
    const Box box = ea::box_of(d, g);
    Item it = static_cast<const Item *>(view.in_items)[i];
    if ((uint32_t)it.ray >= n_rays) {
        rafi_forward_t(view, i, it, RAFI_POISON);
        return;
    }
    log_visit(job, it.ray, d);
    float org[3], dir[3];
    int32_t K;
    job_ray(job, it.ray, org, dir, &K);
    const float gI = grad_image[it.ray];
    const float c = job.c;
    float tau = it.tau, ctau = 0.0f, B = it.I;
    int32_t k = it.k;
    int32_t dest = RAFI_DONE;
    ea::Corners cc;
    for (; k >= 0; --k) {
        float p[3];
        ea::sample_pos(org, dir, job.dt, k, p);
        if (!box.contains(p)) {
            dest = ea::owner_of(p, g);
            break;
        }
        const Tri t = ea::tri_setup(g.n, p);
        const float rho = ea::density_cached(job.volume, g.n, t, cc);
        const float sigma = c * rho;
        // compensated tau -= sigma
        const float yt = -sigma - ctau;
        const float tt = tau + yt;
        ctau = (tt - tau) - yt;
        tau = tt;
        const float T = __expf(-tau);
        const float a = ea::one_minus_exp_neg(sigma);
        const float dIdrho = T * __fmaf_rn(c * (1.0f - a), rho - B, a);
        if (gI != 0.0f) scatter8(grad, g.n, t, gI * dIdrho);
        B = __fmaf_rn(a, rho - B, B);
    }
    it.k = k;
    it.tau = tau - ctau;
    it.I = B;
    if (k >= 0 && dest >= 0) rafi_forward_t(view, i, it, dest);
    else rafi_done(view, i);
}

// LDS-privatised backward: the workgroup accumulates dL/dV for the voxels its
// brick's samples touch -- the brick plus a one-voxel rim, (b+2)^3 floats -- in
// LDS, and each lane first sums its ray's contributions in registers while
// consecutive samples stay in the same trilinear cell. At the end the non-zero
// LDS entries are added to the global gradient. Bound by the latency of a
// turn's LDS round trips with the 16 waves one region leaves room for, and by
// VALU issue (58% of the slots): 64 views of 128^3 in 64 bricks, all backward
// launches 7.7 ms with lanes in queue order, both cells' corners swapped at
// every move and a brick test per sample, 3.9 ms in the form below.

// Add v[j] to the LDS floats p[o[j]], j < 4, as compare-and-swaps of the
// words' bits: the same single rounded float addition as an atomic add, in the
// same unspecified order. On gfx950 the native LDS float32 add (ds_add_f32)
// costs about 200 cycles per full wave, some 3 per active lane, while a 32-bit
// compare-and-swap costs about 27 (measured, 64 distinct words per wave).
// Every word is read, then every swap issued, then one wait. Swaps that lost a
// race (64 rays in a brick's cross-section of 1000 cells: about one a word)
// are tried again together with the value they found; a word already done
// takes a swap of some other value for that same value, which fails or
// rewrites the word unchanged.
__device__ inline void lds_add4(float *p, const int32_t o[4], const float v[4])
{
    uint32_t *w = reinterpret_cast<uint32_t *>(p);
    // the word as read, and as the swap found it: equal when it took
    uint32_t old[4], seen[4], miss[4];
    auto swap = [&](int j, uint32_t want) {
        (void)__hip_atomic_compare_exchange_strong(w + o[j], &seen[j], want, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WORKGROUP);
    };
#pragma unroll
    for (int j = 0; j < 4; ++j)
        seen[j] = old[j] = __hip_atomic_load(w + o[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
    for (int j = 0; j < 4; ++j) swap(j, __float_as_uint(__uint_as_float(old[j]) + v[j]));
#pragma unroll
    for (int j = 0; j < 4; ++j) miss[j] = seen[j] ^ old[j];
    while (miss[0] | miss[1] | miss[2] | miss[3]) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            seen[j] = old[j] = miss[j] ? seen[j] : ~seen[j];
            swap(j, miss[j] ? __float_as_uint(__uint_as_float(old[j]) + v[j]) : old[j]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) miss[j] = miss[j] ? seen[j] ^ old[j] : 0u;
    }
}

// A ray's pending gradient at the 8 corners of its current cell. The walk is
// monotone along each axis, so corners are numbered in the direction of
// travel: bit a of q set = ahead along axis a. Crossing a face leaves the 4
// corners behind it, which go to LDS, and keeps the other 4.
struct Pending {
    float a0, a1, a2, a3, a4, a5, a6, a7;
    float *p;            // corner 0
    int32_t ox, oy, oz;  // word offsets of the corner ahead, per axis

    __device__ void enter(float *corner)
    {
        p = corner;
        a0 = a1 = a2 = a3 = a4 = a5 = a6 = a7 = 0.0f;
    }
    // One cell on, along x, else along y, else along z.
    __device__ void cross(bool x, bool y)
    {
        const int32_t dx = ox, dy = oy, dz = oz;
        const float c0 = a0, c1 = a1, c2 = a2, c3 = a3, c4 = a4, c5 = a5, c6 = a6, c7 = a7;
        const int32_t o1 = x ? dy : dx, o2 = x || y ? dz : dy;
        const int32_t o[4] = {0, o1, o2, o1 + o2};
        const float v[4] = {c0, x ? c2 : c1, x || y ? c4 : c2, x ? c6 : (y ? c5 : c3)};
        lds_add4(p, o, v);
        p += x ? dx : (y ? dy : dz);
        a0 = x ? c1 : (y ? c2 : c4);
        a1 = x ? 0.0f : (y ? c3 : c5);
        a2 = x ? c3 : (y ? 0.0f : c6);
        a3 = x || y ? 0.0f : c7;
        a4 = x ? c5 : (y ? c6 : 0.0f);
        a5 = y ? c7 : 0.0f;
        a6 = x ? c7 : 0.0f;
        a7 = 0.0f;
    }
    __device__ void flush()
    {
        const int32_t lo[4] = {0, ox, oy, ox + oy}, hi[4] = {oz, oz + ox, oz + oy, oz + ox + oy};
        const float a[4] = {a0, a1, a2, a3}, b[4] = {a4, a5, a6, a7};
        lds_add4(p, lo, a);
        lds_add4(p, hi, b);
    }
};

// One ray's walk back through brick d (box, region r with its gradient gl).
__device__ inline void bwd_ray(const rafi_device_view &view, const rafi_ea_job &job,
                               const float *__restrict__ grad_image, uint32_t n_rays, int32_t d, const Geo &g,
                               const Box &box, const ea::Region &r, uint64_t slot, float *gl)
{
    Item it = static_cast<const Item *>(view.in_items)[slot];
    if ((uint32_t)it.ray >= n_rays) {
        rafi_forward_t(view, slot, it, RAFI_POISON);
        return;
    }
    log_visit(job, it.ray, d);
    float org[3], dir[3];
    int32_t K;
    job_ray(job, it.ray, org, dir, &K);
    const float gI = grad_image[it.ray], c = job.c, dt = job.dt;
    const int32_t first = ea::entry_sample(box, org, dir, dt, it.k);
    float tau = it.tau, ctau = 0.0f, B = it.I;
    int32_t k = it.k;
    if (k >= first) {
        // travel is toward smaller coordinates where dir dt > 0
        const bool nx = (dir[0] > 0.0f) == (dt > 0.0f), ny = (dir[1] > 0.0f) == (dt > 0.0f),
                   nz = (dir[2] > 0.0f) == (dt > 0.0f);
        Pending pend;
        pend.ox = nx ? -1 : 1;
        pend.oy = ny ? -r.ex : r.ex;
        pend.oz = nz ? -r.ex * r.ey : r.ex * r.ey;
        // the first sample's cell, then the cell of every sample, in local voxels
        auto corner = [&](int32_t x, int32_t y, int32_t z) {
            return gl + ((x + nx - r.ox) + r.ex * ((y + ny - r.oy) + r.ey * (z + nz - r.oz)));
        };
        auto setup = [&](int32_t j) {
            float p[3];
            ea::sample_pos(org, dir, dt, j, p);
            return ea::tri_setup_small(g.n, p);
        };
        Tri t = setup(k);
        int32_t mx = 0, my = 0, mz = 0;  // cells between the pending cell and sample k's
        pend.enter(corner(t.x, t.y, t.z));
        ea::Corners cc;
        ea::fetch_corners(job.volume, g.n, t, cc);
        // Per turn a lane crosses at most one face, and takes its sample once
        // it has reached the sample's cell: a lane that crosses two faces
        // between samples falls a turn behind instead of holding the wave's
        // other lanes in a second crossing.
        while (k >= first) {
            // A crossing flushes the corners the lane leaves, which hold only
            // earlier samples' terms: its LDS round trips overlap the gathers
            // issued for sample k.
            if (mx + my + mz > 3) {
                pend.flush();
                pend.enter(corner(t.x, t.y, t.z));
                mx = my = mz = 0;
            } else if (mx + my + mz > 0) {
                const bool x = mx > 0, y = !x && my > 0;
                pend.cross(x, y);
                mx -= x;
                my -= y;
                mz -= !x && !y;
            }
            if (mx + my + mz == 0) {
                // the forward march's per-sample forms: cached corners, the
                // hardware exponential, the series for 1 - exp(-sigma)
                const float rho = ea::interp_corners(cc, t);
                const float sigma = c * rho;
                const float yt = -sigma - ctau;
                const float tt = tau + yt;
                ctau = (tt - tau) - yt;
                tau = tt;
                const float T = __expf(-tau);
                const float a = ea::one_minus_exp_neg(sigma);
                const float dIdrho = T * __fmaf_rn(c * (1.0f - a), rho - B, a);
                B = __fmaf_rn(a, rho - B, B);
                if (gI != 0.0f) {
                    const float s = gI * dIdrho;
                    const float gx = 1.0f - t.f0, gy = 1.0f - t.f1, gz = 1.0f - t.f2;
                    // weights behind and ahead
                    const float x0 = nx ? t.f0 : gx, x1 = nx ? gx : t.f0;
                    const float y0 = ny ? t.f1 : gy, y1 = ny ? gy : t.f1;
                    const float z0 = nz ? t.f2 : gz, z1 = nz ? gz : t.f2;
                    const float a00 = s * z0 * y0, a01 = s * z0 * y1, a10 = s * z1 * y0, a11 = s * z1 * y1;
                    pend.a0 += a00 * x0;
                    pend.a1 += a00 * x1;
                    pend.a2 += a01 * x0;
                    pend.a3 += a01 * x1;
                    pend.a4 += a10 * x0;
                    pend.a5 += a10 * x1;
                    pend.a6 += a11 * x0;
                    pend.a7 += a11 * x1;
                }
                --k;
                const Tri u = setup(max(k, first));
                if (gI != 0.0f) {
                    mx = abs(u.x - t.x);
                    my = abs(u.y - t.y);
                    mz = abs(u.z - t.z);
                }
                t = u;
                ea::fetch_corners(job.volume, g.n, t, cc);
            }
            // one latch: every lane ends its turn here (without it the
            // compiler makes two nested loops of the two kinds of turns)
            __builtin_amdgcn_wave_barrier();
        }
        if (gI != 0.0f) pend.flush();
    }
    it.k = k;
    it.tau = tau - ctau;
    it.I = B;
    int32_t dest = RAFI_DONE;
    if (k >= 0) {
        float p[3];
        ea::sample_pos(org, dir, dt, k, p);
        dest = ea::owner_of(p, g);
    }
    if (dest >= 0) rafi_forward_t(view, slot, it, dest);
    else rafi_done(view, slot);
}

// The backward of the queue items [first, last), all in domain d, by the whole
// workgroup: zero the brick's gradient region in LDS, walk every ray back
// through the brick accumulating into it, then add its non-zero entries to
// the global gradient. Rays go through in batches of kBrickBatch ordered by
// the samples they have left in the brick; ordered = 0: in queue order, where
// the LDS has no room for the order; order = nullptr: by a fixed stride, where it
// has none beside the region (8 x 62 x 62 voxels and their rim).
__device__ inline void bwd_segment(const rafi_device_view &view, const rafi_ea_job &job,
                                   const float *__restrict__ grad_image, float *__restrict__ grad, uint32_t n_rays,
                                   int32_t d, uint64_t first, uint64_t last, int ordered, float *gl, BrickOrder *order)
{
    const Geo g = job_geo(job);
    const Box box = ea::box_of(d, g);
    const ea::Region r = ea::region_of(box, g);
    const int32_t nl = r.ex * r.ey * r.ez;
    const uint32_t lane = threadIdx.x & 63;
    for (int32_t k = threadIdx.x; k < nl; k += kBrickThreads) gl[k] = 0.0f;
    uint16_t *s_idx = reinterpret_cast<uint16_t *>(gl + nl);
    const float per_key = (float)kBrickKeys * job.dt / (float)(g.b0 + g.b1 + g.b2);
    if (!order) {
        __syncthreads();
        for (uint64_t i = first + threadIdx.x; i < last; i += kBrickThreads)
            bwd_ray(view, job, grad_image, n_rays, d, g, box, r, i, gl);
        __syncthreads();
        first = last;
    }
    for (uint64_t i = first; i < last; i += kBrickBatch) {
        const uint32_t m = (uint32_t)min((uint64_t)kBrickBatch, last - i);
        if (ordered) {
            order_batch(*order, s_idx, m, per_key, [&](uint32_t q) {
                const Item it = static_cast<const Item *>(view.in_items)[i + q];
                if ((uint32_t)it.ray >= n_rays) return 0.0f;
                float org[3], dir[3];
                int32_t K;
                job_ray(job, it.ray, org, dir, &K);
                return (float)it.k - fmaxf(ea::entry_estimate(box, org, dir, job.dt), 0.0f);
            });
        } else {
            if (threadIdx.x == 0) order->next = 0;
            __syncthreads();
        }
        for (uint32_t c; (c = next_places(*order)) < m;)
            if (c + lane < m)
                bwd_ray(view, job, grad_image, n_rays, d, g, box, r, i + (ordered ? s_idx[c + lane] : c + lane), gl);
        __syncthreads();  // the order is reused, and after the last batch the region is complete
    }
    for (ea::RegionWalk<kBrickThreads> at(r); at.k < nl; at.step(r)) {
        const float v = gl[at.k];
        if (v != 0.0f)
            unsafeAtomicAdd(&grad[(r.ox + at.x) + (int64_t)g.n * ((r.oy + at.y) + (int64_t)g.n * (r.oz + at.z))], v);
    }
    __syncthreads();  // the region is reused by the next segment
}

// The brick's order outside the dynamic LDS, or none (kOrder = false).
template <bool kOrder>
__device__ inline BrickOrder *brick_order()
{
    if constexpr (kOrder) {
        __shared__ BrickOrder order;
        return &order;
    }
    return nullptr;
}

// One workgroup per domain-pure tile of the input queue.
template <bool kOrder>
__global__ void __launch_bounds__(kBrickThreads)
bwd_march_lds_kernel(rafi_device_view view, rafi_ea_job job, const float *__restrict__ grad_image,
                     float *__restrict__ grad, uint32_t n_rays, int ordered)
{
    extern __shared__ float gl[];
    uint64_t tb, te;
    const int32_t d = rafi_tile(view, rafi_xcd_block(blockIdx.x, gridDim.x), &tb, &te);
    bwd_segment(view, job, grad_image, grad, n_rays, d, tb, te, ordered, gl, brick_order<kOrder>());
}

// One workgroup per CU, each taking an equal contiguous slice of the queue
// and working through the brick segments it spans (usually one or two), so
// every CU is busy for the whole launch and the gradient region is flushed
// about once per workgroup.
template <bool kOrder>
__global__ void __launch_bounds__(kBrickThreads)
bwd_march_range_kernel(rafi_device_view view, rafi_ea_job job, const float *__restrict__ grad_image,
                       float *__restrict__ grad, uint32_t n_rays, int ordered)
{
    extern __shared__ float gl[];
    const uint64_t w = rafi_xcd_block(blockIdx.x, gridDim.x);
    const uint64_t n = rafi_queue_length(view);
    uint64_t i = n * w / gridDim.x;
    const uint64_t end = n * (w + 1) / gridDim.x;
    while (i < end) {
        const int32_t d = ea::find_domain(view.in_offsets, view.n_domains, i);
        const uint64_t seg_end = min(end, view.in_offsets[d + 1]);
        bwd_segment(view, job, grad_image, grad, n_rays, d, i, seg_end, ordered, gl, brick_order<kOrder>());
        i = seg_end;
    }
}

// Bytes of a brick region (brick + one-voxel rim) in LDS.
size_t region_bytes(const rafi_ea_job *j)
{
    return sizeof(float) * (size_t)(j->n / j->grid[0] + 2) * (j->n / j->grid[1] + 2) * (j->n / j->grid[2] + 2);
}

// The brick kernels' batch order and their static LDS (rounded up).
constexpr size_t kOrderBytes = kBrickBatch * sizeof(uint16_t);
constexpr size_t kBrickStatic = (sizeof(BrickOrder) + 63) / 64 * 64;

size_t max_lds_bytes()
{
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        return 0;
    return (size_t)v;
}

bool job_ok(const rafi_ctx *c, const rafi_ea_job *j)
{
    if (!c || !j || !j->volume || !j->views || !j->image) return false;
    if (j->n < 2 || j->n_views < 1 || j->width < 1 || j->height < 1) return false;
    for (int a = 0; a < 3; ++a)
        if (j->grid[a] < 1 || j->n % j->grid[a] != 0) return false;
    if (c->D != j->grid[0] * j->grid[1] * j->grid[2] || c->S != RAFI_EA_ITEM_BYTES) return false;
    if (j->visit_log && (!j->visit_count || j->visit_stride < 1)) return false;
    if (j->emit_mode != RAFI_SLOTS_ORDERED && j->emit_mode != RAFI_SLOTS_APPEND) return false;
    const uint64_t rays = (uint64_t)j->n_views * j->width * j->height;
    return rays <= c->cap && rays < (1ull << 31);
}

int cu_count(int *cus)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || *cus < 1)
        return RAFI_ERR_HIP;
    return RAFI_OK;
}

uint32_t n_rays_of(const rafi_ea_job *j) { return (uint32_t)((uint64_t)j->n_views * j->width * j->height); }

// The brick kernel is taken when a segment holds 1536 rays or more on average:
// the part of a workgroup's slice that lies in one brick, of which there are at
// most the workgroups' number and the bricks' together. Below that the bricks'
// loads and barriers, and the longest chords of a part-filled batch, cost more
// than the gathers. 64-view render of 128^3 in 64 bricks: all launches brick 1.77
// ms, from 100 K rays 1.72, from 400 K 1.645, never 2.26. Launches of 0.5 to 2 M
// rays over 64 to 8000 bricks, us brick and gather: 2.0 M in 512 bricks 143 and
// 230 (2700 rays a segment), in 1024 bricks 1.9 M 207 and 166 (1480), in 8000
// 0.49 M 590 and 53 (60).
constexpr uint64_t kBrickRays = 1536;

// One march launch over the view's n_in queued rays (an upper bound is enough).
template <bool kLib>
void launch_march_as(const rafi_device_view &v, const rafi_ea_job *job, int cus, hipStream_t s)
{
    if (!v.n_in) return;
    const size_t lds = region_bytes(job) + kOrderBytes;
    const uint64_t segments = (uint64_t)cus + (uint64_t)v.n_domains;
    if (job->n <= ea::kSmallN && v.n_in >= kBrickRays * segments && lds + kBrickStatic <= max_lds_bytes())
        hipLaunchKernelGGL(march_brick_kernel<kLib>, dim3(cus), dim3(kBrickThreads), lds, s, v, *job,
                           n_rays_of(job));
    else
        hipLaunchKernelGGL(march_kernel<kLib>, dim3((uint32_t)((v.n_in + 255) / 256)), dim3(256), 0, s, v, *job,
                           n_rays_of(job));
}

// Contexts with tiles of 512 items or more, and bricks that fit in LDS, march
// with the library's exponentials (rafi_set_tile_items).
int launch_march(rafi_ctx *c, const rafi_device_view &v, const rafi_ea_job *job)
{
    int cus = 0;
    if (cu_count(&cus) != RAFI_OK) return RAFI_ERR_HIP;
    const int ph = prof_domain_begin(c);
    if (v.tile_items >= 512 && region_bytes(job) <= max_lds_bytes()) launch_march_as<true>(v, job, cus, c->stream);
    else launch_march_as<false>(v, job, cus, c->stream);
    prof_domain_end(c, ph);
    RAFI_LAUNCH_CHECK();
    return RAFI_OK;
}

}  // namespace
}  // namespace rafi

using namespace rafi;

extern "C" {

int rafi_ea_raygen(rafi_ctx *c, const rafi_ea_job *job)
{
    if (!job_ok(c, job)) return RAFI_ERR_ARG;
    const uint64_t rays = n_rays_of(job);
    int rc = rafi_begin(c, rays);
    if (rc != RAFI_OK) return rc;
    rafi_device_view v;
    rafi_view(c, &v);
    if (rays)
        hipLaunchKernelGGL(raygen_kernel, dim3((uint32_t)((rays + 255) / 256)), dim3(256), 0, c->stream, v,
                           *job, rays);
    RAFI_LAUNCH_CHECK();
    return RAFI_OK;
}

int rafi_ea_march(rafi_ctx *c, const rafi_ea_job *job)
{
    if (!job_ok(c, job)) return RAFI_ERR_ARG;
    rafi_device_view v;
    rafi_view(c, &v);
    return launch_march(c, v, job);
}

int rafi_ea_render(rafi_ctx *c, const rafi_ea_job *job, int32_t max_rounds, int32_t *rounds)
{
    if (!job_ok(c, job) || max_rounds < 1) return RAFI_ERR_ARG;
    const int rc = rafi_ea_raygen(c, job);
    if (rc != RAFI_OK) return rc;
    // launched one step ahead of the host (run_rounds)
    auto launch = [&](uint64_t bound) -> int {
        const int orc = rafi_open(c, bound, job->emit_mode);
        if (orc != RAFI_OK) return orc;
        rafi_device_view v;
        rafi_view(c, &v);
        v.n_in = bound;
        return launch_march(c, v, job);
    };
    return run_rounds(c, max_rounds, rounds, nullptr, launch, [](uint64_t n) { return n; });
}

int rafi_ea_backward(rafi_ctx *c, const rafi_ea_job *job, const float *grad_image, float *grad_volume,
                     int32_t max_rounds, int32_t *rounds)
{
    if (!job_ok(c, job) || !job->tau || !job->klast || !grad_image || !grad_volume || max_rounds < 1)
        return RAFI_ERR_ARG;
    const uint64_t rays = n_rays_of(job);
    int rc = rafi_begin(c, rays);
    if (rc != RAFI_OK) return rc;
    rafi_device_view v;
    rafi_view(c, &v);
    if (rays)
        hipLaunchKernelGGL(bwd_seed_kernel, dim3((uint32_t)((rays + 255) / 256)), dim3(256), 0, c->stream, v,
                           *job, rays);
    RAFI_LAUNCH_CHECK();
    // LDS privatisation when the brick's region fits a workgroup's LDS
    const size_t room = max_lds_bytes(), need = region_bytes(job) + kBrickStatic;
    // (a brick that fits, of at most 8192, makes n < 690: the 32-bit cell index)
    const bool use_lds = region_bytes(job) <= room && job->n <= ea::kSmallN, alone = need > room;
    const int ordered = need + kOrderBytes <= room;
    const size_t lds = region_bytes(job) + (ordered ? kOrderBytes : 0);
    int cus = 0;
    if (cu_count(&cus) != RAFI_OK) return RAFI_ERR_HIP;
    if (use_lds && job->bwd_tile_items) {  // tile per workgroup: the host's tile count sizes the grid
        const uint32_t saved_tile = c->tile_items;
        c->tile_items = job->bwd_tile_items;
        int32_t r = 0;
        for (;;) {
            uint64_t total = 0;
            rc = rafi_round(c, nullptr, &total);
            ++r;
            if (rc != RAFI_OK || total == 0) break;
            if (r >= max_rounds) { rc = RAFI_ERR_MAX_ROUNDS; break; }
            rafi_view(c, &v);
            const int ph = prof_domain_begin(c);
            hipLaunchKernelGGL(alone ? bwd_march_lds_kernel<false> : bwd_march_lds_kernel<true>, dim3(v.n_tiles),
                               dim3(kBrickThreads), lds, c->stream, v, *job, grad_image, grad_volume, (uint32_t)rays,
                               ordered);
            prof_domain_end(c, ph);
            rc = hipGetLastError() == hipSuccess ? RAFI_OK : RAFI_ERR_HIP;
            if (rc != RAFI_OK) break;
        }
        c->tile_items = saved_tile;
        if (rounds) *rounds = r;
        return rc;
    }
    // one workgroup per CU over slices of the queue (or global atomics when the
    // brick's region does not fit), launched one step ahead of the host
    auto launch = [&](uint64_t bound) -> int {
        const int orc = rafi_open(c, bound, RAFI_SLOTS_ORDERED);
        if (orc != RAFI_OK) return orc;
        rafi_device_view lv;
        rafi_view(c, &lv);
        lv.n_in = bound;
        const int ph = prof_domain_begin(c);
        if (bound && use_lds) {
            // at least 256 rays a workgroup: a small launch spreads over the CUs,
            // where its few waves take turns four times as fast (128^3, 64 views:
            // the 100 K rays of round 9 241 us in 100 workgroups, 229 in 256)
            const uint64_t want = (bound + 255) / 256;
            const uint32_t blocks = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(want, cus));
            hipLaunchKernelGGL(alone ? bwd_march_range_kernel<false> : bwd_march_range_kernel<true>, dim3(blocks),
                               dim3(kBrickThreads), lds, c->stream, lv, *job, grad_image, grad_volume, (uint32_t)rays,
                               ordered);
        } else if (bound) {
            hipLaunchKernelGGL(bwd_march_kernel, dim3((uint32_t)((bound + 255) / 256)), dim3(256), 0, c->stream,
                               lv, *job, grad_image, grad_volume, (uint32_t)rays);
        }
        prof_domain_end(c, ph);
        RAFI_LAUNCH_CHECK();
        return RAFI_OK;
    };
    return run_rounds(c, max_rounds, rounds, nullptr, launch, [](uint64_t n) { return n; });
}

}  // extern "C"
