// Stable multi-split by destination: the forward step of the library.
//
// What it computes (Sec. 4.2.1-4.2.2 of the paper, collapsed to one device):
// slot i with destination e in [0, D) lands at
//     offset[e] + #{ j < i : dest[j] == e },
// offset[] being the exclusive prefix of the per-destination counts; slots
// with RAFI_DONE leave, slots with any other out-of-range value are dropped;
// both are counted. The paper reaches the same placement with a radix sort of
// (dest << 32 | i) keys, a gather and a begin/end tally; here it is three
// HBM-streaming passes (the second, for few destinations, inside the third):
//
//   1. hist    per tile of T slots, a destination histogram (LDS atomics),
//              written destination-major: table[e * n_tiles + tile].
//   2. scan    one exclusive scan over the flattened table. Entry
//              (e, tile) then holds the output position of the tile's first
//              item bound for e, and row starts are the offsets.
//   3. scatter per tile, each wavefront owns a contiguous quarter; per-wave
//              counts give each wave its base per destination, and inside a
//              wave the rank of a lane among same-destination lanes comes from
//              a ballot match over the destination bits. Items are copied as
//              4-byte words (16-byte vectors when the size allows).
#include "internal.h"
#include "split_device.h"

#include <algorithm>

namespace rafi {
namespace {

constexpr int kScanThreads = 256;
constexpr int kScanPer = 16;                       // elements per thread
constexpr int kScanChunk = kScanThreads * kScanPer;  // 4096
constexpr int kPartThreads = 1024;
constexpr int kPartMax = kPartThreads * kScanPer;  // 16384 partial sums
// Up to this many scan chunks, each chunk of the apply pass sums the earlier
// chunks' totals itself (at most 2 MiB read over the whole launch), which
// saves the launch that scans the partial sums.
constexpr uint32_t kDirectMaxBlocks = 1024;

using dev::block_excl_scan;
using dev::bucket_of;
using dev::load_nt4;
using dev::match_peers;

// ---------------------------------------------------------------- pass 1 ---
// Where the count of destination e in column c of a table is: at
// e * row + c * col, destination-major for the scans (col = 1), or column by
// column for the scatter that sums the columns itself (row = 1).
struct TableLayout {
    uint32_t row, col;
    __device__ uint64_t at(uint32_t e, uint32_t c) const { return (uint64_t)e * row + (uint64_t)c * col; }
};

// Four destinations into an LDS histogram; four equal ones are one addition
// (lanes that add to one word take turns).
__device__ inline void add_four(uint32_t *h, const uint4 &d, int32_t D)
{
    const uint32_t x = bucket_of((int32_t)d.x, D), y = bucket_of((int32_t)d.y, D), z = bucket_of((int32_t)d.z, D),
                   w = bucket_of((int32_t)d.w, D);
    if (x == y && x == z && x == w) {
        atomicAdd(&h[x], 4u);
    } else {
        atomicAdd(&h[x], 1u);
        atomicAdd(&h[y], 1u);
        atomicAdd(&h[z], 1u);
        atomicAdd(&h[w], 1u);
    }
}

// Destination histogram of tile blockIdx.x into column blockIdx.x of table.
__device__ inline void hist_tile(const int32_t *__restrict__ dest, uint64_t n, int32_t D, uint32_t T,
                                 TableLayout layout, uint32_t *__restrict__ table, uint32_t *h)
{
    const uint32_t rows = (uint32_t)D + 2u;
    for (uint32_t e = threadIdx.x; e < rows; e += blockDim.x) h[e] = 0;
    __syncthreads();
    const uint64_t start = (uint64_t)blockIdx.x * T;
    const uint64_t end = min(start + T, n);
    // T is a multiple of 1024 and dest is 16-byte aligned: whole int4 groups,
    // loaded kU at a time before the LDS atomics so the loads overlap.
    constexpr int kU = 8;
    const uint64_t vend = start + ((end - start) & ~(uint64_t)3);
    const uint64_t stride = 4ull * blockDim.x;
    uint64_t i = start + 4ull * threadIdx.x;
    for (; i + (kU - 1) * stride < vend; i += kU * stride) {
        uint4 d4[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) d4[u] = load_nt4(dest + i + u * stride);
#pragma unroll
        for (int u = 0; u < kU; ++u) add_four(h, d4[u], D);
    }
    for (; i < vend; i += stride) {
        add_four(h, *reinterpret_cast<const uint4 *>(dest + i), D);
    }
    for (uint64_t j = vend + threadIdx.x; j < end; j += blockDim.x) atomicAdd(&h[bucket_of(dest[j], D)], 1u);
    __syncthreads();
    for (uint32_t e = threadIdx.x; e < rows; e += blockDim.x) table[layout.at(e, blockIdx.x)] = h[e];
}

__global__ void __launch_bounds__(256)
hist_kernel(const int32_t *__restrict__ dest, uint64_t n, int32_t D, uint32_t T, TableLayout layout,
            uint32_t *__restrict__ table)
{
    extern __shared__ uint32_t h[];  // D + 2
    hist_tile(dest, n, D, T, layout, table, h);
}

// Lockstep plans: tiles of kLockTile chunks of kLockChunk slots. Besides the
// tile's column of the table, pre[c * D + e] = items of chunk c's tile bound
// for e in the chunks before c (at most (kLockTile - 1) * kLockChunk, which
// fits 16 bits).
constexpr uint32_t kLockChunk = 2048;  // slots per chunk: 8 waves x 4 rounds x 64 lanes
constexpr uint32_t kLockTile = 32;     // chunks per tile: one per CU of an XCD
constexpr uint32_t kLockXcds = 8;
static_assert((kLockTile - 1) * kLockChunk < 65536, "chunk prefixes are 16-bit");

// s_waitcnt immediate for lgkmcnt(0) alone (vmcnt and expcnt at their
// maxima, i.e. not waited on).
constexpr int kWaitLds = 0xc07f;

__global__ void __launch_bounds__(256)
hist_lock_kernel(const int32_t *__restrict__ dest, uint64_t n, int32_t D, uint32_t n_tiles, uint32_t n_chunks,
                 uint32_t *__restrict__ table, uint16_t *__restrict__ pre)
{
    extern __shared__ uint32_t h[];  // D + 2
    const uint32_t rows = (uint32_t)D + 2u;
    for (uint32_t e = threadIdx.x; e < rows; e += blockDim.x) h[e] = 0;
    __syncthreads();
    const uint32_t c_first = blockIdx.x * kLockTile;
    const uint32_t c_end = min(c_first + kLockTile, n_chunks);
    static_assert(kLockChunk == 2 * 4 * 256, "two int4 groups per thread per chunk");
    for (uint32_t c = c_first; c < c_end; ++c) {
        const uint64_t s0 = (uint64_t)c * kLockChunk;
        const bool full = s0 + kLockChunk <= n;
        // dest is 16-byte aligned and chunks start at multiples of 2048
        uint4 a = make_uint4(0, 0, 0, 0), b = make_uint4(0, 0, 0, 0);
        if (full) {
            a = load_nt4(dest + s0 + 4 * threadIdx.x);
            b = load_nt4(dest + s0 + 1024 + 4 * threadIdx.x);
        }
        for (uint32_t e = threadIdx.x; e < (uint32_t)D; e += blockDim.x)
            pre[(uint64_t)c * (uint32_t)D + e] = (uint16_t)h[e];
        __syncthreads();  // every count read before it changes
        if (full) {
            atomicAdd(&h[bucket_of((int32_t)a.x, D)], 1u);
            atomicAdd(&h[bucket_of((int32_t)a.y, D)], 1u);
            atomicAdd(&h[bucket_of((int32_t)a.z, D)], 1u);
            atomicAdd(&h[bucket_of((int32_t)a.w, D)], 1u);
            atomicAdd(&h[bucket_of((int32_t)b.x, D)], 1u);
            atomicAdd(&h[bucket_of((int32_t)b.y, D)], 1u);
            atomicAdd(&h[bucket_of((int32_t)b.z, D)], 1u);
            atomicAdd(&h[bucket_of((int32_t)b.w, D)], 1u);
        } else {
            for (uint64_t i = s0 + threadIdx.x; i < n; i += blockDim.x) atomicAdd(&h[bucket_of(dest[i], D)], 1u);
        }
        // Every wave's LDS atomics complete before the barrier: LDS requests
        // of different waves can complete out of order, and the compiler
        // has been seen to drop this wait when the next read of the counts
        // is reached through the loop's back edge.
        __builtin_amdgcn_s_waitcnt(kWaitLds);
        __syncthreads();
    }
    for (uint32_t e = threadIdx.x; e < rows; e += blockDim.x)
        table[(uint64_t)e * n_tiles + blockIdx.x] = h[e];
}

// ---------------------------------------------------------------- pass 2 ---
__device__ inline void load16(const uint32_t *__restrict__ a, uint64_t M, uint64_t base, uint32_t v[kScanPer])
{
    if (base + kScanPer <= M) {
        const uint4 *p = reinterpret_cast<const uint4 *>(a + base);
#pragma unroll
        for (int k = 0; k < kScanPer / 4; ++k) {
            uint4 q = p[k];
            v[4 * k] = q.x; v[4 * k + 1] = q.y; v[4 * k + 2] = q.z; v[4 * k + 3] = q.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < kScanPer; ++k) v[k] = (base + k < M) ? a[base + k] : 0u;
    }
}

// a[base + k] = run + v[0] + ... + v[k - 1] for the thread's 16 entries
__device__ inline void store16_excl(uint32_t *__restrict__ a, uint64_t M, uint64_t base, const uint32_t v[kScanPer],
                                    uint32_t run)
{
    if (base + kScanPer <= M) {
        uint4 *p = reinterpret_cast<uint4 *>(a + base);
#pragma unroll
        for (int k = 0; k < kScanPer / 4; ++k) {
            uint4 q;
            q.x = run; run += v[4 * k];
            q.y = run; run += v[4 * k + 1];
            q.z = run; run += v[4 * k + 2];
            q.w = run; run += v[4 * k + 3];
            p[k] = q;
        }
    } else {
#pragma unroll
        for (int k = 0; k < kScanPer; ++k) {
            if (base + k < M) a[base + k] = run;
            run += v[k];
        }
    }
}

__global__ void __launch_bounds__(kScanThreads)
scan_reduce_kernel(const uint32_t *__restrict__ a, uint64_t M, uint32_t *__restrict__ part)
{
    __shared__ uint32_t lds[kScanThreads / 64 + 1];
    uint32_t v[kScanPer];
    load16(a, M, (uint64_t)blockIdx.x * kScanChunk + (uint64_t)threadIdx.x * kScanPer, v);
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) s += v[k];
    uint32_t tot;
    block_excl_scan<kScanThreads>(s, lds, &tot);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(kPartThreads)
scan_partials_kernel(uint32_t *__restrict__ part, uint32_t nb)
{
    __shared__ uint32_t lds[kPartThreads / 64 + 1];
    uint32_t v[kScanPer];
    const uint64_t base = (uint64_t)threadIdx.x * kScanPer;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) v[k] = (base + k < nb) ? part[base + k] : 0u;
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) s += v[k];
    uint32_t tot;
    uint32_t run = block_excl_scan<kPartThreads>(s, lds, &tot);
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        if (base + k < nb) part[base + k] = run;
        run += v[k];
    }
}

__global__ void __launch_bounds__(kScanThreads)
scan_apply_kernel(uint32_t *__restrict__ a, uint64_t M, const uint32_t *__restrict__ part)
{
    __shared__ uint32_t lds[kScanThreads / 64 + 1];
    uint32_t v[kScanPer];
    const uint64_t base = (uint64_t)blockIdx.x * kScanChunk + (uint64_t)threadIdx.x * kScanPer;
    load16(a, M, base, v);
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) s += v[k];
    uint32_t tot;
    uint32_t run = block_excl_scan<kScanThreads>(s, lds, &tot) + part[blockIdx.x];
    store16_excl(a, M, base, v, run);
}

// scan_apply_kernel with the chunk's offset summed here from the chunks'
// totals (part as scan_reduce_kernel left it) instead of by a separate scan.
__global__ void __launch_bounds__(kScanThreads)
scan_apply_direct_kernel(uint32_t *__restrict__ a, uint64_t M, const uint32_t *__restrict__ part)
{
    __shared__ uint32_t lds[kScanThreads / 64 + 1];
    uint32_t before = 0;
    for (uint32_t j = threadIdx.x; j < blockIdx.x; j += kScanThreads) before += part[j];
    uint32_t off;
    (void)block_excl_scan<kScanThreads>(before, lds, &off);
    uint32_t v[kScanPer];
    const uint64_t base = (uint64_t)blockIdx.x * kScanChunk + (uint64_t)threadIdx.x * kScanPer;
    load16(a, M, base, v);
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) s += v[k];
    uint32_t tot;
    uint32_t run = block_excl_scan<kScanThreads>(s, lds, &tot) + off;
    store16_excl(a, M, base, v, run);
}

// Offsets, summary and the tile table for domain-pure launches, from the
// scanned table; with `dropped`, its count goes to summary[4] and is reset
// (the domain kernels that add to it have completed).
struct Results {
    uint64_t *offsets, *summary;
    uint32_t *tile_offsets;
    uint32_t tile_items;
    unsigned long long *dropped;
    HostOut host;
};

template <int NT, typename RowStart>
__device__ inline void finalize_body(RowStart row_start, int32_t D, uint64_t n, const Results &to, uint32_t *lds)
{
    uint64_t *__restrict__ offsets = to.offsets, *__restrict__ summary = to.summary;
    uint32_t *__restrict__ tile_offsets = to.tile_offsets;
    const uint32_t tile_items = to.tile_items;
    unsigned long long *__restrict__ dropped = to.dropped;
    const HostOut &host = to.host;
    for (int32_t e = threadIdx.x; e <= D; e += NT) {
        const uint64_t o = row_start(e);
        offsets[e] = o;
        if (host.offsets) host.offsets[e] = o;
    }
    const uint64_t total = row_start(D);
    const uint64_t done_end = row_start(D + 1);
    // per-domain tile counts, scanned (each thread owns a contiguous run)
    const int32_t per = (D + NT - 1) / NT;
    const int32_t e0 = threadIdx.x * per;
    uint32_t local = 0;
    for (int32_t e = e0; e < min(e0 + per, D); ++e) {
        uint64_t c = row_start(e + 1) - row_start(e);
        local += (uint32_t)((c + tile_items - 1) / tile_items);
    }
    uint32_t tot;
    uint32_t run = block_excl_scan<NT>(local, lds, &tot);
    if (tile_offsets) {
        for (int32_t e = e0; e < min(e0 + per, D); ++e) {
            tile_offsets[e] = run;
            uint64_t c = row_start(e + 1) - row_start(e);
            run += (uint32_t)((c + tile_items - 1) / tile_items);
        }
        if (threadIdx.x == 0) tile_offsets[D] = tot;
    }
    if (host.offsets) {
        __threadfence_system();
        __syncthreads();  // the offsets before the sequence number
    }
    if (threadIdx.x == 0) {
        const uint64_t lost = dropped ? *dropped : 0ull;
        summary[0] = total;
        summary[1] = done_end - total;
        summary[2] = n - done_end;
        summary[3] = tot;
        if (dropped) {
            summary[4] = lost;
            *dropped = 0;
        }
        if (host.words) {
            host.words[0] = total;
            host.words[1] = done_end - total;
            host.words[2] = n - done_end;
            host.words[3] = tot;
            host.words[4] = lost;
            __threadfence_system();
            __hip_atomic_store(host.words + 7, host.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

__global__ void __launch_bounds__(1024)
finalize_kernel(const uint32_t *__restrict__ table, uint32_t n_cols, int32_t D, uint64_t n, Results to)
{
    __shared__ uint32_t lds[1024 / 64 + 1];
    finalize_body<1024>(
        [&](int32_t e) { return n_cols ? (uint64_t)table[(uint64_t)e * n_cols] : 0ull; }, D, n, to, lds);
}

// The scan and finalize in one launch by one workgroup, 16 entries a thread:
// 5 us, where the three launches take about 8 back to back; a loop over twice
// the entries takes 9.
constexpr uint64_t kOneScanMax = 1024ull * kScanPer;

__global__ void __launch_bounds__(1024)
scan_one_kernel(uint32_t *__restrict__ table, uint64_t M, uint32_t n_cols, int32_t D, uint64_t n, Results to)
{
    __shared__ uint32_t lds[1024 / 64 + 1];
    const uint64_t mine = (uint64_t)threadIdx.x * kScanPer;
    uint32_t v[kScanPer], s = 0, tot;
    load16(table, M, mine, v);
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) s += v[k];
    const uint32_t run = block_excl_scan<1024>(s, lds, &tot);
    store16_excl(table, M, mine, v, run);
    __syncthreads();
    finalize_body<1024>([&](int32_t e) { return (uint64_t)table[(uint64_t)e * n_cols]; }, D, n, to, lds);
}

// True in exactly one workgroup of the launch: the last to get here. Each
// workgroup's global writes before the call are visible to that one (device
// fences around a count of finished workgroups). The counter is zero between
// launches: the last workgroup resets it.
__device__ inline bool last_workgroup(uint32_t *counter, uint32_t n_groups)
{
    __shared__ uint32_t is_last;
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) is_last = atomicAdd(counter, 1u) == n_groups - 1 ? 1u : 0u;
    __syncthreads();
    if (!is_last) return false;
    __threadfence();
    if (threadIdx.x == 0) atomicExch(counter, 0u);
    return true;
}

// Exclusive scan of a[0, m) in place by one workgroup of NT threads, each
// owning a contiguous run (m small).
template <int NT>
__device__ inline void block_scan_inplace(uint32_t *a, uint64_t m, uint32_t *lds)
{
    const uint64_t per = (m + NT - 1) / NT;
    const uint64_t b0 = min((uint64_t)threadIdx.x * per, m), b1 = min(b0 + per, m);
    uint32_t sum = 0;
    for (uint64_t k = b0; k < b1; ++k) sum += a[k];
    uint32_t tot;
    uint32_t run = block_excl_scan<NT>(sum, lds, &tot);
    for (uint64_t k = b0; k < b1; ++k) {
        const uint32_t v = a[k];
        a[k] = run;
        run += v;
    }
    __syncthreads();
}

// ----------------------------------------------------- passes 1 + 2 fused ---
// For a small count table (M entries): every workgroup writes its tile's
// histogram, and the last one to finish (a device-scope fence, then an atomic
// count of finished tiles) scans the whole table in place and finalizes. No
// workgroup waits for another. The counter is zero between launches: the last
// workgroup resets it.
constexpr uint64_t kFusedMaxM = 4096;     // at most 16 entries per thread in the last workgroup's scan
constexpr uint32_t kFusedMaxTiles = 512;  // workgroups, each with its own fence

__global__ void __launch_bounds__(256)
hist_scan_kernel(const int32_t *__restrict__ dest, uint64_t n, int32_t D, uint32_t T, uint32_t n_tiles,
                 uint32_t *__restrict__ table, uint64_t M, uint32_t *__restrict__ counter, Results to)
{
    extern __shared__ uint32_t h[];  // D + 2
    __shared__ uint32_t lds[256 / 64 + 1];
    hist_tile(dest, n, D, T, TableLayout{n_tiles, 1}, table, h);
    if (!last_workgroup(counter, n_tiles)) return;
    block_scan_inplace<256>(table, M, lds);
    finalize_body<256>([&](int32_t e) { return (uint64_t)table[(uint64_t)e * n_tiles]; }, D, n, to, lds);
}

// ------------------------------------------------------ grouped pass 1 ---
// Grouped plans: one workgroup per table column of 4 tiles, a wave per tile
// with a histogram of its own. The tiles' running sums go to pre, the sum of
// all to the table, which is 4 times smaller than with a column per tile: for
// 64 destinations up to 1M slots then fit scan_one_kernel (a round of 1M slots:
// histogram and scan 10 us for 18 in four launches). Wider groups are slower:
// queues hold long runs of one destination, whose LDS adds are serial, and 16
// tiles in one workgroup took 20 to 50 us.
constexpr uint32_t kGroupBits = 2, kGroupTiles = 1u << kGroupBits;

__global__ void __launch_bounds__(64 * kGroupTiles)
hist_group_kernel(const int32_t *__restrict__ dest, uint64_t n, int32_t D, uint32_t T, uint32_t n_tiles,
                  TableLayout layout, uint32_t *__restrict__ table, uint16_t *__restrict__ pre)
{
    extern __shared__ uint32_t h[];  // [kGroupTiles][D + 2]
    const uint32_t rows = (uint32_t)D + 2u, w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (uint32_t e = threadIdx.x; e < kGroupTiles * rows; e += blockDim.x) h[e] = 0;
    __syncthreads();
    const uint32_t first = blockIdx.x * kGroupTiles;
    uint32_t *mine = h + w * rows;
    const uint64_t start = min((uint64_t)(first + w) * T, n), end = min(start + T, n);
    // T is a multiple of 1024 and dest is 16-byte aligned: whole int4 groups,
    // four loads in flight
    uint64_t i = start + 4 * lane;
    for (; i + 768 + 4 <= end; i += 1024) {
        uint4 d4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) d4[u] = load_nt4(dest + i + 256 * u);
#pragma unroll
        for (int u = 0; u < 4; ++u) add_four(mine, d4[u], D);
    }
    for (; i < end; i += 256)
        for (uint64_t j = i; j < min(i + 4, end); ++j) atomicAdd(&mine[bucket_of(dest[j], D)], 1u);
    __syncthreads();
    for (uint32_t e = threadIdx.x; e < rows; e += blockDim.x) {
        uint32_t run = 0;
#pragma unroll
        for (uint32_t q = 0; q < kGroupTiles; ++q) {
            if (e < (uint32_t)D && first + q < n_tiles) pre[(uint64_t)(first + q) * (uint32_t)D + e] = (uint16_t)run;
            run += h[q * rows + e];
        }
        table[layout.at(e, blockIdx.x)] = run;
    }
}

// ---------------------------------------------------------------- pass 3 ---
// Output slot of a tile's first item bound for e, from the scanned table and,
// where a column stands for several tiles, the tile's prefix inside it. With
// self set, the scatter's workgroups find it themselves (self_base), from the
// unscanned table, column by column (kSumTable), or from the destinations
// (kCountSlots); workgroup 0 then has no tile and writes the results
// (self_results).
enum { kScanned, kGrouped, kSelf };  // which of these, an instance of each kernel for each
struct RunBases {
    const uint32_t *__restrict__ table;
    const uint16_t *__restrict__ pre;
    uint32_t n_cols, group_bits, self;
    __device__ uint32_t in_group(uint32_t tile, int32_t e, int32_t D) const
    {
        return group_bits ? pre[(uint64_t)tile * (uint32_t)D + (uint32_t)e] : 0u;
    }
    template <int KIND>
    __device__ uint32_t at(uint32_t tile, int32_t e, int32_t D) const
    {
        if constexpr (KIND == kScanned) return table[(uint64_t)e * n_cols + tile];
        return table[(uint64_t)e * n_cols + (tile >> group_bits)] + in_group(tile, e, D);
    }
};

// Sums of the first `rows` counts over all columns and over those before col,
// for row threadIdx.x, by a workgroup of NT threads: up to kSumParts threads
// share a row, 16 loads in flight each. scratch: 2 NT words.
constexpr uint32_t kSumParts = 16;
constexpr int kSelfD = 128;                                  // destinations at most
constexpr size_t kSelfLds = (2 * 256 + kSelfD + 2 + 8) * 4;  // bytes of LDS for 256 threads

template <int NT>
__device__ inline void sum_columns(const RunBases &b, uint32_t col, uint32_t rows, uint32_t stride, uint32_t *scratch,
                                   uint32_t &all, uint32_t &before)
{
    uint32_t lg = 0;
    while ((1u << lg) < rows) ++lg;
    const uint32_t parts = min((uint32_t)NT >> lg, kSumParts), e = threadIdx.x & ((1u << lg) - 1), part = threadIdx.x >> lg;
    all = before = 0;
    if (e < rows && part < parts) {
        for (uint32_t c0 = part; c0 < b.n_cols; c0 += 16 * parts) {
            uint32_t v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const uint32_t c = c0 + u * parts;
                v[u] = c < b.n_cols ? b.table[(uint64_t)c * stride + e] : 0u;
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                all += v[u];
                before += c0 + u * parts < col ? v[u] : 0u;
            }
        }
    }
    scratch[threadIdx.x] = all;
    scratch[NT + threadIdx.x] = before;
    __syncthreads();
    if (threadIdx.x < rows)
        for (uint32_t q = 1; q < parts; ++q) {
            all += scratch[(q << lg) + threadIdx.x];
            before += scratch[NT + (q << lg) + threadIdx.x];
        }
    __syncthreads();
}

// The same from the destinations of all n slots, of which those before `mid` (a
// multiple of 4) count as before.
template <int NT>
__device__ inline void count_slots(const int32_t *__restrict__ dest, uint64_t n, uint64_t mid, int32_t D,
                                   uint32_t *scratch, uint32_t &all, uint32_t &before)
{
    const uint32_t rows = (uint32_t)D + 2u;
    uint32_t *h0 = scratch, *h1 = scratch + rows;
    for (uint32_t e = threadIdx.x; e < 2 * rows; e += NT) scratch[e] = 0;
    __syncthreads();
    constexpr int kU = 4;
    for (uint64_t i0 = 4ull * threadIdx.x; i0 < n; i0 += kU * 4ull * NT) {
        uint4 d[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint64_t i = i0 + u * 4ull * NT;
            d[u] = i + 4 <= n ? *reinterpret_cast<const uint4 *>(dest + i) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint64_t i = i0 + u * 4ull * NT;
            uint32_t *h = i < mid ? h0 : h1;
            if (i + 4 <= n) {
                add_four(h, d[u], D);
            } else {
                for (uint64_t j = i; j < n; ++j) atomicAdd(&h[bucket_of(dest[j], D)], 1u);
            }
        }
    }
    __syncthreads();
    before = threadIdx.x < rows ? h0[threadIdx.x] : 0u;
    all = threadIdx.x < rows ? before + h1[threadIdx.x] : 0u;
    __syncthreads();
}

enum : uint32_t { kSumTable = 1, kCountSlots = 2 };

// RunBases::at(tile, e) of destination e = threadIdx.x, for tiles of T slots.
// scratch is free again on return.
template <int NT>
__device__ inline uint32_t self_base(const RunBases &b, const int32_t *__restrict__ dest, uint64_t n, uint32_t tile,
                                     uint32_t T, int32_t D, uint32_t *scratch)
{
    static_assert(NT >= kSelfD + 2, "a thread per row");
    uint32_t all, before, total;
    if (b.self == kCountSlots)
        count_slots<NT>(dest, n, (uint64_t)tile * T, D, scratch, all, before);
    else
        sum_columns<NT>(b, tile >> b.group_bits, (uint32_t)D, (uint32_t)D + 2u, scratch, all, before);
    const bool own = (int32_t)threadIdx.x < D;
    const uint32_t start = block_excl_scan<NT>(own ? all : 0u, scratch, &total);  // ends with a barrier
    return own ? start + before + b.in_group(tile, (int32_t)threadIdx.x, D) : 0u;
}

// Offsets and summary.
template <int NT>
__device__ inline void self_results(const RunBases &b, const int32_t *__restrict__ dest, int32_t D, uint64_t n,
                                    const Results &to, uint32_t *scratch)
{
    const uint32_t rows = (uint32_t)D + 2u;
    uint32_t all, before, total;
    if (b.self == kCountSlots)
        count_slots<NT>(dest, n, 0, D, scratch, all, before);
    else
        sum_columns<NT>(b, 0, rows, rows, scratch, all, before);
    uint32_t *starts = scratch + 2 * NT;
    const uint32_t start = block_excl_scan<NT>(threadIdx.x < rows ? all : 0u, scratch, &total);
    if (threadIdx.x < rows) starts[threadIdx.x] = start;
    __syncthreads();
    finalize_body<NT>([&](int32_t e) { return (uint64_t)starts[e]; }, D, n, to, scratch);
}

template <int NW>
__device__ inline void copy_item(const uint32_t *__restrict__ src, uint32_t *__restrict__ dst)
{
    if constexpr (NW % 4 == 0) {
        const uint4 *s = reinterpret_cast<const uint4 *>(src);
        uint4 *d = reinterpret_cast<uint4 *>(dst);
#pragma unroll
        for (int k = 0; k < NW / 4; ++k) d[k] = s[k];
    } else if constexpr (NW % 2 == 0) {
        const uint2 *s = reinterpret_cast<const uint2 *>(src);
        uint2 *d = reinterpret_cast<uint2 *>(dst);
#pragma unroll
        for (int k = 0; k < NW / 2; ++k) d[k] = s[k];
    } else {
#pragma unroll
        for (int k = 0; k < NW; ++k) dst[k] = src[k];
    }
}

// KIND: where the run bases come from. In one instance the three cost the
// plain table's splits 4% (1.67 M x 12-byte items, 45 destinations: 44.4 us,
// 46.2 with them).
template <int NW, int KIND>
__global__ void __launch_bounds__(256)
scatter_kernel(const uint32_t *__restrict__ items, const int32_t *__restrict__ dest, uint64_t n,
               int32_t D, int nbits, uint32_t T, RunBases bases, uint32_t *__restrict__ out, uint32_t nw_runtime,
               Results results)
{
    extern __shared__ uint32_t cnt[];  // [4][D]
    const uint32_t nw = NW > 0 ? (uint32_t)NW : nw_runtime;
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    uint32_t tile = blockIdx.x, own_base = 0;
    if constexpr (KIND == kSelf) {
        if (tile == 0) {
            self_results<256>(bases, dest, D, n, results, cnt);
            return;
        }
        --tile;
        own_base = self_base<256>(bases, dest, n, tile, T, D, cnt);
    }
    const uint64_t start = (uint64_t)tile * T;
    const uint64_t end = min(start + T, n);
    const uint64_t q = T / 4;
    const uint64_t wstart = min(start + w * q, end), wend = min(wstart + q, end);
    uint32_t *mycnt = cnt + (uint64_t)w * D;

    for (uint32_t e = tid; e < 4u * (uint32_t)D; e += 256) cnt[e] = 0;
    __syncthreads();
    for (uint64_t i = wstart + lane; i < wend; i += 64) {
        const int32_t d = dest[i];
        if (d >= 0 && d < D) atomicAdd(&mycnt[d], 1u);
    }
    __syncthreads();
    for (int32_t e = tid; e < D; e += 256) {
        uint32_t run = KIND == kSelf ? own_base : bases.at<KIND>(tile, e, D);  // kSelf: D <= 128, so e is tid
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) {
            const uint32_t c = cnt[ww * D + e];
            cnt[ww * D + e] = run;
            run += c;
        }
    }
    __syncthreads();
    const uint64_t lt = (1ull << lane) - 1ull;
    for (uint64_t b = wstart; b < wend; b += 64) {
        const uint64_t i = b + lane;
        const bool in = i < wend;
        const int32_t d = in ? dest[i] : RAFI_DONE;
        const bool ok = in && d >= 0 && d < D;
        const uint64_t peers = match_peers((uint32_t)d, ok, nbits);
        uint32_t pos = 0;
        if (ok) pos = mycnt[d] + (uint32_t)__popcll(peers & lt);
        __builtin_amdgcn_wave_barrier();
        if (ok && (peers & lt) == 0ull) mycnt[d] = pos + (uint32_t)__popcll(peers);
        // positions of kept items are < n by construction; the guard keeps a
        // corrupted table from ever writing outside the output buffer
        if (ok && pos < n) {
            const uint32_t *src = items + i * nw;
            uint32_t *dst = out + (uint64_t)pos * nw;
            if constexpr (NW > 0) {
                copy_item<NW>(src, dst);
            } else {
                for (uint32_t k = 0; k < nw; ++k) dst[k] = src[k];
            }
        }
    }
}

// ------------------------------------------------------- pass 3, staged ---
template <int NW, int R, int W, int OCC, bool DB, int KIND>
__global__ void __launch_bounds__(64 * W, OCC)
scatter_staged_kernel(const uint32_t *__restrict__ items, const int32_t *__restrict__ dest, uint64_t n,
                      int32_t D, int nbits, uint32_t T, RunBases bases, uint32_t *__restrict__ out, Results results)
{
    extern __shared__ __align__(16) uint32_t lds[];
    uint32_t tile = blockIdx.x, own_base = 0;
    if constexpr (KIND == kSelf) {
        if (tile == 0) {
            self_results<256>(bases, dest, D, n, results, lds);
            return;
        }
        --tile;
        own_base = self_base<256>(bases, dest, n, tile, T, D, lds);
    }
    const uint64_t tstart = (uint64_t)tile * T;
    const uint64_t tend = min(tstart + T, n);
    dev::staged_scatter_tile<NW, R, W, DB>(
        items, dest, tstart, tend, D, 0, nbits,
        [&](int32_t e) { return KIND == kSelf ? own_base : bases.at<KIND>(tile, e, D); }, out, n, lds);
}

// One (rounds, waves, workgroups per CU) shape of the staged scatter; it is
// launched only if its LDS fits that many workgroups per CU.
template <int NW, int R, int W, int BPC, bool DB = false>
bool try_staged(const SplitPlan &p, const uint32_t *items, const int32_t *dest, const RunBases &bases,
                uint32_t *out, hipStream_t s, const Results &results)
{
    const size_t lds = dev::staged_lds_bytes<NW, R, W>(p.D) + 64;
    if (p.D > dev::kStagedMaxD || lds * BPC > dev::kStagedLdsPerCu) return false;
    int nbits = 1;
    while ((1 << nbits) < p.D) ++nbits;
    constexpr int OCC = (W * BPC + 3) / 4;  // waves per SIMD
    if (p.self || p.group_bits) {  // plans for the automatic shapes
        if constexpr (W == 4 && !DB) {
            if (p.self) {
                if (lds < kSelfLds) return false;
                hipLaunchKernelGGL((scatter_staged_kernel<NW, R, W, OCC, false, kSelf>), dim3(p.n_tiles + 1),
                                   dim3(64 * W), lds, s, items, dest, p.n, p.D, nbits, p.tile, bases, out, results);
            } else {
                hipLaunchKernelGGL((scatter_staged_kernel<NW, R, W, OCC, false, kGrouped>), dim3(p.n_tiles),
                                   dim3(64 * W), lds, s, items, dest, p.n, p.D, nbits, p.tile, bases, out, results);
            }
            return true;
        }
        return false;
    }
    hipLaunchKernelGGL((scatter_staged_kernel<NW, R, W, OCC, DB, kScanned>), dim3(p.n_tiles), dim3(64 * W), lds, s,
                       items, dest, p.n, p.D, nbits, p.tile, bases, out, results);
    return true;
}

template <int NW, int R, int W, int OCC>
__global__ void __launch_bounds__(64 * W, OCC)
scatter_gather_kernel(const uint32_t *__restrict__ items, const int32_t *__restrict__ dest, uint64_t n,
                      int32_t D, int nbits, uint32_t T, uint32_t n_tiles, const uint32_t *__restrict__ table,
                      uint32_t *__restrict__ out)
{
    extern __shared__ __align__(16) uint32_t lds[];
    const uint64_t tstart = (uint64_t)blockIdx.x * T;
    const uint64_t tend = min(tstart + T, n);
    const uint32_t tile = blockIdx.x;
    dev::gather_scatter_tile<NW, R, W>(
        items, dest, tstart, tend, D, 0, nbits,
        [&](int32_t e) { return table[(uint64_t)e * n_tiles + tile]; }, out, n, lds);
}

template <int NW, int R, int W, int BPC>
bool try_gather(const SplitPlan &p, const uint32_t *items, const int32_t *dest, const uint32_t *table,
                uint32_t *out, hipStream_t s)
{
    const size_t lds = dev::gather_lds_bytes<R, W>(p.D) + 64;
    if (p.D > dev::kStagedMaxD || lds * BPC > dev::kStagedLdsPerCu) return false;
    int nbits = 1;
    while ((1 << nbits) < p.D) ++nbits;
    constexpr int OCC = (W * BPC + 3) / 4;
    hipLaunchKernelGGL((scatter_gather_kernel<NW, R, W, OCC>), dim3(p.n_tiles), dim3(64 * W), lds, s, items, dest,
                       p.n, p.D, nbits, p.tile, p.n_tiles, table, out);
    return true;
}

template <int NW, int R, int W, bool DB>
__global__ void __launch_bounds__(64 * W, (W + 3) / 4)
scatter_wide_kernel(const uint32_t *__restrict__ items, const int32_t *__restrict__ dest, uint64_t n,
                    int32_t D, int nbits, uint32_t T, uint32_t n_tiles, const uint32_t *__restrict__ table,
                    uint32_t *__restrict__ out, uint32_t *__restrict__ dummy)
{
    extern __shared__ __align__(16) uint32_t lds[];
    const uint64_t tstart = (uint64_t)blockIdx.x * T;
    const uint64_t tend = min(tstart + T, n);
    const uint32_t tile = blockIdx.x;
    dev::wide_scatter_tile<NW, R, W, DB>(
        items, dest, tstart, tend, D, 0, nbits,
        [&](int32_t e) { return table[(uint64_t)e * n_tiles + tile]; }, out, n, dummy, lds);
}

// The wide shape: one workgroup per CU with a chunk as large as LDS allows.
template <int NW, int R, int W, bool DB>
bool try_wide(const SplitPlan &p, const uint32_t *items, const int32_t *dest, const uint32_t *table,
              uint32_t *out, uint32_t *dummy, hipStream_t s)
{
    const size_t lds = dev::wide_lds_bytes_c<NW, R, W>(p.D) + 64;
    if (p.D > dev::kStagedMaxD || lds > dev::kStagedLdsPerCu) return false;
    int nbits = 1;
    while ((1 << nbits) < p.D) ++nbits;
    hipLaunchKernelGGL((scatter_wide_kernel<NW, R, W, DB>), dim3(p.n_tiles), dim3(64 * W), lds, s, items, dest,
                       p.n, p.D, nbits, p.tile, p.n_tiles, table, out, dummy);
    return true;
}

// The line-aligned shape: one workgroup per CU, each over a group of
// consecutive histogram tiles, so that only the two ends of a destination's
// run per group are partial lines.
template <int NW, int R, int W, int PMAX, bool DB>
__global__ void __launch_bounds__(64 * W)
scatter_line_kernel(const uint32_t *__restrict__ items, const int32_t *__restrict__ dest, uint64_t n,
                    int32_t D, int nbits, uint32_t T, uint32_t n_tiles, uint32_t group,
                    const uint32_t *__restrict__ table, uint32_t *__restrict__ out)
{
    extern __shared__ __align__(16) uint32_t lds[];
    const uint32_t tile = blockIdx.x * group;
    const uint64_t tstart = (uint64_t)tile * T;
    const uint64_t tend = min(tstart + (uint64_t)group * T, n);
    dev::line_scatter_tile<NW, R, W, PMAX, DB>(
        items, dest, tstart, tend, D, nbits,
        [&](int32_t e) { return table[(uint64_t)e * n_tiles + tile]; }, out, n, lds);
}

// The wide shape with raw staging (item sizes that are not a multiple of 16
// bytes): one workgroup per CU, the chunk's bytes in LDS in load order.
template <int NW, int R, int W, int KIND, bool TAIL>
__global__ void __launch_bounds__(64 * W, (W + 3) / 4)
scatter_wide_raw_kernel(const uint32_t *__restrict__ items, const int32_t *__restrict__ dest, uint64_t n,
                        uint64_t words, int32_t D, int nbits, uint32_t T, RunBases bases,
                        uint32_t *__restrict__ out, uint32_t *__restrict__ dummy)
{
    extern __shared__ __align__(16) uint32_t lds[];
    const uint64_t tstart = (uint64_t)blockIdx.x * T;
    const uint64_t tend = min(tstart + T, n);
    const uint32_t tile = blockIdx.x;
    dev::wide_raw_scatter_tile<NW, R, W, TAIL>(
        items, dest, tstart, tend, words, D, nbits, [&](int32_t e) { return bases.at<KIND>(tile, e, D); }, out, n,
        dummy, lds);
}

template <int NW, int R, int W>
bool try_wide_raw(const SplitPlan &p, const uint32_t *items, const int32_t *dest, const RunBases &bases,
                  uint32_t *out, uint32_t *dummy, hipStream_t s)
{
    const size_t lds = dev::wide_raw_lds_bytes_c<NW, R, W>(p.D) + 64;
    if (p.D > dev::kStagedMaxD || lds > dev::kStagedLdsPerCu) return false;
    const uint64_t words = p.n * (uint64_t)NW;
    if (words < 4) return false;
    int nbits = 1;
    while ((1 << nbits) < p.D) ++nbits;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(p.n_tiles), dim3(64 * W), lds, s, items, dest, p.n, words, p.D, nbits, p.tile,
                           bases, out, dummy);
    };
    const bool tail = words % 4 != 0;
    if (p.group_bits && tail) launch(scatter_wide_raw_kernel<NW, R, W, kGrouped, true>);
    else if (p.group_bits) launch(scatter_wide_raw_kernel<NW, R, W, kGrouped, false>);
    else if (tail) launch(scatter_wide_raw_kernel<NW, R, W, kScanned, true>);
    else launch(scatter_wide_raw_kernel<NW, R, W, kScanned, false>);
    return true;
}

// The raw shape over a lockstep schedule: kLockXcds * kLockTile persistent
// workgroups, one per CU. The dispatcher deals workgroups to the XCDs in
// turn, so workgroup b runs on XCD b % 8 as its (b / 8)-th. At step j the 32
// workgroups of XCD x take the 32 chunks of tile 8 j + x: the line a
// destination's runs in two neighbouring chunks share is then written twice
// into one L2 within the same step and leaves it whole, where chunks far
// apart in time would each send a partial line to HBM. Every workgroup loads
// its next chunk (and that chunk's run bases) while it writes the current one.
template <int NW, int R, int W, bool TAIL>
__global__ void __launch_bounds__(64 * W, (W + 3) / 4)
scatter_lock_raw_kernel(const uint32_t *__restrict__ items, const int32_t *__restrict__ dest, uint64_t n,
                        uint64_t words, int32_t D, int nbits, uint32_t n_tiles, uint32_t n_chunks,
                        const uint32_t *__restrict__ table, const uint16_t *__restrict__ pre,
                        uint32_t *__restrict__ out, uint32_t *__restrict__ dummy)
{
    static_assert(W * 64 * R == (int)kLockChunk, "a chunk of the schedule is one chunk of the kernel");
    extern __shared__ __align__(16) uint32_t lds[];
    const uint32_t x = blockIdx.x % kLockXcds, k = blockIdx.x / kLockXcds;
    const dev::LockChunks<kLockChunk, kLockTile> sched{n, x * kLockTile + k, kLockXcds * kLockTile, n_chunks,
                                                       n_tiles, D, table, pre};
    dev::wide_raw_scatter<NW, R, W, TAIL>(items, dest, words, D, nbits, sched, out, n, dummy, lds);
}

template <int NW>
bool try_lock_raw(const SplitPlan &p, const uint32_t *items, const int32_t *dest, const uint32_t *table,
                  const uint16_t *pre, uint32_t *out, uint32_t *dummy, hipStream_t s)
{
    constexpr int R = 4, W = 8;
    const size_t lds = dev::wide_raw_lds_bytes_c<NW, R, W>(p.D) + 64;
    if (p.lock != kLockTile || p.D > dev::kStagedMaxD || lds > dev::kStagedLdsPerCu) return false;
    const uint64_t words = p.n * (uint64_t)NW;  // n >= kLockMinN: at least 4
    int nbits = 1;
    while ((1 << nbits) < p.D) ++nbits;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(kLockXcds * kLockTile), dim3(64 * W), lds, s, items, dest, p.n, words, p.D,
                           nbits, p.n_tiles, p.n_chunks, table, pre, out, dummy);
    };
    if (words % 4 != 0) launch(scatter_lock_raw_kernel<NW, R, W, true>);
    else launch(scatter_lock_raw_kernel<NW, R, W, false>);
    return true;
}

int g_cus = 0;

int cu_count()
{
    if (g_cus == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 1)
            v = 256;
        g_cus = v;
    }
    return g_cus;
}

// Whether one workgroup per CU covers at least two histogram tiles and
// 16384 slots: then the partial lines at the ends of each workgroup's runs
// are few and the line-aligned shape pays.
bool line_spans_tiles(const SplitPlan &p)
{
    const uint32_t cus = (uint32_t)cu_count();
    const uint64_t group = (p.n_tiles + cus - 1) / cus;
    return p.n_tiles >= 2u * cus && group * p.tile >= 16384;
}

template <int NW, int R, int W, int PMAX, bool DB>
bool try_line(const SplitPlan &p, const uint32_t *items, const int32_t *dest, const uint32_t *table,
              uint32_t *out, hipStream_t s)
{
    const size_t lds = dev::line_lds_bytes_c<NW, R, W, PMAX>(p.D) + 64;
    if (p.D > dev::kStagedMaxD || lds > dev::kStagedLdsPerCu) return false;
    if ((reinterpret_cast<uintptr_t>(out) & 127) != 0) return false;
    if (p.n * (uint64_t)p.S > 0xfffffff0ull) return false;  // 32-bit buffer offsets
    const uint32_t cus = (uint32_t)cu_count();
    const uint32_t group = (p.n_tiles + cus - 1) / cus;
    const uint32_t grid = (p.n_tiles + group - 1) / group;
    int nbits = 1;
    while ((1 << nbits) < p.D) ++nbits;
    hipLaunchKernelGGL((scatter_line_kernel<NW, R, W, PMAX, DB>), dim3(grid), dim3(64 * W), lds, s, items, dest,
                       p.n, p.D, nbits, p.tile, p.n_tiles, group, table, out);
    return true;
}

// Process-wide choice among the scatter shapes (0 = automatic).
int g_split_variant = 0;

template <int NW>
bool launch_staged(const SplitPlan &p, const uint32_t *items, const int32_t *dest, const RunBases &bases,
                   uint32_t *out, uint32_t *dummy, hipStream_t s, const Results &results)
{
    const uint32_t *table = bases.table;
    // a plan with grouped tiles or an unscanned table (made for the automatic
    // choice) takes only shapes that read their run bases through `bases`
    int v = p.group_bits || p.self ? 0 : g_split_variant;
    if constexpr (NW >= 11) {
        // automatic: items of 44 bytes and more, few destinations and at most
        // 64 MiB: the plain per-thread scatter (each wave's run of a
        // destination is already long; the staged shapes' ranking costs
        // more than it saves there, 5-15% at 1M slots)
        if (v == 0 && p.D <= 128 && p.n * (uint64_t)p.S <= (1ull << 26) && !p.lock) return false;
    }
    if constexpr (NW % 4 != 0 && NW >= 3 && NW <= 15) {
        // large splits: the lockstep schedule (its plan has the chunk prefixes)
        if ((v == 0 || v == 17) && p.lock && try_lock_raw<NW>(p, items, dest, table, bases.pre, out, dummy, s))
            return true;
    }
    if (v == 17) v = 0;  // no lockstep plan for this split: automatic
    if constexpr (NW % 4 != 0 && NW >= 3 && NW <= 15) {
        // item sizes that are not a multiple of 16 bytes: raw staging, one
        // workgroup per CU (automatic when a tile fills a 2048-slot chunk)
        if ((v == 16 || (v == 0 && p.tile >= 8 * 64 * 4 && !p.self)) &&
            try_wide_raw<NW, 4, 8>(p, items, dest, bases, out, dummy, s))
            return true;
    }
    if (v == 16) v = 0;  // shape 16 does not take this item size: automatic
    if (v >= 14) {  // line-aligned writes, one workgroup per CU over a group of tiles
        if constexpr (NW == 8) {
            if (v == 14 && try_line<8, 4, 8, 1792, false>(p, items, dest, table, out, s)) return true;
            if (v == 15 && try_line<8, 4, 8, 1792, true>(p, items, dest, table, out, s)) return true;
        } else if constexpr (NW == 4) {
            if (v == 14 && try_line<4, 6, 8, 3840, false>(p, items, dest, table, out, s)) return true;
            if (v == 15 && try_line<4, 6, 8, 3840, true>(p, items, dest, table, out, s)) return true;
        }
        v = 0;  // item size or output alignment the line shapes do not take
    }
    if (v >= 12) {  // one workgroup per CU, 4096-slot (32-byte) or 6144-slot (16-byte) chunks
        if constexpr (NW == 8) {
            if (v == 12) return try_wide<8, 8, 8, false>(p, items, dest, table, out, dummy, s);
            if (v == 13) return try_wide<8, 8, 8, true>(p, items, dest, table, out, dummy, s);
        } else if constexpr (NW == 4) {
            if (v == 12) return try_wide<4, 12, 8, false>(p, items, dest, table, out, dummy, s);
            if (v == 13) return try_wide<4, 12, 8, true>(p, items, dest, table, out, dummy, s);
        }
        return false;
    }
    if (v == 0) {
        // automatic: few destinations and at most 256 MiB of items (every
        // context round of the workloads here): 1024-slot chunks give each
        // destination a run of about 1024 / D items per chunk, long enough
        // that the small staged shapes write whole lines without the
        // line-aligned shape's carry (16-byte items: shape 4, 32-byte items:
        // shape 2, 25-40% faster than the others there); else line-aligned
        // writes when each workgroup spans several tiles, else the wide shape
        // when a tile fills at least one of its chunks
        if (p.D <= 128 && p.n * (uint64_t)p.S <= (1ull << 28)) {
            if constexpr (NW == 8) {
                if (try_staged<8, 4, 4, 3>(p, items, dest, bases, out, s, results)) return true;
            } else if constexpr (NW == 4) {
                if (try_staged<4, 4, 4, 4>(p, items, dest, bases, out, s, results)) return true;
            }
        }
        if (line_spans_tiles(p)) {
            if constexpr (NW == 8) {
                if (try_line<8, 4, 8, 1792, false>(p, items, dest, table, out, s)) return true;
            } else if constexpr (NW == 4) {
                if (try_line<4, 6, 8, 3840, false>(p, items, dest, table, out, s)) return true;
            }
        }
        if constexpr (NW == 8) {
            if (p.tile >= 8 * 8 * 64 && try_wide<8, 8, 8, false>(p, items, dest, table, out, dummy, s)) return true;
        } else if constexpr (NW == 4) {
            if (p.tile >= 8 * 12 * 64 && try_wide<4, 12, 8, false>(p, items, dest, table, out, dummy, s)) return true;
        }
    }
    if (v >= 8) {  // shapes 1-4 with double-buffered chunk loads
        if constexpr (NW == 8) {
            if (v == 8) return try_staged<8, 7, 4, 2, true>(p, items, dest, bases, out, s, results);
            if (v == 9) return try_staged<8, 4, 4, 3, true>(p, items, dest, bases, out, s, results);
            if (v == 10) return try_staged<8, 3, 8, 2, true>(p, items, dest, bases, out, s, results);
            if (v == 11) return try_staged<8, 2, 4, 4, true>(p, items, dest, bases, out, s, results);
        } else if constexpr (NW == 4) {
            if (v == 8) return try_staged<4, 12, 4, 2, true>(p, items, dest, bases, out, s, results);
            if (v == 9) return try_staged<4, 8, 4, 3, true>(p, items, dest, bases, out, s, results);
            if (v == 10) return try_staged<4, 5, 8, 2, true>(p, items, dest, bases, out, s, results);
            if (v == 11) return try_staged<4, 4, 4, 4, true>(p, items, dest, bases, out, s, results);
        }
        return false;
    }
    if (v >= 5) {
        if (v == 5) return try_gather<NW, 16, 4, 4>(p, items, dest, table, out, s);  // 4096-slot chunks
        if (v == 6) return try_gather<NW, 32, 4, 2>(p, items, dest, table, out, s);  // 8192-slot chunks
        if (v == 7) return try_gather<NW, 16, 8, 2>(p, items, dest, table, out, s);  // 8192, 8 waves
        return false;
    }
    if constexpr (NW == 8) {
        if ((v == 0 || v == 1) && try_staged<8, 7, 4, 2>(p, items, dest, bases, out, s, results)) return true;
        if ((v == 0 || v == 2) && try_staged<8, 4, 4, 3>(p, items, dest, bases, out, s, results)) return true;
        if ((v == 0 || v == 3) && try_staged<8, 3, 8, 2>(p, items, dest, bases, out, s, results)) return true;
        if ((v == 0 || v == 4) && try_staged<8, 2, 4, 4>(p, items, dest, bases, out, s, results)) return true;
        return false;
    } else if constexpr (NW == 4) {
        if ((v == 0 || v == 1) && try_staged<4, 12, 4, 2>(p, items, dest, bases, out, s, results)) return true;
        if ((v == 0 || v == 2) && try_staged<4, 8, 4, 3>(p, items, dest, bases, out, s, results)) return true;
        if ((v == 0 || v == 3) && try_staged<4, 5, 8, 2>(p, items, dest, bases, out, s, results)) return true;
        if ((v == 0 || v == 4) && try_staged<4, 4, 4, 4>(p, items, dest, bases, out, s, results)) return true;
        return false;
    } else if constexpr (NW <= 3) {
        return try_staged<NW, 16, 4, 2>(p, items, dest, bases, out, s, results);
    } else if constexpr (56 / NW > 0) {
        return try_staged<NW, 56 / NW, 4, 2>(p, items, dest, bases, out, s, results);
    } else {
        return false;
    }
}

template <int NW>
void launch_scatter(const SplitPlan &p, const uint32_t *items, const int32_t *dest, const RunBases &bases,
                    uint32_t *out, uint32_t *dummy, hipStream_t s, const Results &results)
{
    if constexpr (NW > 0) {
        if (launch_staged<NW>(p, items, dest, bases, out, dummy, s, results)) return;
    }
    int nbits = 1;
    while ((1 << nbits) < p.D) ++nbits;
    const size_t lds = sizeof(uint32_t) * 4 * (size_t)p.D;
    if (p.self)
        hipLaunchKernelGGL((scatter_kernel<NW, kSelf>), dim3(p.n_tiles + 1), dim3(256), std::max(lds, kSelfLds), s,
                           items, dest, p.n, p.D, nbits, p.tile, bases, out, p.S / 4, results);
    else if (p.group_bits)
        hipLaunchKernelGGL((scatter_kernel<NW, kGrouped>), dim3(p.n_tiles), dim3(256), lds, s, items, dest, p.n, p.D,
                           nbits, p.tile, bases, out, p.S / 4, results);
    else
        hipLaunchKernelGGL((scatter_kernel<NW, kScanned>), dim3(p.n_tiles), dim3(256), lds, s, items, dest, p.n, p.D,
                           nbits, p.tile, bases, out, p.S / 4, results);
}

}  // namespace

namespace {
constexpr uint64_t kMaxTiles = 4096;

uint64_t min_tile(int32_t D)
{
    // at least 1024 slots and about one table byte per slot
    const uint64_t t = std::max<uint64_t>(1024, 4ull * (uint64_t)(D + 2));
    return (t + 1023) / 1024 * 1024;
}

void finish_plan(SplitPlan &p)
{
    p.rows = (uint64_t)p.D + 2;
    p.n_cols = (p.n_tiles + (1u << p.group_bits) - 1) >> p.group_bits;
    p.M = p.rows * p.n_cols;
    p.scan_blocks = (uint32_t)((p.M + kScanChunk - 1) / kScanChunk);
    // fixed head: the fused scan's finished-tile counter, then the dummy slot
    p.off_done = 0;
    p.off_dummy = 256;
    p.off_table = 512;
    p.off_part = p.off_table + (p.M * 4 + 255) / 256 * 256;
    p.bytes = p.off_part + ((uint64_t)std::max<uint32_t>(p.scan_blocks, 1) * 4 + 255) / 256 * 256;
    p.off_pre = p.bytes;
    if (p.lock) p.bytes += ((uint64_t)p.n_chunks * (uint64_t)p.D * 2 + 255) / 256 * 256;
    if (p.group_bits) {
        // 3 (D + 2) bytes of table per tile are saved, 2 D go to the prefixes.
        // The size asked for is that of a column per tile all the same: with
        // the smaller one a workspace made for n slots would not do for fewer,
        // nor for another scatter shape.
        p.bytes += ((uint64_t)p.n_tiles * (uint64_t)p.D * 2 + 255) / 256 * 256;
        SplitPlan u = p;
        u.group_bits = 0;
        finish_plan(u);
        p.bytes = std::max(p.bytes, u.bytes);
    }
}

// Items the per-thread scatter takes (launch_staged, launch_scatter), at most
// 128 destinations: sizes without staged shapes, and 44 bytes and more up to
// 64 MiB.
bool plain_scatter(const SplitPlan &p)
{
    const uint32_t nw = p.S / 4;
    if (nw >= 11) return p.n * (uint64_t)p.S <= (1ull << 26) || (nw != 11 && nw != 12 && nw != 16);
    return nw == 5 || nw == 7 || nw == 9;
}

// What a launch costs besides its work. A context's round waits on the host
// for its results: a launch more is 3 to 5 us more, and its destinations come in
// long runs. Stateless splits are queued ahead of the card, where only the
// kernels' times count. So the two differ in where fewer launches with more
// work in them pay (a round of 1 M slots of 48 bytes over 64 destinations 131 us
// in two launches, 147 in five; the split alone, queued, 42 and 37).

// The grouped histogram: where the automatic scatter shape is one of the
// small staged ones or the plain one (at most 128 destinations and 256 MiB of
// items), a tile's prefix fits 16 bits, and the one-launch scan takes the grouped
// table but not the other. Other shapes read the table by tile.
// Stateless, with over 24 destinations only up to 1280 tiles (32-byte items, 35
// destinations, 1.2 M slots 28.8 us for 29.9, 1.5 M 35.2 for 34.2), and not before
// the plain scatter, which reads the destinations twice and finds them in its
// XCD's L2 when workgroup t has read tile t before (44-byte items, 100
// destinations, 1.4 M slots: 62 us grouped, 51 not).
// Rounds also where both tables are too large by far, not where the grouped one is
// just too large as well: the wavefront a tile gets then costs what the smaller
// table saves (64 destinations, 1.4 M slots: 26 us grouped, 23 not; 4 M slots: 46
// grouped, 49 not).
bool group_eligible(const SplitPlan &p, bool round)
{
    const uint64_t rows = (uint64_t)p.D + 2, m = rows * ((p.n_tiles + kGroupTiles - 1) / kGroupTiles);
    if (g_split_variant != 0 || p.D > 128 || p.n * (uint64_t)p.S > (1ull << 28) || rows * p.n_tiles <= kOneScanMax ||
        (uint64_t)p.tile * (kGroupTiles - 1) >= 65536)
        return false;
    if (round) return m <= kOneScanMax || m > 2 * kOneScanMax;
    return m <= kOneScanMax && !plain_scatter(p) && (p.n_tiles <= 1280 || p.D <= 24);
}

// Whether the scatter's workgroups find their run bases and the results
// themselves. A round of few slots is a chain of launches, each some 5 us for
// little work, and the scan is one workgroup. The shapes are those of the
// grouped plans, with tiles below the raw shape's chunk.
//   up to kCountTiles tiles every workgroup counts all destinations, and the
//     split is one launch: 4 K slots 12.2 us, 15.5 with a histogram launch,
//     19.0 with histogram and scan; at 16 tiles the count costs what the
//     launch does;
//   else every workgroup sums the table's columns, in turns of 16 loads a
//     thread, each turn a trip past the L2.
// Rounds: not when the workgroups' threads make more than kSelfLoads loads one
//   after another, all workgroups together: 64 destinations, 1 M slots (60 K
//   loads) 18.4 us for 21.6 with a scan, 1.4 M slots (117 K) 26.8 for 23.2.
//   Columns stand for 4 tiles from kSelfPlain entries or 32 loads a thread on
//   (460 K slots 18 us for 24; 1 destination, 2 M slots 23.5 for 37).
// Stateless, measured over 4- to 64-byte items, 1 to 128 destinations and 9 K to
//   4 M slots, us with the sums and with a scan:
//   staged scatters: up to 7 turns where all tiles are on the card at once (24
//     bytes, 64 destinations, 492 K slots 20.2 for 21.9), up to 2 where a
//     second generation of workgroups makes them again (32 bytes, 16
//     destinations, 1 M slots 24.9 for 27.5; 64 destinations 28.1 for 25.2; 12
//     bytes, 8 destinations, 1.5 M slots 43.4 for 40.0). Columns stand for 4
//     tiles from kSelfPlain entries or 16 loads a thread on;
//   plain scatter, all of it on the card at once: up to 8 turns (44 bytes, 16
//     destinations, 1 M slots 28.5 for 32.2; 50 destinations, 830 K slots, 13
//     turns, 38.9 for 34.7). Columns stand for 4 tiles from kSelfPlain entries
//     on, up to kPlainGroupTiles tiles (see group_eligible).
constexpr uint32_t kCountTiles = 8, kPlainGroupTiles = 350, kCus = 256;
constexpr uint64_t kSelfPlain = 1ull << 13, kSelfMax = 1ull << 15, kSelfLoads = 1ull << 16;

void finish_self_plan(SplitPlan &p, bool round)
{
    if (g_split_variant != 0 || p.D > kSelfD || p.n * (uint64_t)p.S > (1ull << 28) || p.tile >= 8 * 64 * 4 ||
        p.n_tiles == 0)
        return;
    if (p.n_tiles <= kCountTiles) {
        p.self = kCountSlots;
        return;
    }
    uint32_t parts = 256;  // threads that share a row (sum_columns)
    while (parts > 1 && parts * (uint32_t)p.D > 256) parts /= 2;
    parts = std::min(parts, kSumParts);
    const bool plain = plain_scatter(p);
    bool group = p.rows * p.n_tiles > kSelfPlain;
    if (round) group = group || p.n_tiles > 32 * parts;
    else if (plain) group = group && p.n_tiles <= kPlainGroupTiles;
    else group = group || p.n_tiles > 16 * parts;
    SplitPlan c = p;
    c.group_bits = group ? kGroupBits : 0;
    finish_plan(c);
    const uint32_t loads = (c.n_cols + parts - 1) / parts, turns = (loads + 15) / 16;
    if (round) {
        if (c.M > kSelfMax || (uint64_t)c.n_tiles * loads > kSelfLoads) return;
    } else if (plain) {
        if (!group && turns > 8) return;
    } else {
        // workgroups a CU of the shapes that launch_staged takes
        const uint32_t resident = kCus * (p.S == 16 ? 4 : p.S == 32 ? 3 : 2);
        if (turns > (c.n_tiles <= resident ? 7u : c.n_tiles <= 2 * resident ? 2u : 0u)) return;
    }
    p = c;
    p.self = kSumTable;
}

// The lockstep scatter takes items that are not whole 16-byte pieces (the
// raw shape's sizes), at most the staged shapes' destination count, and
// splits of at least 2^21 slots (four chunks per workgroup) whose table the
// scan takes in one partial-sum pass.
constexpr uint64_t kLockMinN = 1ull << 21;

bool lock_eligible(uint64_t n, int32_t D, uint32_t S)
{
    const uint32_t NW = S / 4;
    const uint64_t tiles = (n + kLockTile * kLockChunk - 1) / (kLockTile * kLockChunk);
    return S % 4 == 0 && NW % 4 != 0 && NW >= 3 && NW <= 15 && D <= dev::kStagedMaxD && n >= kLockMinN &&
           ((uint64_t)D + 2) * tiles <= (uint64_t)kPartMax * kScanChunk;
}

SplitPlan lock_plan(uint64_t n, int32_t D, uint32_t S)
{
    SplitPlan p;
    p.n = n;
    p.D = D;
    p.S = S;
    p.tile = kLockTile * kLockChunk;
    p.n_tiles = (uint32_t)((n + p.tile - 1) / p.tile);
    p.lock = kLockTile;
    p.n_chunks = (uint32_t)((n + kLockChunk - 1) / kLockChunk);
    finish_plan(p);
    return p;
}
}  // namespace

int split_set_variant(int v)
{
    if (v < 0 || v > 17) return RAFI_ERR_ARG;
    g_split_variant = v;
    return RAFI_OK;
}

SplitPlan split_plan(uint64_t n, int32_t D, uint32_t S, bool allow_lock, bool round)
{
    if (allow_lock && (g_split_variant == 0 || g_split_variant == 17) && lock_eligible(n, D, S))
        return lock_plan(n, D, S);
    SplitPlan p;
    p.n = n;
    p.D = D;
    p.S = S;
    uint64_t t = std::max<uint64_t>(min_tile(D), (n + kMaxTiles - 1) / kMaxTiles);
    t = (t + 1023) / 1024 * 1024;
    p.tile = (uint32_t)t;
    p.n_tiles = (uint32_t)((n + t - 1) / t);
    if (group_eligible(p, round)) p.group_bits = kGroupBits;
    finish_plan(p);
    finish_self_plan(p, round);
    return p;
}

SplitPlan split_plan_bound(uint64_t cap, int32_t D, uint32_t S)
{
    // every n <= cap uses a tile >= min_tile(D) and at most kMaxTiles tiles
    SplitPlan p;
    p.n = cap;
    p.D = D;
    p.S = S;
    p.tile = (uint32_t)min_tile(D);
    p.n_tiles = (uint32_t)std::min<uint64_t>(kMaxTiles, (cap + p.tile - 1) / p.tile);
    finish_plan(p);
    // a lockstep plan for some n <= cap (whatever shape is selected later):
    // its workspace grows with n
    if (lock_eligible(cap, D, S)) p.bytes = std::max(p.bytes, lock_plan(cap, D, S).bytes);
    return p;
}

int split_run(const SplitPlan &p, const void *items, const int32_t *dest, void *out,
              uint64_t *offsets, uint64_t *summary, uint32_t *tile_offsets, uint32_t tile_items,
              void *workspace, hipStream_t s, const SplitEvents *ev, unsigned long long *dropped, bool fused,
              const HostOut &host)
{
    if (p.scan_blocks > (uint32_t)kPartMax) return RAFI_ERR_ARG;
    if (ev) RAFI_HIP_CHECK(hipEventRecord(ev->begin, s));
    uint32_t *table = reinterpret_cast<uint32_t *>(static_cast<char *>(workspace) + p.off_table);
    uint32_t *part = reinterpret_cast<uint32_t *>(static_cast<char *>(workspace) + p.off_part);
    uint32_t *dummy = reinterpret_cast<uint32_t *>(static_cast<char *>(workspace) + p.off_dummy);
    uint32_t *counters = reinterpret_cast<uint32_t *>(static_cast<char *>(workspace) + p.off_done);
    uint16_t *pre = reinterpret_cast<uint16_t *>(static_cast<char *>(workspace) + p.off_pre);
    const Results results{offsets, summary, tile_offsets, tile_items ? tile_items : 1u, dropped, host};
    const TableLayout layout = p.self ? TableLayout{1, (uint32_t)p.rows} : TableLayout{p.n_cols, 1};
    // The fused launch costs one device-scope fence (an L2 write-back on this
    // multi-XCD part) per workgroup: worth it only for small tables.
    if (p.n_tiles > 0 && fused && !p.lock && !p.group_bits && !p.self && p.M <= kFusedMaxM && p.n_tiles <= kFusedMaxTiles) {
        hipLaunchKernelGGL(hist_scan_kernel, dim3(p.n_tiles), dim3(256), sizeof(uint32_t) * p.rows, s, dest, p.n,
                           p.D, p.tile, p.n_tiles, table, p.M, counters, results);
        RAFI_LAUNCH_CHECK();
    } else {
        if (p.n_tiles > 0 && p.self != kCountSlots) {
            if (p.lock)
                hipLaunchKernelGGL(hist_lock_kernel, dim3(p.n_tiles), dim3(256), sizeof(uint32_t) * p.rows, s,
                                   dest, p.n, p.D, p.n_tiles, p.n_chunks, table, pre);
            else if (p.group_bits)
                hipLaunchKernelGGL(hist_group_kernel, dim3(p.n_cols), dim3(64 * kGroupTiles),
                                   sizeof(uint32_t) * kGroupTiles * p.rows, s, dest, p.n, p.D, p.tile, p.n_tiles,
                                   layout, table, pre);
            else
                hipLaunchKernelGGL(hist_kernel, dim3(p.n_tiles), dim3(256), sizeof(uint32_t) * p.rows, s,
                                   dest, p.n, p.D, p.tile, layout, table);
            RAFI_LAUNCH_CHECK();
        }
        if (p.self) {
            // the scatter scans
        } else if (p.n_tiles > 0 && p.M <= kOneScanMax) {
            hipLaunchKernelGGL(scan_one_kernel, dim3(1), dim3(1024), 0, s, table, p.M, p.n_cols, p.D, p.n, results);
            RAFI_LAUNCH_CHECK();
        } else {
            if (p.n_tiles > 0) {
                hipLaunchKernelGGL(scan_reduce_kernel, dim3(p.scan_blocks), dim3(kScanThreads), 0, s, table, p.M,
                                   part);
                if (p.scan_blocks <= kDirectMaxBlocks) {
                    hipLaunchKernelGGL(scan_apply_direct_kernel, dim3(p.scan_blocks), dim3(kScanThreads), 0, s,
                                       table, p.M, part);
                } else {
                    hipLaunchKernelGGL(scan_partials_kernel, dim3(1), dim3(kPartThreads), 0, s, part,
                                       p.scan_blocks);
                    hipLaunchKernelGGL(scan_apply_kernel, dim3(p.scan_blocks), dim3(kScanThreads), 0, s, table,
                                       p.M, part);
                }
                RAFI_LAUNCH_CHECK();
            }
            hipLaunchKernelGGL(finalize_kernel, dim3(1), dim3(1024), 0, s, table, p.n_cols, p.D, p.n, results);
            RAFI_LAUNCH_CHECK();
        }
    }
    if (ev) RAFI_HIP_CHECK(hipEventRecord(ev->before_scatter, s));
    if (p.n_tiles == 0) {
        if (ev) RAFI_HIP_CHECK(hipEventRecord(ev->end, s));
        return RAFI_OK;
    }
    const uint32_t *it = static_cast<const uint32_t *>(items);
    uint32_t *o = static_cast<uint32_t *>(out);
    const RunBases bases{table, pre, p.n_cols, p.group_bits, p.self};
    switch (p.S / 4) {
    case 1: launch_scatter<1>(p, it, dest, bases, o, dummy, s, results); break;
    case 2: launch_scatter<2>(p, it, dest, bases, o, dummy, s, results); break;
    case 3: launch_scatter<3>(p, it, dest, bases, o, dummy, s, results); break;
    case 4: launch_scatter<4>(p, it, dest, bases, o, dummy, s, results); break;
    case 6: launch_scatter<6>(p, it, dest, bases, o, dummy, s, results); break;
    case 8: launch_scatter<8>(p, it, dest, bases, o, dummy, s, results); break;
    case 10: launch_scatter<10>(p, it, dest, bases, o, dummy, s, results); break;
    case 11: launch_scatter<11>(p, it, dest, bases, o, dummy, s, results); break;
    case 12: launch_scatter<12>(p, it, dest, bases, o, dummy, s, results); break;
    case 16: launch_scatter<16>(p, it, dest, bases, o, dummy, s, results); break;
    default: launch_scatter<0>(p, it, dest, bases, o, dummy, s, results); break;
    }
    RAFI_LAUNCH_CHECK();
    if (ev) RAFI_HIP_CHECK(hipEventRecord(ev->end, s));
    return RAFI_OK;
}

}  // namespace rafi
