// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <chrono>
#include <cstdint>
#include <cstdio>
#include <thread>

#include "rafi.h"

#define RAFI_HIP_CHECK(expr)                                                        \
    do {                                                                            \
        hipError_t rafi_e_ = (expr);                                                \
        if (rafi_e_ != hipSuccess) {                                                \
            std::fprintf(stderr, "librafi: %s failed: %s (%s:%d)\n", #expr,         \
                         hipGetErrorString(rafi_e_), __FILE__, __LINE__);           \
            return RAFI_ERR_HIP;                                                    \
        }                                                                           \
    } while (0)

#define RAFI_LAUNCH_CHECK()                                                         \
    do {                                                                            \
        hipError_t rafi_e_ = hipGetLastError();                                     \
        if (rafi_e_ != hipSuccess) {                                                \
            std::fprintf(stderr, "librafi: launch failed: %s (%s:%d)\n",            \
                         hipGetErrorString(rafi_e_), __FILE__, __LINE__);           \
            return RAFI_ERR_HIP;                                                    \
        }                                                                           \
    } while (0)

namespace rafi {

// ------------------------------------------------------------ split plan ---
// The forward step runs as: per-tile destination histogram -> exclusive scan
// over the (destination-major, tile-minor) count table -> stable scatter.
struct SplitPlan {
    uint64_t n = 0;          // slots
    int32_t D = 0;           // domains
    uint32_t S = 0;          // item bytes
    uint32_t tile = 0;       // slots per tile
    uint32_t n_tiles = 0;
    uint64_t rows = 0;       // D + 2 (domains, done, bad)
    uint64_t M = 0;          // rows * n_cols table entries
    uint32_t scan_blocks = 0;
    uint64_t off_table = 0, off_part = 0, off_dummy = 0, off_done = 0, bytes = 0;  // workspace layout
    // off_dummy: 16 bytes any scatter lane may overwrite; off_done: the finished-tile
    // counter of the fused histogram + scan launch (zero between launches)
    // Lockstep scatter (large splits of items that are not whole 16-byte
    // pieces): tiles of `lock` chunks of 2048 slots; the workspace at
    // off_pre holds, per chunk and destination, the items bound there in the
    // earlier chunks of the chunk's tile (u16). lock = 0: off.
    uint32_t lock = 0;
    uint32_t n_chunks = 0;
    uint64_t off_pre = 0;
    // Grouped histogram (few destinations, the context rounds' sizes): the
    // table has one column per 2^group_bits tiles, and the workspace at off_pre
    // holds, per tile and destination, the items bound there in the earlier
    // tiles of its column (u16). 0: a column per tile.
    uint32_t group_bits = 0;
    uint32_t n_cols = 0;  // table columns
    // The scatter finds its run bases and the results itself, without a scan:
    // from the unscanned table, or from the destinations without a histogram.
    // 0: off.
    uint32_t self = 0;
};

// allow_lock: the plan may use the lockstep scatter (its workspace grows by
// 2 bytes per chunk and destination). round: the plan of a context's round, whose
// host waits for its launches.
SplitPlan split_plan(uint64_t n, int32_t D, uint32_t S, bool allow_lock = true, bool round = false);
// Select the staged scatter shape (0 = automatic, 1..17 = fixed shapes).
int split_set_variant(int v);
// A plan whose workspace covers every n <= cap.
SplitPlan split_plan_bound(uint64_t cap, int32_t D, uint32_t S);

// Where a split leaves its results for the host (pinned memory), before or while
// the scatter runs: the five summary words, then `seq` (nonzero) at words[7]
// once they and, with offsets set, the D + 1 offsets are written.
struct HostOut {
    uint64_t *words = nullptr;
    uint64_t *offsets = nullptr;
    uint64_t seq = 0;
};

// Optional events recorded around the split's passes (on the split stream).
struct SplitEvents {
    hipEvent_t begin = nullptr, before_scatter = nullptr, end = nullptr;
};

// Run the split. offsets: device u64 [D+1]; summary: device u64 [4], or [5]
// with dropped: {total, done, bad, n_tiles_app, dropped}; tile_offsets
// (optional): device u32 [D+1] built for tiles of tile_items. dropped
// (optional): device counter read into summary[4] and reset. fused: allow the
// one-launch histogram + scan + finalize for small tables (the workspace's
// first 4 bytes must be zero, as the context keeps them). host (optional):
// the results for the host.
int split_run(const SplitPlan &p, const void *items, const int32_t *dest, void *out,
              uint64_t *offsets, uint64_t *summary, uint32_t *tile_offsets, uint32_t tile_items,
              void *workspace, hipStream_t stream, const SplitEvents *ev = nullptr,
              unsigned long long *dropped = nullptr, bool fused = false, const HostOut &host = HostOut());

}  // namespace rafi

// ------------------------------------------------------------- context ---
struct rafi_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    int32_t D = 0;
    uint32_t S = 0;
    uint64_t cap = 0;
    void *buf[2] = {nullptr, nullptr};
    int cur_in = 0;                     // buf[cur_in] is the input queue
    int32_t *dest = nullptr;            // [cap]
    uint64_t *offsets = nullptr;        // [D+1]
    uint32_t *tile_offsets = nullptr;   // [D+1]
    uint64_t *summary = nullptr;        // [4] device
    unsigned long long *dropped = nullptr;  // device counter
    // Persistent domain kernels: [0] next queue index to hand out, [1] waves
    // that have exited. Zero between launches: the last wave to exit resets both.
    unsigned long long *work = nullptr;
    unsigned long long *append = nullptr;  // slots taken by rafi_emit since the last rafi_open
    uint64_t *host_summary = nullptr;   // pinned [8 + D + 1]: summary words, sequence number, offsets
    uint64_t *host_summary_dev = nullptr;  // its device address
    uint64_t round_seq = 0;             // sequence number of the last enqueued round
    bool in_flight = false;             // the last step's scatter may still read the output slots
    void *ws = nullptr;
    uint64_t ws_bytes = 0;
    uint64_t n_in = 0, n_slots = 0;
    uint64_t wave_slots = 0;            // n_slots of the last rafi_begin (item ids stay below it)
    uint32_t tile_items = 256, n_tiles = 0;
    int debug = 0;
    rafi_stats_t stats{};
    // profiling: event pairs waiting to be resolved
    int prof_on = 0;
    rafi_profile prof{};
    struct Pending {
        int kind;  // 0 split (3 events), 1 domain (2 events)
        hipEvent_t e[3];
        uint64_t slots;
    };
    static constexpr int kMaxPending = 64;
    Pending pending[kMaxPending];
    int n_pending = 0;
    hipEvent_t pool[3 * kMaxPending];
    int pool_size = 0;
};

namespace rafi {
int ctx_fill_poison(rafi_ctx *ctx, uint64_t n);
// Domain-kernel timing: prof_domain_begin returns a handle (or -1 when off)
// to pass to prof_domain_end after the launch.
int prof_domain_begin(rafi_ctx *ctx);
void prof_domain_end(rafi_ctx *ctx, int h);
// Resolve pending event pairs: all of them after synchronising the context
// stream (wait), or only those already complete, in order.
int prof_resolve(rafi_ctx *ctx, bool wait);
// The two halves of rafi_round: enqueue the split of the current output slots,
// which writes its results to pinned memory (want_counts: the offsets
// too); then wait for them and take them (queue length, statistics; counts,
// optional: items per domain). The wait ends before the scatter does: what is
// enqueued next on the stream follows it. round_finish does not touch the
// output slots.
int round_enqueue(rafi_ctx *ctx, bool want_counts = false);
int round_finish(rafi_ctx *ctx, uint64_t *total, uint64_t *counts = nullptr);
// Both halves and the refill of the slots in debug mode: rafi_round without
// its synchronisation of the stream.
int round_run(rafi_ctx *ctx, uint64_t *counts, uint64_t *total);
// A word from behind what is on the stream, as the scatter of the round before,
// and the wait for it; work enqueued in between is not waited for. The two of an
// N-body seed and step cost 8 us together (3.5 K particles, 4 domains: 253 us
// without them, 261 with).
// round_settled: round_run with the queue whole on return.
int settle_enqueue(rafi_ctx *ctx);
int settle_finish(rafi_ctx *ctx);
int round_settled(rafi_ctx *ctx, uint64_t *total);

// A word of host_summary free for what a step needs on the host besides its
// rounds' results.
constexpr int kHostExtra = 6;

// Waits until a kernel on the context's stream has left a word that `arrived`
// takes at host_summary[index]. The word is polled (a copy and an event cost
// a launch, 10 us); after a second the stream is synchronised instead, which
// also reports a failed launch.
template <typename Arrived>
int wait_host_word(rafi_ctx *c, int index, Arrived arrived)
{
    auto look = [&] { return arrived(__atomic_load_n(c->host_summary + index, __ATOMIC_ACQUIRE)); };
    const auto t0 = std::chrono::steady_clock::now();
    for (uint32_t i = 1; !look(); ++i) {
        __builtin_ia32_pause();
        if (i % 256 != 0) continue;
        const auto waited = std::chrono::steady_clock::now() - t0;
        if (waited > std::chrono::seconds(1)) {
            RAFI_HIP_CHECK(hipStreamSynchronize(c->stream));
            return look() ? RAFI_OK : RAFI_ERR_HIP;
        }
        if (waited > std::chrono::microseconds(200)) std::this_thread::yield();
    }
    return RAFI_OK;
}

// The round loop with the host one step ahead of the device. After a forward
// step is enqueued, the next domain launch is enqueued at once as
// launch(bound), with bound >= the queue length that step will produce (the
// kernel reads the exact length on the device), and only then does the host
// wait for the step's total; so the device never waits for the host between
// the two. slots(n): output slots a launch over n queued items writes. The
// last launch, over an empty queue, does nothing. *rounds: forward steps;
// *forwarded: items they delivered. On an error the stream is drained: the
// results reach the host before their step's scatter is done, and the caller
// may read the queue on another stream. At the end the queue is empty, and
// what is left of the last step and launch writes nothing; a stream that the
// context is moved to waits for it (rafi_set_stream), the same one is ordered
// behind it (drained here, the card idles for 20 to 35 us: a render of 64^3,
// 128 x 128 rays 93 -> 116 us).
template <typename Launch, typename Slots>
int run_rounds(rafi_ctx *c, int32_t max_rounds, int32_t *rounds, uint64_t *forwarded, Launch launch, Slots slots)
{
    int32_t r = 0;
    uint64_t fwd = 0;
    int rc = round_enqueue(c);
    uint64_t bound = c->n_slots;
    while (rc == RAFI_OK) {
        ++r;
        const bool more = r < max_rounds;
        const int lrc = more ? launch(bound) : RAFI_OK;
        uint64_t total = 0;
        rc = round_finish(c, &total);
        fwd += total;
        if (rc == RAFI_OK) rc = lrc;
        if (rc != RAFI_OK || total == 0) break;
        if (!more) {
            rc = RAFI_ERR_MAX_ROUNDS;
            break;
        }
        c->n_slots = slots(total);
        bound = c->n_slots;
        rc = round_enqueue(c);
    }
    if (rounds) *rounds = r;
    if (forwarded) *forwarded = fwd;
    c->in_flight = rc == RAFI_OK;
    if (rc != RAFI_OK) (void)hipStreamSynchronize(c->stream);
    return rc;
}
}
