// Host-side definitions shared by the library's translation units.
#pragma once

#include <algorithm>
#include <new>

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <mutex>
#include <type_traits>

#include "lhs.h"
#include "lhs_device.h"

// Device counters of one BFS level.
struct LevelCounters {
    uint32_t n_next;              // append cursor of the next frontier
    uint32_t abort;               // set once n_next exceeds the level's limit
    unsigned long long edges;     // successors generated by this level
    unsigned long long deadlocks; // expanded states without successors
};

struct lhs_table {
    int device = 0;
    int ncu = 0;               // the device's CUs
    uint64_t capacity = 0;
    uint32_t W = 0;
    uint32_t lines = 0;
    uint32_t max_rounds = 0;
    uint32_t line_slots = 16;  // slots per probed line (8, 16, 32)
    uint32_t probe = 0;        // lhs_probe
    uint32_t tps_fop = 0;      // lanes cooperating on one operation (1, 4, 8,
    uint32_t tps_exp = 0;      // 16) in find-or-put / BFS; 0 = default
    bool tuned = false;        // ... come from the tuning table (tps_of_call)
    uint32_t counters = 0;     // LHS_COUNT_* requested by lhs_set_counters
    uint32_t merge = 0;        // lhs_merge mode of explorations (lhs_set_merge)
    uint32_t workers = 0;      // cap on exploration workgroups (0 = all resident)
    uint64_t seed = 0;
    uint64_t *bucket = nullptr;
    uint32_t *data = nullptr;
    lhs::DevStatus *status = nullptr;   // first member of a TableStatus
    hipStream_t last_stream = nullptr;
    // BFS buffers, allocated on first use by reach_explore and kept.
    uint32_t *frontier[2] = {nullptr, nullptr};
    LevelCounters *level = nullptr;        // + the segment cursors, 256 bytes on
    uint32_t *segs = nullptr;              //   (same allocation)
    // pinned summary of the last level (a LevelSummary): its counters, the
    // segment counts and the table's status; summary_dev is its device address
    LevelCounters *level_host = nullptr;
    uint32_t *seg_n_host = nullptr;
    lhs::DevStatus *status_host = nullptr;
    void *summary_dev = nullptr;
    // graph-driven BFS (REACH_F_GRAPH): device context, level counts and the
    // captured level graph (rebuilt when the LDS layout changes)
    void *gctx = nullptr;
    unsigned long long *glevels = nullptr;
    uint32_t glevels_cap = 0;
    hipStream_t gstream = nullptr;
    hipGraphExec_t gexec = nullptr;
    uint64_t gexec_tcap = 0;
    // predecessor records of the last BFS with REACH_F_PARENTS
    uint32_t *parent = nullptr;     // [capacity]
    uint32_t *dead_rec = nullptr;   // [1 + kDeadRecord]
    bool has_parents = false;
    // the server running a query on this table (reach_server_submit_ex),
    // from submission until the query is collected
    std::atomic<const void *> served_by{nullptr};
};

namespace lhs {

// Run an entry point's body, turning a C++ exception (an allocation that
// failed, a thread or lock that could not be had) into a status: nothing
// unwinds through the C ABI.
template <class F>
lhs_status guard(F &&f) noexcept {
    try {
        return f();
    } catch (const std::bad_alloc &) {
        return LHS_ENOMEM;
    } catch (...) {
        return LHS_EDEVICE;
    }
}

inline TableView view(const lhs_table *t) {
    TableView v;
    v.bucket = t->bucket;
    v.data = t->data;
    v.seed = t->seed;
    v.W = t->W;
    v.line_mask = t->lines - 1;
    v.max_rounds = t->max_rounds;
    v.probe = t->probe;
    v.status = t->status;
    v.parent = nullptr;
    v.dead_rec = nullptr;
    v.flags = (t->counters & LHS_COUNT_LINES ? kCountLines : 0u) |
              (t->counters & LHS_COUNT_MERGED ? kCountMerged : 0u) |
              (t->merge == LHS_MERGE_OFF ? kNoMerge : 0u) |
              (t->merge == LHS_MERGE_NARROW_TAGS ? kNarrowTags : 0u);
    return v;
}

// Defaults measured on MI355X (2^26-op stream, 2^27-state BFS): the batched
// find-or-put is fastest with 4-lane groups, the BFS expansion with one lane
// per successor and wavefront-cooperative memory accesses.
constexpr uint32_t kDefaultTpsFindOrPut = 4;
constexpr uint32_t kDefaultTpsExpand = 1;
inline uint32_t tps_find_or_put(const lhs_table *t) { return t->tps_fop ? t->tps_fop : kDefaultTpsFindOrPut; }
inline uint32_t tps_expand(const lhs_table *t) { return t->tps_exp ? t->tps_exp : kDefaultTpsExpand; }
// Workgroups of an exploration launch: the resident ones, or fewer when the
// table caps its workers (lhs_set_workers).
inline uint32_t exploration_grid(const lhs_table *t, uint64_t resident) {
    const uint64_t g = t->workers ? std::min<uint64_t>(resident, t->workers) : resident;
    return (uint32_t)std::max<uint64_t>(1, g);
}

inline bool valid_tps(uint32_t tps) { return tps == 0 || tps == 1 || tps == 4 || tps == 8 || tps == 16; }
inline bool valid_line_slots(uint32_t ls) { return ls == 8 || ls == 16 || ls == 32; }

// Kernels are instantiated per (lanes per operation G, line slots LS); these
// call f(G, LS) with both as std::integral_constant for the runtime values.
template <int V>
using IntC = std::integral_constant<int, V>;
template <uint32_t V>
using U32C = std::integral_constant<uint32_t, V>;

template <class F>
lhs_status with_line_slots(uint32_t ls, F &&f) {
    switch (ls) {
    case 8: return f(U32C<8>{});
    case 16: return f(U32C<16>{});
    case 32: return f(U32C<32>{});
    }
    return LHS_EINVAL;
}

template <class F>
lhs_status with_shape(uint32_t tps, uint32_t ls, F &&f) {
    auto per_g = [&](auto G) { return with_line_slots(ls, [&](auto L) { return f(G, L); }); };
    switch (tps) {
    case 1: return per_g(IntC<1>{});
    case 4: return per_g(IntC<4>{});
    case 8: return per_g(IntC<8>{});
    case 16: return per_g(IntC<16>{});
    }
    return LHS_EINVAL;
}

// ... and f(G, LS, R{}) with the element type R of the expansion's LDS rows:
// bytes where the models allow it and one lane runs an operation.
template <class F>
lhs_status with_tile(uint32_t tps, uint32_t ls, bool bytes, F &&f) {
    return with_shape(tps, ls, [&](auto G, auto L) {
        if constexpr (decltype(G)::value == 1)
            if (bytes)
                return f(G, L, uint8_t{});
        return f(G, L, uint32_t{});
    });
}

// Tuned table configuration for (kind, W, capacity) from the loaded tuning
// table, or the defaults; never fails.
lhs_config tuned_config(uint32_t kind, uint32_t W, uint64_t capacity);

// Reusable scratch of one device (workspace.cpp): hold `mu` while using it.
struct Workspace {
    std::mutex mu;
    void *dev = nullptr;      // device region
    size_t dev_bytes = 0;
    void *host = nullptr;     // pinned host region
    size_t host_bytes = 0;
    hipEvent_t ev[2] = {nullptr, nullptr};
};
Workspace &workspace(int device);
// Grow the regions to at least the given sizes (contents are not kept).
lhs_status ws_reserve(Workspace &w, size_t dev_bytes, size_t host_bytes);

// Byte offsets of arrays carved out of one region (256-byte aligned).
struct Carve {
    size_t off = 0;
    template <class T>
    size_t take(size_t n) {
        off = (off + 255) & ~size_t(255);
        const size_t o = off;
        off += n * sizeof(T);
        return o;
    }
};
template <class T>
inline T *at(void *base, size_t off) {
    return reinterpret_cast<T *>(static_cast<char *>(base) + off);
}

inline bool is_pow2(uint64_t x) { return x && !(x & (x - 1)); }

// ceil(2^32 / W): __umulhi(f, magic) == f / W for f < 2^13 and 2 <= W <= 32.
inline uint32_t div_magic(uint32_t W) {
    return W <= 1 ? 0u : (uint32_t)(((1ull << 32) + W - 1) / W);
}

lhs_status launch_find_or_put(lhs_table *t, const uint32_t *d_states, uint64_t n,
                              uint8_t *d_seen, uint32_t *d_index, hipStream_t s);
lhs_status launch_zero_u64(uint64_t *p, uint64_t n, hipStream_t s);
// A table's status with its striped counters added in.
DevStatus sum_status(const TableStatus &ts);
lhs_status read_status(lhs_table *t, DevStatus *out);
lhs_status alloc_table(uint64_t capacity, uint32_t state_words, const lhs_config *cfg, lhs_table **out);

}  // namespace lhs

#define LHS_HIP(call)                                   \
    do {                                                \
        if ((call) != hipSuccess)                       \
            return LHS_EDEVICE;                         \
    } while (0)
