// The persistent level driver of the batch (csrc/batch.hip), of the levels of
// a single-model BFS that are too small to fill the GPU, and of the server
// (csrc/serve.hip): one launch of resident workgroups runs every level of
// every model, each model at its own pace, without grid-wide barriers.
//
// Work is handed out by tickets, one 64-bit word per model: the current
// level's shape (tiles, rows per tile, frontier buffer) in the upper half,
// the next tile in the lower.  A workgroup takes a tile with one atomic add
// and knows from the returned word what to expand; a word whose next tile is
// not below its tiles has no work.  The workgroup that completes a level's
// last tile finalises the level (cap rollback, level count, frontier swap)
// and writes the next level's ticket.  Everything one workgroup hands to
// another goes through agent-scope (coherent) accesses, completed (vmcnt(0))
// before the ticket or counter that announces it.
//
// A workgroup takes its next tile from a model picked at random among those
// that have tiles, not in the order the levels were finished: a batch's
// makespan is its deepest models' chains of narrow levels, and in a common
// FIFO each of those levels waited behind all tiles of the wide models (80 to
// 420 us a level, 5.8 of 10.2 ms).
//
// What bounds a narrow level is its chain of memory round trips (0.7 us
// each).  So the finaliser keeps tile 0 of the next level for itself, and a
// level of at most kSoloStates states never leaves its workgroup: its
// frontier and counts stay in LDS (solo levels), which leaves the trips of
// the expansion itself (row, slot line, claim, row write).  A one-state level
// takes 7.8 us so and took 15 us through the queue; a level of some hundred
// states handed out in tiles takes 19 us.  Against the queue: 64-model batch
// 8.8 -> 8.2 ms, 5.7k-state search 535 -> 465 us, 10^6-state search (whose
// last narrow levels no longer go through the host) 2.44 -> 2.06 ms.
//
// The workgroups need not all be resident at once: a workgroup waits only
// for tickets, which finalisers write without waiting for anyone, so one
// that starts late takes a tile or finds the launch finished.  Every wait is
// bounded; on timeout the error flag is set and all workgroups leave.
#pragma once

#include "expand_device.h"
#include "internal.h"
#include "reach_internal.h"

namespace lhs {

// An idle workgroup's wait is bounded by the time since the launch last gave a
// sign of progress (BoardCtl::beat: a level handed out, 32 levels run alone, a
// model finished), on the GPU's constant 100 MHz clock.  Not by its polls: a
// poll takes 1 to 40 us, by the naps after it and by how many poll.  The
// longest stretch without a beat is that of an operation on a full table,
// which probes every line before it reports EFULL: 1.4 us a line, 2.9 s at
// 2^24 slots in lines of 8 (5.5 us a line if all 2^18 resident lanes do so, at
// the 48 G random lines a second that this GPU reads).
// So the bound is 30 s and 8 us for each line of the launch's largest table: a
// model that overflows ends with EFULL, and a chain of any number of levels
// ends.
constexpr uint64_t kWallKHz = 100000;
__host__ __device__ inline uint32_t stall_ms(uint64_t lines) { return (uint32_t)(30000 + lines / 125); }
constexpr uint32_t kBeatPolls = 16;   // polls between an idle workgroup's looks at the beat

// Per-model constants (written by the host before the launch, or before the
// server admits the model).
struct ModelState {
    TableView t;
    ModelView m;
    uint32_t *fr[2];
    unsigned long long *levels;   // [max_levels] level counts (coherent stores)
    unsigned long long *host_levels;   // server: where they go at the end (pinned)
    unsigned long long cap;
    uint32_t max_levels;
    uint32_t handover;            // stop after a level of more states (0 = never)
    uint32_t words;               // some word of its states may not fit a byte
    uint32_t pad;
};

// Shared by all workgroups of a launch; idle ones poll its first line.
struct alignas(128) BoardCtl {
    uint32_t remaining;   // unfinished models
    uint32_t error;
    uint32_t idle;        // workgroups without a tile
    uint32_t slots;       // server: tickets in use are below this
    alignas(128) uint32_t beat;   // signs of progress
    uint32_t stall_ms;            // an idle workgroup's wait without one
};

// One model's level and progress: written by whichever workgroup finalises a
// level; and the counters its tiles update, on a line of their own.
struct BoardModel {
    alignas(128) uint32_t n_front;   // states of the current level
    uint32_t limit;                  // new states it may add (the cap)
    uint32_t cur;                    // its frontier buffer
    uint32_t n_levels;
    unsigned long long total, edges, deadlocks;
    uint32_t done, capped, overflow, handed;   // handed: stopped after a level above handover
    uint32_t status_error;           // the table's sticky error and waits at the end
    uint32_t pad;
    unsigned long long wait_hits;
    unsigned long long key;          // server: the query's ModelView key
    alignas(128) LevelCounters lc;
    uint32_t tiles_done;
};

// Tickets.
constexpr uint32_t kTicketTiles = (1u << 26) - 1;
__host__ __device__ inline unsigned long long make_ticket(uint32_t tiles, uint32_t cur, uint32_t rows, uint32_t next) {
    const uint32_t shape = tiles | cur << 26 | (rows == 32 ? 0u : rows == 64 ? 1u : rows == 128 ? 2u : 3u) << 27;
    return (unsigned long long)shape << 32 | next;
}
__device__ __forceinline__ uint32_t ticket_tiles(unsigned long long t) { return (uint32_t)(t >> 32) & kTicketTiles; }
__device__ __forceinline__ uint32_t ticket_cur(unsigned long long t) { return (uint32_t)(t >> 58) & 1u; }
__device__ __forceinline__ uint32_t ticket_rows(unsigned long long t) { return 32u << ((uint32_t)(t >> 59) & 3u); }
__device__ __forceinline__ uint32_t ticket_next(unsigned long long t) { return (uint32_t)t; }
constexpr uint32_t kSmallLevel = 32768;
constexpr uint32_t kMinTileRows = 32;
constexpr uint32_t kFewModels = 8;
// While at most kFewModels models are unfinished, workgroups of a number from
// kFewGrid (the CUs of the whole GPU; a partition of it has no such workgroups
// to put to sleep) on wait kSleepyNaps naps (40 us) between polls: one workgroup per
// CU takes these models' levels soonest, and 768 more that poll slow them
// down (3 models of 64: 3.69 -> 3.34 ms, 6: 4.1 -> 3.65 ms).
constexpr uint32_t kFewGrid = 256;
constexpr uint32_t kSleepyNaps = 96;   // of 1024 cycles
static_assert(kExpandBlock == 256 && kMinTileRows == 32, "rows of a ticket: 32, 64, 128 or 256");

// A level of at most this many states stays with the workgroup that finished
// the level before it.  Larger ones (in tiles of 32 states on an otherwise
// idle GPU) pass through the tickets: a level's fixed cost is about 12 round
// trips there and four here, but each further 256 successors take three more.
constexpr uint32_t kSoloStates = 96;
// ... as long as its successors cannot come near the cap.
constexpr uint32_t kSoloRoom = 1u << 17;

// Rows per tile of a level.  Once at most kFewModels models remain and at
// least half the workgroups are idle, a level of at most kSmallLevel states
// is cut into tiles of down to kMinTileRows states, about one per workgroup
// that is there to take it: the deepest models' narrow levels, run after the
// rest of the batch has finished, then spread over the idle GPU instead of one
// full tile's latency chain per workgroup.  Otherwise tiles stay full (less
// per-tile work while the GPU is busy).
// There are the workgroups below kFewGrid, the others being asleep, and the
// other models' levels take theirs too: their wide levels seldom come at the
// same moment, so a level counts on twice its share.  One tile per idle
// workgroup, sleeping or not, made more and shorter tiles than were taken at
// once (batches of 3, 7, 8, 9 and 16 models: that, one per workgroup below
// kFewGrid, and one per twice the share): 3.28, 2.67, 2.68 ms; 2.20, 1.79,
// 1.72; 1.45, 1.36, 1.39; 4.31, 3.71, 3.48; 4.99, 4.39, 4.15.  With full
// tiles while more than four models remain: 3.28, 1.78, 1.66, 3.48, 4.35.
__device__ __forceinline__ uint32_t board_tile_rows(uint32_t remaining, uint32_t idle, uint32_t n_states) {
    if (n_states > kSmallLevel || remaining > kFewModels || idle < gridDim.x / 2)
        return kExpandBlock;
    const uint32_t takers = 2u * min(idle, kFewGrid) / (1u + remaining);
    uint32_t rows = kMinTileRows;
    while (rows < kExpandBlock && (uint64_t)rows * (takers + 1) < n_states)
        rows <<= 1;
    return rows;
}

// What a workgroup does next: tile `tile` of model `model`'s level of ticket
// `ticket`, or (server) a query to admit, or leave.
struct BoardItem {
    uint32_t model, tile, rows, limit, exit, admit;
    unsigned long long ticket, key;
};

// How the driver differs between the batch and the server:
//   kServe                the server: models come and go during the launch
//   model(ms, i, key)     model i's constants (block-wide call)
//   idle_check(...)       server: what an idle workgroup does besides looking
//                         for tiles (lane 0): 0 nothing, 1 admit, 2 leave
//   admit(M, B, i)        server: model i's level 0 (block-wide call)
//   level(M, k, n)        store a level's count (thread 0)
//   finished(M, i, own)   model i is finished (block-wide call)
struct BatchDriver {
    static constexpr bool kServe = false;
    __device__ const ModelState &model(const ModelState *ms, uint32_t i, unsigned long long) { return ms[i]; }
    __device__ uint32_t idle_check(BoardCtl *, uint32_t, uint32_t, uint32_t &) { return 0; }
    __device__ void admit(const ModelState &, BoardModel &, uint32_t) {}
    __device__ void level(const ModelState &M, uint32_t k, uint32_t n) {
        st_coherent(M.levels + k, (unsigned long long)n);
    }
    template <class Own>
    __device__ void finished(const ModelState &, uint32_t, const Own &) {}
};

// Take a tile (one wavefront, all lanes; `h` a lane-uniform random state).
// Each poll reads 64 tickets at once.  An idle GPU has more workgroups than
// new tiles, and their failed adds to one ticket would be served one after
// the other, so an idle workgroup tries with the probability that about two
// try for each tile; and it waits the longer between polls the more are idle:
// all polls read the same few lines, which the working workgroups' tickets and
// counts need too, and a workgroup that has just finished a tile looks again
// at once in any case.  With 768 idle workgroups that polled every 0.4 us, the
// server's 147-level queries took 11.5 ms and now take 8.5, 60 of a few
// thousand states each 6.7 and 3.4 ms; the 64-model batch 8.1 and 7.6 ms.
// The batch's naps are the shorter ones: a single model's levels, whose 255
// idle workgroups see all of a level's tiles at once, lose with longer ones
// (437 -> 500 us at 2.4 us).
template <class Driver>
__device__ inline void board_take(Driver &drv, const ModelState *ms, BoardModel *bm, unsigned long long *tickets,
                                  BoardCtl *ctl, uint32_t n, uint32_t &h, BoardItem *out) {
    constexpr bool kServe = Driver::kServe;
    const uint32_t lane = __lane_id();
    uint32_t polls = 0, scanned = 0, beat = 0;
    uint64_t since = 0;   // when this workgroup last saw the beat change
    h = h * 1664525u + 1013904223u;
    uint32_t slots = kServe ? min(ld_coherent(&ctl->slots), n) : n;
    uint32_t w0 = slots > 64 ? (h >> 8) % ((slots + 63) / 64) * 64 : 0;   // any window first
    bool idle = false;
    BoardItem it{};
    it.exit = 1;
    while (true) {
        const uint32_t i = w0 + lane;
        const unsigned long long tk = i < slots ? ld_coherent(tickets + i) : 0ull;
        const uint32_t remaining = ld_coherent(&ctl->remaining), error = ld_coherent(&ctl->error);
        const uint32_t idlers = ld_coherent(&ctl->idle);
        const uint32_t quota = remaining <= kFewModels ? kFewGrid : 0xFFFFFFFFu;
        if ((!kServe && remaining == 0u) || error != 0u)
            break;
        const uint32_t tiles = ticket_tiles(tk), avail = tiles - min(ticket_next(tk), tiles);
        const uint64_t mask = __ballot(avail != 0u);
        h = h * 1664525u + 1013904223u;
        if (mask) {
            const uint32_t r = h >> 8;
            bool go = true;
            if (idle) {
                const uint32_t all = wave_sum(min(avail, 1u << 16));
                go = r % max(min(idlers, quota), 1u) < 2u * all;
            }
            if (go) {
                const uint32_t k = r % (uint32_t)__popcll(mask);
                const uint32_t src = (uint32_t)__builtin_ctzll(__ballot(avail != 0u && mbcnt(mask) == k));
                unsigned long long got = 0;
                if (lane == src)
                    got = atomicAdd(tickets + i, 1ull);
                got = (unsigned long long)__shfl((uint32_t)got, (int)src, 64) |
                      (unsigned long long)__shfl((uint32_t)(got >> 32), (int)src, 64) << 32;
                if (ticket_next(got) < ticket_tiles(got)) {
                    it.exit = 0;
                    it.model = w0 + src;
                    it.tile = ticket_next(got);
                    it.ticket = got;
                    break;
                }
                continue;
            }
        }
        w0 = w0 + 64 < slots ? w0 + 64 : 0u;
        if (++scanned * 64 < slots)
            continue;   // the other windows
        scanned = 0;
        if (!idle) {
            idle = true;
            if (lane == 0)
                atomicAdd(&ctl->idle, 1u);
        }
        if (++polls % kBeatPolls == 0) {   // not in a short wait: the look delays the next poll
            const uint32_t b = ld_coherent(&ctl->beat);
            const uint64_t now = wall_clock64();
            if (polls == kBeatPolls || b != beat || remaining == 0u)
                since = now;
            else if (now - since > ld_coherent(&ctl->stall_ms) * kWallKHz && lane == 0)
                atomicCAS(&ctl->error, 0u, (uint32_t)LHS_ESTALL);
            beat = b;
        }
        if constexpr (kServe) {
            uint32_t act = 0, slot = 0;
            if (lane == 0)
                act = drv.idle_check(ctl, polls, remaining, slot);
            act = (uint32_t)__builtin_amdgcn_readfirstlane((int)act);
            if (act == 2u)
                break;
            if (act == 1u) {
                it.exit = 0;
                it.admit = 1;
                it.model = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot);
                break;
            }
            slots = min(ld_coherent(&ctl->slots), n);
            // the last query gone: wake up for the next one soon
            const uint32_t naps = remaining == 0u           ? min(polls, 8u)
                                  : blockIdx.x >= quota      ? kSleepyNaps
                                  : remaining <= kFewModels ? 2u
                                                            : 2u + 2u * (idlers >> 4);
            for (uint32_t k = 0; k < naps; ++k)
                __builtin_amdgcn_s_sleep(16);
        } else {
            const uint32_t naps = blockIdx.x >= quota ? 4u * kSleepyNaps : 1u + (min(idlers, quota) >> 5);
            for (uint32_t k = 0; k < naps; ++k)
                __builtin_amdgcn_s_sleep(4);
        }
    }
    if (idle && lane == 0)
        atomicSub(&ctl->idle, 1u);
    if (!it.exit && !it.admit) {
        // the level record was complete before its ticket; the batch reads it
        // only for the level's last tile and where there is a cap
        const uint32_t tiles = ticket_tiles(it.ticket);
        it.rows = ticket_rows(it.ticket);
        it.limit = 0xFFFFFFFFu;
        if (kServe || it.tile + 1 == tiles || ms[it.model].cap != 0) {
            const BoardModel &B = bm[it.model];
            const uint32_t nf = ld_coherent(&B.n_front), lim = ld_coherent(&B.limit);
            it.key = kServe ? ld_coherent(&B.key) : 0ull;
            it.rows = min(it.rows, nf - it.tile * it.rows);
            it.limit = lim;
        }
    }
    if (lane == 0)
        *out = it;
}

// The progress of the model whose level this workgroup has finalised or runs
// alone, and what it does next.
struct BoardOwn {
    unsigned long long total, edges, deadlocks;
    uint32_t cur, n_levels;         // frontier buffer of the level just found; levels so far
    uint32_t n_next, limit;         // its states, and the new states it may add
    uint32_t tiles, rows;           // its tiles, of `rows` states (0: the model is finished)
    uint32_t solo;                  // it stays with this workgroup
    uint32_t finished, err, over, overflow;   // the model has ended, and how
    unsigned long long waits;
};

// Whether a level of n_next states found after own.n_levels levels stays
// with its workgroup (whose tiles hold at most area_rows states).
__device__ __forceinline__ bool solo_next(const ModelState &M, const BoardOwn &own, uint32_t n_next,
                                          uint32_t area_rows) {
    return n_next != 0 && n_next <= min(kSoloStates, area_rows) && own.n_levels + 1 < M.max_levels &&
           (!M.cap || M.cap - own.total > (uint64_t)n_next + kSoloRoom);
}

// A level of n_next states of model M has been found (own: the progress
// before it).  End the model, keep the level whole (`solo`), or hand its
// tiles out and keep tile 0.  Thread 0.  Unless solo, the level's frontier is
// complete in fr[own.cur ^ 1].  err: the table's sticky error (server: ends
// the model).
template <class Driver>
__device__ inline void board_next(Driver &drv, const ModelState &M, BoardModel &B, unsigned long long *tickets,
                                  uint32_t i, BoardCtl *ctl, BoardOwn &own, uint32_t n_next, bool over, uint32_t err,
                                  bool solo, uint32_t remaining, uint32_t idle, uint32_t area_rows) {
    bool done = false;
    uint32_t overflow = 0;
    own.finished = 0;
    own.n_next = n_next;
    own.tiles = 0;
    own.solo = 0;
    if (err || n_next == 0) {
        done = true;
    } else if (over) {
        st_coherent(&B.capped, 1u);
        done = true;
    } else if (own.n_levels == M.max_levels) {
        overflow = 1;
        st_coherent(&B.overflow, 1u);
        done = true;
    } else {
        drv.level(M, own.n_levels, n_next);
        ++own.n_levels;
        own.total += n_next;
        own.cur ^= 1u;
        if (M.handover && (n_next > M.handover || own.n_levels == M.max_levels)) {
            // a level too wide (or one level array full): the caller
            // expands it and the rest
            st_coherent(&B.handed, 1u);
            done = true;
        }
    }
    const uint64_t room = M.cap ? M.cap - own.total : 0xFFFFFFFFull;
    own.limit = (uint32_t)min<uint64_t>(room, 0xFFFFFFFFull);
    if (solo) {
        own.tiles = 1;
        own.rows = kExpandBlock;
        own.solo = 1;
        return;
    }
    unsigned long long waits = 0;
    if (!done) {
        own.rows = min(board_tile_rows(remaining, idle, n_next), area_rows);
        own.tiles = (n_next + own.rows - 1) / own.rows;
        st_coherent(&B.n_front, n_next);
        st_coherent(&B.limit, own.limit);
    } else {
        err = ld_coherent(&M.t.status->error);
        waits = ld_coherent(&M.t.status->wait_hits);
        st_coherent(&B.status_error, err);
        st_coherent(&B.wait_hits, waits);
        st_coherent(&B.done, 1u);
    }
    st_coherent(&B.total, own.total);
    st_coherent(&B.edges, own.edges);
    st_coherent(&B.deadlocks, own.deadlocks);
    st_coherent(&B.cur, own.cur);
    st_coherent(&B.n_levels, own.n_levels);
    wait_vm_complete();
    if (done) {
        own.finished = 1;
        own.err = err;
        own.over = over;
        own.overflow = overflow;
        own.waits = waits;
    } else {
        if (own.tiles > 1)
            st_coherent(tickets + i, make_ticket(own.tiles, own.cur, own.rows, 1u));
        atomicAdd(&ctl->beat, 1u);
    }
}

// Rows of W words that fit a tile area of area_words: a power of two from
// kMinTileRows to kExpandBlock.  A byte row of Wmax words takes at least a
// quarter of W <= Wmax words, and a stride of one more at most: 32 rows fit
// wherever 256 byte rows do.
__host__ __device__ constexpr uint32_t word_rows(uint32_t area_words, uint32_t W) {
    uint32_t rows = kExpandBlock;
    while (rows > kMinTileRows && rows * row_stride<uint32_t>(W) > area_words)
        rows /= 2;
    return rows;
}
constexpr bool word_rows_fit() {
    for (uint32_t wmax = 1; wmax <= 32; ++wmax)
        for (uint32_t w = 1; w <= wmax; ++w)
            if (word_rows(kExpandBlock * row_stride<uint8_t>(wmax), w) * row_stride<uint32_t>(w) >
                kExpandBlock * row_stride<uint8_t>(wmax))
                return false;
    return true;
}
static_assert(word_rows_fit(), "a word query always has a tile in a byte launch");

// One launch: all levels of the n models (server: of the queries in n slots).
// area_words (server, byte rows): the launch's tile area.  A query whose words
// do not fit bytes joins such a launch with word rows and as many of them as
// the area holds.
template <int G, uint32_t LS, class R, class Driver>
__device__ __forceinline__ void board_run(Driver &drv, uint32_t *smem, const ModelState *__restrict__ ms,
                                          BoardModel *bm, unsigned long long *tickets, BoardCtl *ctl, uint32_t n,
                                          uint32_t tcap, uint32_t area_words = 0) {
    constexpr bool kServe = Driver::kServe;
    constexpr bool kBoth = kServe && sizeof(R) == 1;   // word queries among byte ones
    __shared__ BoardItem s_it;
    __shared__ BoardOwn s_own;
    __shared__ uint32_t s_fin, s_over;
    enum : uint32_t { kTake, kKept, kSolo };
    const uint32_t tid = threadIdx.x;
    uint32_t h = (blockIdx.x + 1u) * 2654435761u, mode = kTake, solo_levels = 0;
    expand_begin();
    while (true) {
        if (mode == kTake) {
            if (tid < 64)
                board_take(drv, ms, bm, tickets, ctl, n, h, &s_it);
            __syncthreads();
            if (s_it.exit)
                break;
        }
        const uint32_t i = s_it.model;
        const ModelState &M = drv.model(ms, i, s_it.key);
        BoardModel &B = bm[i];
        if (kServe && mode == kTake && s_it.admit) {
            // a query's level 0: s0, kept like a level this workgroup found
            drv.admit(M, B, i);
            if (tid == 0) {
                s_own = BoardOwn{};
                s_own.total = 1;
                s_own.n_levels = 1;
                s_own.n_next = 1;
                s_own.tiles = 1;
                s_own.rows = kExpandBlock;
                s_own.limit = M.cap ? (uint32_t)min<unsigned long long>(M.cap - 1, 0xFFFFFFFFull) : 0xFFFFFFFFu;
                s_own.solo = !M.cap || M.cap > 2 * kSoloRoom;
                s_it.tile = 0;
                s_it.rows = 1;
                s_it.limit = s_own.limit;
                s_it.key = M.m.key;
            }
            __syncthreads();
            solo_levels = 0;
            mode = s_own.solo ? kSolo : kKept;
        }
        const bool solo = mode == kSolo;
        const uint32_t cur = mode == kTake ? ticket_cur(s_it.ticket) : s_own.cur;
        const uint32_t rows = s_it.rows, tiles = mode == kTake ? ticket_tiles(s_it.ticket) : s_own.tiles;
        const uint64_t base = mode == kTake ? (uint64_t)s_it.tile * ticket_rows(s_it.ticket) : 0u;
        const uint32_t limit = solo ? 0xFFFFFFFFu : s_it.limit;
        bool words = false;
        uint32_t area_rows = kExpandBlock;
        if constexpr (kBoth) {
            words = __builtin_amdgcn_readfirstlane((int)M.words) != 0;
            if (words)
                area_rows = word_rows(area_words, (uint32_t)__builtin_amdgcn_readfirstlane((int)M.m.W));
        }
        uint32_t *nbuf = words ? expand_nbuf<G, uint32_t>(smem, M.m.W, tcap, area_rows)
                               : expand_nbuf<G, R>(smem, M.m.W, tcap);
        uint32_t *lds_front = nbuf + kHoldFront;
        // a solo level's frontier is in LDS from the second one on
        const uint32_t *held = solo && solo_levels ? lds_front : nullptr;
        if (tid == 0)
            s_pushed = 0;
        if (words)
            expand_tile<G, LS, uint32_t, true, false, false, false, kServe>(
                smem, M.t, M.m, M.fr[cur], base, rows, M.fr[cur ^ 1u], &B.lc, limit, tcap, SegOut{}, solo, held,
                area_rows);
        else
            expand_tile<G, LS, R, true, false, false, false, kServe>(
                smem, M.t, M.m, M.fr[cur], base, rows, M.fr[cur ^ 1u], &B.lc, limit, tcap, SegOut{}, solo, held);
        if (!solo) {
            // this workgroup's stores of the tile are complete before it
            // counts the tile as done
            wait_vm_complete();
            __syncthreads();
            if (tid == 0)
                s_fin = atomicAdd(&B.tiles_done, 1u) + 1u == tiles;
            __syncthreads();
            if (!s_fin) {
                mode = kTake;
                continue;
            }
            // the level is complete: its counts, and the progress so far
            uint32_t n_next = 0, remaining = 0, idle = 0, error = 0, err = 0;
            if (tid == 0) {
                n_next = ld_coherent(&B.lc.n_next);
                err = kServe ? ld_coherent(&M.t.status->error) : 0u;
                const unsigned long long e = ld_coherent(&B.lc.edges), d = ld_coherent(&B.lc.deadlocks);
                const unsigned long long pt = ld_coherent(&B.total), pe = ld_coherent(&B.edges),
                                         pd = ld_coherent(&B.deadlocks);
                const uint32_t nl = ld_coherent(&B.n_levels);
                remaining = ld_coherent(&ctl->remaining);
                idle = ld_coherent(&ctl->idle);
                error = ld_coherent(&ctl->error);
                const bool over = !err && M.cap && n_next > limit;
                s_own.total = pt;
                s_own.edges = pe + (over ? 0 : e);
                s_own.deadlocks = pd + (over ? 0 : d);
                s_own.cur = cur;
                s_own.n_levels = nl;
                s_own.n_next = n_next;
                s_over = over;
            }
            __syncthreads();
            if (s_over) {
                // discard the partial level: zero every slot it claimed
                const uint32_t *next = M.fr[cur ^ 1u];
                for (uint32_t j = tid; j < s_own.n_next; j += kExpandBlock)
                    st_coherent(M.t.bucket + ld_coherent(next + j), 0ull);
                wait_vm_complete();
                __syncthreads();
            }
            if (tid == 0) {
                st_coherent(&B.lc.n_next, 0u);
                st_coherent(&B.lc.abort, 0u);
                st_coherent(&B.lc.edges, 0ull);
                st_coherent(&B.lc.deadlocks, 0ull);
                st_coherent(&B.tiles_done, 0u);
                board_next(drv, M, B, tickets, i, ctl, s_own, n_next, s_over != 0, err,
                           solo_next(M, s_own, n_next, area_rows) && !s_over && !err, remaining, idle, area_rows);
                s_it.exit = error;
            }
        } else {
            __syncthreads();
            // found: in the buffer, or (it filled up) in the next frontier
            const bool spilled = s_pushed != 0;
            if (spilled)
                flush_new_slots<true>(nbuf, M.fr[cur ^ 1u], &B.lc, 0xFFFFFFFFu);
            const uint32_t found = spilled ? s_pushed : s_nnew;
            const bool failed = kServe && s_failed != 0;   // the query ends with the table's error
            const bool stay = !spilled && !failed && solo_next(M, s_own, found, area_rows);
            if (!spilled)
                for (uint32_t j = tid; j < found; j += kExpandBlock) {
                    if (stay)
                        lds_front[j] = nbuf[j];
                    else
                        st_coherent(M.fr[cur ^ 1u] + j, nbuf[j]);
                }
            if (!stay)
                wait_vm_complete();
            __syncthreads();
            if (tid == 0) {
                s_own.edges += s_acc_edges;
                s_own.deadlocks += s_acc_dead;
                s_acc_edges = 0;
                s_acc_dead = 0;
                s_nnew = 0;
                flush_counters(M.t.status);
                uint32_t remaining = 0, idle = 0, error = 0, err = 0;
                if (failed)
                    err = ld_coherent(&M.t.status->error);
                if (!stay || (solo_levels & 31u) == 31u) {
                    remaining = ld_coherent(&ctl->remaining);
                    idle = ld_coherent(&ctl->idle);
                    error = ld_coherent(&ctl->error);
                }
                if (spilled)
                    st_coherent(&B.lc.n_next, 0u);
                if ((solo_levels & 31u) == 31u)
                    atomicAdd(&ctl->beat, 1u);
                board_next(drv, M, B, tickets, i, ctl, s_own, found, false, err, stay, remaining, idle,
                           area_rows);
                s_it.exit = error;
            }
        }
        if (tid == 0 && s_own.tiles) {
            s_it.tile = 0;
            s_it.rows = min(s_own.rows, s_own.n_next);
            s_it.limit = s_own.limit;
        }
        __syncthreads();
        if (s_own.finished) {
            drv.finished(M, i, s_own);
            if (tid == 0) {
                atomicAdd(&ctl->beat, 1u);
                atomicSub(&ctl->remaining, 1u);
            }
        }
        if (s_own.tiles && s_it.exit)
            break;
        solo_levels = s_own.solo && solo ? solo_levels + 1 : 0;
        mode = s_own.solo ? kSolo : (s_own.tiles ? kKept : kTake);
    }
}

// The levels of a single-model BFS that a board launch runs (explore_levels):
// its control words, ticket, level state, model constants and level counts,
// in one region (device, and its pinned mirror).
constexpr uint32_t kBoardLevels = 4096;           // level counts per launch
constexpr uint32_t kBoardHandover = 1u << 16;     // states of a level the launch still expands
constexpr uint32_t kBoardGrid = 256;              // workgroups
struct LevelsArea {
    BoardCtl ctl;
    unsigned long long tickets[64];
    BoardModel bm;
    ModelState ms;
    unsigned long long levels[kBoardLevels];
};

}  // namespace lhs
