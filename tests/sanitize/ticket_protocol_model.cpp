// CPU-thread model of the persistent level driver (csrc/board.h) and of the
// server on it (csrc/serve.hip), for ThreadSanitizer: threads stand for
// workgroups.  The table itself is one atomic byte per state here
// (gpu_protocol_model.cpp, part 1, models find-or-put).
//
// Payload is plain memory, so that TSan reports any access pair that the
// protocol leaves unordered: frontier entries, a model's level record (states,
// limit, buffer, progress, key), a query's constants and level counts, its
// completion record, the admission ring.  Tickets, counters of a level and
// control words are std::atomic; an access that the kernel leaves unordered is
// relaxed.  Where the kernel waits for its earlier accesses to complete before
// an announcing store or atomic, the model uses release; where it issues its
// next accesses only after an observed value returned, acquire.
//
//  * Hand-out: one 64-bit ticket a model, the level's shape above the next
//    tile.  A worker polls the tickets (relaxed), adds one to a model's and
//    knows from the returned word what it got, whatever the poll said: the
//    level, or the query in the slot, may have changed in between.
//  * Finalising: the worker that counts a level's last tile done reads its
//    counters, rolls back a level beyond the cap, resets the counters, writes
//    the next level's record and only then its ticket; tile 0 it keeps.
//  * Solo levels: a narrow level's states and counts stay with the worker; the
//    record is written when the model leaves it or ends.
//  * Server: a host thread posts queries (constants, emptied table, admission
//    entry, then the tail), an idle worker admits them, and the worker that
//    ends one fills its completion record and publishes it.  The host then
//    reuses the slot at once, before the worker has counted the query as gone;
//    workers tell queries of one slot apart by a key.  Leaving and admitting
//    announce themselves before each looks at the other; the host starts
//    another launch for queries that came too late, and now and then asks a
//    launch to drain.
//
// Models are N independent cyclic processes of L states, with and without a
// cap; every result is compared with a sequential search.
//
// Planted mistakes (-DPLANT=n), each of which TSan or a result has to show:
//   1 a ticket written relaxed              2 a finished tile counted relaxed
//   3 a level's counters reset after the    4 its record written after the
//     next ticket                              ticket
//   5 the admission tail raised relaxed     6 a completion record published
//                                              relaxed
//   7 constants kept by slot, without key   8 a solo level's states written
//                                              after the ticket
//   9 level counts copied after the record  10 the poll's word trusted instead
//                                              of the add's
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <deque>
#include <memory>
#include <random>
#include <thread>
#include <vector>

#ifndef PLANT
#define PLANT 0
#endif

namespace {

using std::memory_order_acq_rel;
using std::memory_order_acquire;
using std::memory_order_relaxed;
using std::memory_order_release;
using std::memory_order_seq_cst;

constexpr uint32_t kMaxStates = 4096, kMaxLevels = 128, kSolo = 6, kRing = 16, kNoLimit = 0xFFFFFFFFu;
constexpr uint32_t kBlockRows = 16;   // the largest tile
constexpr double kStallSeconds = 10;

double now_s() {
    return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

struct Result {
    uint64_t total = 0, edges = 0;
    bool capped = false;
    std::vector<uint64_t> levels;
    bool operator==(const Result &o) const {
        return total == o.total && edges == o.edges && capped == o.capped && levels == o.levels;
    }
};

uint32_t pow_u(uint32_t b, uint32_t e) { return e ? b * pow_u(b, e - 1) : 1; }
uint32_t succ(uint32_t s, uint32_t p, uint32_t L) {
    const uint32_t w = pow_u(L, p), d = (s / w) % L;
    return s - d * w + ((d + 1) % L) * w;
}

Result sequential(uint32_t N, uint32_t L, uint64_t cap) {
    Result r;
    std::vector<char> seen(pow_u(L, N));
    std::vector<uint32_t> front{0};
    seen[0] = 1;
    r.total = 1;
    r.levels.push_back(1);
    while (true) {
        std::vector<uint32_t> next;
        for (uint32_t s : front)
            for (uint32_t p = 0; p < N; ++p) {
                const uint32_t t = succ(s, p, L);
                if (!seen[t]) {
                    seen[t] = 1;
                    next.push_back(t);
                }
            }
        if (cap && r.total + next.size() > cap) {
            r.capped = true;
            return r;
        }
        r.edges += (uint64_t)front.size() * N;
        if (next.empty())
            return r;
        r.levels.push_back(next.size());
        r.total += next.size();
        front.swap(next);
    }
}

// A model's constants (plain; the server's host rewrites a slot's).
struct Consts {
    uint32_t N = 0, L = 0;
    uint64_t cap = 0, key = 0;
};

struct Model {
    // payload: the level record, the level counts, the frontiers
    uint32_t n_front = 0, limit = 0, cur = 0, n_levels = 0;
    uint64_t total = 0, edges = 0, key = 0;
    bool capped = false;
    std::vector<uint64_t> levels = std::vector<uint64_t>(kMaxLevels), host_levels = std::vector<uint64_t>(kMaxLevels);
    std::vector<uint32_t> fr[2] = {std::vector<uint32_t>(kMaxStates), std::vector<uint32_t>(kMaxStates)};
    Consts consts;
    // atomics: the level's counters, the table
    std::atomic<uint32_t> n_next{0}, abort{0}, tiles_done{0};
    std::atomic<uint64_t> lc_edges{0}, ticket{0};
    std::vector<std::atomic<uint8_t>> table = std::vector<std::atomic<uint8_t>>(kMaxStates);
};

uint64_t make_ticket(uint32_t tiles, uint32_t cur, uint32_t rows, uint32_t next) {
    return (uint64_t)(tiles | cur << 20 | rows << 21) << 32 | next;
}
uint32_t t_tiles(uint64_t t) { return (uint32_t)(t >> 32) & 0xFFFFFu; }
uint32_t t_cur(uint64_t t) { return (uint32_t)(t >> 52) & 1u; }
uint32_t t_rows(uint64_t t) { return (uint32_t)(t >> 53); }
uint32_t t_next(uint64_t t) { return (uint32_t)t; }

struct Record {   // payload, published by seq
    std::atomic<uint64_t> seq{0};
    uint32_t slot = 0, n_levels = 0;
    uint64_t total = 0, edges = 0;
    bool capped = false;
};

struct Launch {
    explicit Launch(uint32_t n_models, bool server) : n(n_models), serve(server), m(n_models) {}
    const uint32_t n;
    const bool serve;
    std::deque<Model> m;
    std::atomic<uint32_t> remaining{0}, error{0}, idle{0}, beat{0};
    // server
    std::atomic<uint64_t> admit_tail{0}, admit_head{0}, done_tail{0};
    std::atomic<uint32_t> closing{0}, stop{0};
    uint32_t admit_slot[kRing] = {};
    Record rec[kRing];
};

struct Own {
    uint64_t total = 0, edges = 0;
    uint32_t cur = 0, n_levels = 0, n_next = 0, limit = 0, tiles = 0, rows = 0;
    bool solo = false, finished = false, capped = false;
};

struct Worker {
    Launch &g;
    std::mt19937 rng;
    Consts held;
    uint32_t held_slot = 0xFFFFFFFFu, quiet = 0;
    std::vector<uint32_t> found;   // new states of the tile or the solo level
    uint64_t tile_edges = 0;

    Worker(Launch &l, uint32_t id) : g(l), rng(id * 7919 + 17) {}

    // The states of a tile or of a solo level's frontier; new ones to `found`.
    void expand(Model &M, const Consts &c, const uint32_t *front, uint32_t rows, bool hold) {
        found.clear();
        tile_edges = 0;
        for (uint32_t i = 0; i < rows; ++i) {
            if (!hold && M.abort.load(memory_order_relaxed))
                return;
            for (uint32_t p = 0; p < c.N; ++p) {
                const uint32_t t = succ(front[i], p, c.L);
                if (!M.table[t].exchange(1, memory_order_relaxed))
                    found.push_back(t);
                ++tile_edges;
            }
        }
    }
    void append(Model &M, uint32_t to, uint32_t limit) {
        if (found.empty())
            return;
        const uint32_t at = M.n_next.fetch_add((uint32_t)found.size(), memory_order_relaxed);
        if ((uint64_t)at + found.size() > limit)
            M.abort.store(1, memory_order_relaxed);
        for (uint32_t k = 0; k < found.size(); ++k)
            M.fr[to][at + k] = found[k];
    }

    bool solo_next(const Consts &c, const Own &o, uint32_t n_next) const {
        return n_next && n_next <= kSolo && (!c.cap || c.cap - o.total > n_next + 64);
    }

    void next_level(Model &M, const Consts &c, Own &o, uint32_t n_next, bool over, bool solo) {
        bool done = false;
        o.finished = o.solo = false;
        o.n_next = n_next;
        o.tiles = 0;
        if (n_next == 0) {
            done = true;
        } else if (over) {
            o.capped = true;
            done = true;
        } else {
            M.levels[o.n_levels++] = n_next;
            o.total += n_next;
            o.cur ^= 1u;
        }
        o.limit = c.cap ? (uint32_t)(c.cap - o.total) : kNoLimit;
        if (solo) {
            o.tiles = 1;
            o.rows = kBlockRows;
            o.solo = true;
            return;
        }
        uint32_t shape = 0;
        if (!done) {
            o.rows = 4u << (rng() % 3);   // as few and as many tiles as the idle workers ask for
            o.tiles = shape = (n_next + o.rows - 1) / o.rows;
        }
        auto record = [&] {
            M.n_front = n_next;
            M.limit = o.limit;
            M.total = o.total;
            M.edges = o.edges;
            M.cur = o.cur;
            M.n_levels = o.n_levels;
            M.capped = o.capped;
        };
        if (PLANT != 4)
            record();
        if (done)
            o.finished = true;
        else if (shape > 1)
            M.ticket.store(make_ticket(shape, o.cur, o.rows, 1), PLANT == 1 ? memory_order_relaxed : memory_order_release);
        if (PLANT == 4)
            record();
        g.beat.fetch_add(1, memory_order_relaxed);
    }

    void finished(Model &M, uint32_t slot, const Own &o) {
        if (!g.serve)
            return;
        auto copy = [&] { std::copy_n(M.levels.begin(), o.n_levels, M.host_levels.begin()); };
        if (PLANT != 9)
            copy();
        const uint64_t pos = g.done_tail.fetch_add(1, memory_order_relaxed);
        Record &r = g.rec[pos % kRing];
        r.slot = slot;
        r.n_levels = o.n_levels;
        r.total = o.total;
        r.edges = o.edges;
        r.capped = o.capped;
        r.seq.store(pos + 1, PLANT == 6 ? memory_order_relaxed : memory_order_release);
        if (PLANT == 9)
            copy();
    }

    const Consts &constants(Model &M, uint32_t i, uint64_t key) {
        if (held_slot != i || (PLANT != 7 && held.key != key)) {
            held = M.consts;
            held_slot = i;
        }
        return held;
    }

    // 0 nothing, 1 admit `slot`, 2 leave
    int idle_check(uint32_t &slot) {
        const bool closing = g.closing.load(memory_order_relaxed) != 0;
        uint64_t ah = g.admit_head.load(memory_order_relaxed);
        if (!closing && ah < g.admit_tail.load(memory_order_acquire)) {
            g.remaining.fetch_add(1, memory_order_seq_cst);
            if (!g.closing.load(memory_order_seq_cst) &&
                g.admit_head.compare_exchange_strong(ah, ah + 1, memory_order_relaxed)) {
                slot = g.admit_slot[ah % kRing];
                return 1;
            }
            g.remaining.fetch_sub(1, memory_order_relaxed);
        } else if (g.remaining.load(memory_order_relaxed)) {
            quiet = 0;
        } else if (++quiet > 2000 || closing || g.stop.load(memory_order_relaxed)) {
            g.closing.exchange(1, memory_order_seq_cst);
            if (!g.remaining.load(memory_order_seq_cst))
                return 2;
        }
        return 0;
    }

    void run() {
        enum { kTake, kKept, kSoloMode } mode = kTake;
        uint32_t i = 0, tile = 0, rows = 0, limit = 0, solo_levels = 0;
        uint64_t ticket = 0;
        Own own;
        std::vector<uint32_t> alone;   // a solo level's frontier
        while (true) {
            if (mode == kTake) {
                bool admit = false, got = false;
                bool idle = false;
                uint32_t beat = 0;
                double since = now_s();
                while (!got && !admit) {
                    if (g.error.load(memory_order_relaxed) || (!g.serve && !g.remaining.load(memory_order_relaxed)))
                        break;
                    const uint32_t first = rng() % g.n;
                    for (uint32_t k = 0; k < g.n && !got; ++k) {
                        const uint32_t j = (first + k) % g.n;
                        const uint64_t seen = g.m[j].ticket.load(memory_order_relaxed);
                        if (t_next(seen) >= t_tiles(seen))
                            continue;
                        const uint64_t word = g.m[j].ticket.fetch_add(1, memory_order_acquire);
                        ticket = PLANT == 10 ? seen : word;
                        if (t_next(ticket) < t_tiles(ticket)) {
                            got = true;
                            i = j;
                        }
                    }
                    if (got)
                        break;
                    if (!idle) {
                        idle = true;
                        g.idle.fetch_add(1, memory_order_relaxed);
                    }
                    const uint32_t b = g.beat.load(memory_order_relaxed);
                    if (b != beat || (g.serve && !g.remaining.load(memory_order_relaxed)))
                        since = now_s();
                    else if (now_s() - since > kStallSeconds)
                        g.error.store(1, memory_order_relaxed);
                    beat = b;
                    if (g.serve) {
                        const int act = idle_check(i);
                        if (act == 2)
                            break;
                        admit = act == 1;
                    }
                    if (!admit)
                        std::this_thread::yield();
                }
                if (idle)
                    g.idle.fetch_sub(1, memory_order_relaxed);
                if (!got && !admit)
                    return;
                Model &M = g.m[i];
                if (admit) {
                    const Consts &c = constants(M, i, 0);
                    if (held.key == 0)
                        g.error.store(2, memory_order_relaxed);
                    M.table[0].exchange(1, memory_order_relaxed);
                    M.fr[0][0] = 0;
                    M.levels[0] = 1;
                    M.key = c.key;
                    M.n_next.store(0, memory_order_relaxed);
                    M.abort.store(0, memory_order_relaxed);
                    M.lc_edges.store(0, memory_order_relaxed);
                    M.tiles_done.store(0, memory_order_relaxed);
                    M.total = 1;
                    M.edges = 0;
                    M.n_levels = 1;
                    M.cur = 0;
                    M.capped = false;
                    own = Own{};
                    own.total = own.n_levels = own.n_next = own.tiles = 1;
                    own.rows = kBlockRows;
                    own.limit = c.cap ? (uint32_t)(c.cap - 1) : kNoLimit;
                    own.solo = !c.cap || c.cap > 128;
                    tile = 0;
                    rows = 1;
                    limit = own.limit;
                    solo_levels = 0;
                    mode = own.solo ? kSoloMode : kKept;
                } else {
                    tile = t_next(ticket);
                    rows = std::min(t_rows(ticket), M.n_front - tile * t_rows(ticket));
                    limit = M.limit;
                }
            }
            Model &M = g.m[i];
            const Consts &c = constants(M, i, g.serve ? M.key : 0);
            const bool solo = mode == kSoloMode;
            const uint32_t cur = mode == kTake ? t_cur(ticket) : own.cur;
            const uint32_t tiles = mode == kTake ? t_tiles(ticket) : own.tiles;
            const uint32_t base = mode == kTake ? tile * t_rows(ticket) : 0;
            if (!solo) {
                expand(M, c, M.fr[cur].data() + base, rows, false);   // an aborted tile lists what it claimed
                append(M, cur ^ 1u, limit);
                M.lc_edges.fetch_add(tile_edges, memory_order_relaxed);
                if (M.tiles_done.fetch_add(1, PLANT == 2 ? memory_order_relaxed : memory_order_acq_rel) + 1 != tiles) {
                    mode = kTake;
                    continue;
                }
                const uint32_t n_next = M.n_next.load(memory_order_relaxed);
                const bool over = c.cap && n_next > limit;
                own = Own{};
                own.total = M.total;
                own.edges = M.edges + (over ? 0 : M.lc_edges.load(memory_order_relaxed));
                own.n_levels = M.n_levels;
                own.cur = cur;
                if (over)
                    for (uint32_t k = 0; k < n_next; ++k)
                        M.table[M.fr[cur ^ 1u][k]].store(0, memory_order_relaxed);
                auto reset = [&] {
                    M.n_next.store(0, memory_order_relaxed);
                    M.abort.store(0, memory_order_relaxed);
                    M.lc_edges.store(0, memory_order_relaxed);
                    M.tiles_done.store(0, memory_order_relaxed);
                };
                if (PLANT != 3)
                    reset();
                next_level(M, c, own, n_next, over, solo_next(c, own, n_next) && !over);
                if (PLANT == 3) {
                    std::this_thread::yield();
                    reset();
                }
            } else {
                expand(M, c, solo_levels ? alone.data() : M.fr[cur].data(), rows, true);
                own.edges += tile_edges;
                const uint32_t n_next = (uint32_t)found.size();
                const bool stay = solo_next(c, own, n_next);
                auto hand = [&] { std::copy(found.begin(), found.end(), M.fr[cur ^ 1u].begin()); };
                if (stay)
                    alone = found;
                else if (PLANT != 8)
                    hand();
                next_level(M, c, own, n_next, false, stay);
                if (!stay && PLANT == 8)
                    hand();
            }
            if (own.tiles) {
                tile = 0;
                rows = std::min(own.rows, own.n_next);
                limit = own.limit;
            }
            if (own.finished) {
                finished(M, i, own);
                g.remaining.fetch_sub(1, memory_order_relaxed);
            }
            solo_levels = own.solo && solo ? solo_levels + 1 : 0;
            mode = own.solo ? kSoloMode : own.tiles ? kKept : kTake;
        }
    }
};

struct Shape {
    uint32_t N, L;
    uint64_t cap;
};
const Shape kShapes[] = {{1, 40, 0},  {2, 20, 0},   {3, 8, 0},   {3, 10, 300}, {4, 6, 0},   {2, 30, 500},
                         {5, 4, 0},   {5, 4, 777},  {3, 15, 0},  {1, 3, 0},    {6, 3, 100}, {2, 40, 0},
                         {4, 8, 0},   {4, 8, 3000}, {3, 12, 20}, {1, 60, 0}};

int errors = 0;
void check(const char *what, const Shape &s, const Result &got) {
    const Result want = sequential(s.N, s.L, s.cap);
    if (!(got == want)) {
        std::printf("WRONG %s N=%u L=%u cap=%llu: total %llu (%llu) edges %llu (%llu) levels %zu (%zu)\n", what, s.N, s.L,
                    (unsigned long long)s.cap, (unsigned long long)got.total, (unsigned long long)want.total,
                    (unsigned long long)got.edges, (unsigned long long)want.edges, got.levels.size(), want.levels.size());
        ++errors;
    }
}

void batch(uint32_t workers, uint32_t rep) {
    const uint32_t n = sizeof(kShapes) / sizeof(kShapes[0]);
    Launch g(n, false);
    g.remaining = n;
    for (uint32_t i = 0; i < n; ++i) {
        Model &M = g.m[i];
        M.consts = Consts{kShapes[i].N, kShapes[i].L, kShapes[i].cap, 0};
        M.table[0] = 1;
        M.n_front = 1;
        M.limit = kShapes[i].cap ? (uint32_t)(kShapes[i].cap - 1) : kNoLimit;
        M.total = M.n_levels = 1;
        M.levels[0] = 1;
        M.ticket = make_ticket(1, 0, kBlockRows, 0);
    }
    std::vector<std::thread> th;
    for (uint32_t w = 0; w < workers; ++w)
        th.emplace_back([&g, w, rep] { Worker(g, w + 100 * rep).run(); });
    for (auto &t : th)
        t.join();
    if (g.error) {
        std::printf("WRONG batch error %u\n", g.error.load());
        ++errors;
        return;
    }
    for (uint32_t i = 0; i < n; ++i) {
        Model &M = g.m[i];
        check("batch", kShapes[i], Result{M.total, M.edges, M.capped, {M.levels.begin(), M.levels.begin() + M.n_levels}});
    }
}

void server(uint32_t workers, uint32_t slots, uint32_t queries, uint32_t seed) {
    Launch g(slots, true);
    std::mt19937 rng(seed);
    std::vector<uint32_t> free_slots;
    for (uint32_t k = 0; k < slots; ++k)
        free_slots.push_back(k);
    std::vector<Shape> of(slots);
    uint32_t submitted = 0, live = 0;
    uint64_t posted = 0, done_head = 0, key = 1;
    std::vector<std::thread> th;
    double since = now_s();
    while (submitted < queries || live) {
        bool progress = false;
        uint32_t burst = rng() % 4;
        while (burst-- && submitted < queries && !free_slots.empty()) {
            const uint32_t slot = free_slots.back();
            free_slots.pop_back();
            of[slot] = kShapes[rng() % (sizeof(kShapes) / sizeof(kShapes[0]))];
            Model &M = g.m[slot];
            M.consts = Consts{of[slot].N, of[slot].L, of[slot].cap, key++};
            for (auto &b : M.table)
                b.store(0, memory_order_relaxed);
            g.admit_slot[posted % kRing] = slot;
            ++posted;
            g.admit_tail.store(posted, PLANT == 5 ? memory_order_relaxed : memory_order_release);
            ++submitted;
            ++live;
            progress = true;
        }
        if (th.empty() && live) {
            g.closing = 0;
            for (uint32_t w = 0; w < workers; ++w)
                th.emplace_back([&g, w, seed] { Worker(g, w + 31 * seed).run(); });
        }
        Record &r = g.rec[done_head % kRing];
        if (r.seq.load(memory_order_acquire) == done_head + 1) {
            ++done_head;
            Model &M = g.m[r.slot];
            check("server", of[r.slot],
                  Result{r.total, r.edges, r.capped, {M.host_levels.begin(), M.host_levels.begin() + r.n_levels}});
            free_slots.push_back(r.slot);
            --live;
            progress = true;
        }
        if (!th.empty() && rng() % 2048 == 0)
            g.closing.exchange(1);       // drain: no more admissions to this launch
        if (!th.empty() && g.closing.load() && (rng() % 16 == 0 || !live)) {
            for (auto &t : th)
                t.join();
            th.clear();
        }
        if (progress)
            since = now_s();
        else if (g.error.load() || now_s() - since > 2 * kStallSeconds) {
            std::printf("WRONG server stalled, error %u\n", g.error.load());
            ++errors;
            g.error.store(1);
            break;
        } else {
            std::this_thread::yield();
        }
    }
    g.stop = 1;
    for (auto &t : th)
        t.join();
}

}  // namespace

int main(int argc, char **argv) {
    const uint32_t reps = argc > 1 ? (uint32_t)std::atoi(argv[1]) : 6;
    for (uint32_t rep = 0; rep < reps && !errors; ++rep) {
        for (uint32_t w : {1u, 3u, 6u})
            batch(w, rep);
        server(1 + rep % 5, 1 + rep % 4, 60, rep + 1);
    }
    std::printf("errors %d\n", errors);
    return errors != 0;
}
