// Device-side core of the lockless table: slot encoding, the vector hash and
// find-or-put (Algorithm 3 with walking-the-line, Algorithm 4) executed by a
// group of G cooperating lanes per operation.
//
// Slot (64 bits): 0 = empty; bit 63 OCC = claimed; bit 62 DONE = the vector
// has been written to the data array; bits 61..0 = memoised hash (the low 62
// bits of h1).  A slot goes empty -> claimed(memo) -> done(memo) and never
// changes again (figure "State diagram of buckets"): a slot seen non-empty
// keeps its memo forever, which is what makes a stale snapshot of a line safe.
//
// Memory ordering on gfx950 (8 XCDs, one L2 each).  The paper's requirement
// (section on the algorithm's memory-model needs): the vector must not be
// written before its slot is claimed, and a reader that sees DONE must see
// the whole vector.  Here:
//  * the claim is a 64-bit agent-scope CAS; the row is written only by the
//    winner, after the CAS returned (control dependency);
//  * row words are written and read with agent-scope atomic accesses, which
//    are coherent across the XCDs' L2 caches (no write-back or invalidate of
//    whole caches is needed for them);
//  * the publisher waits for its row stores to complete (vmcnt(0)) before
//    storing DONE; a reader issues its row loads only after its load of the
//    slot returned DONE.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lhs {

constexpr uint64_t kOcc = 1ull << 63;
constexpr uint64_t kDone = 1ull << 62;
constexpr uint64_t kMemoMask = kDone - 1;
constexpr uint32_t kLineSlots = 16;          // default line: 128 bytes of 8-byte slots
constexpr uint32_t kNoSlot = 0xFFFFFFFFu;
constexpr uint32_t kSpinLimit = 1u << 22;    // bound on one wait (ESTALL)

enum : uint32_t { kNew = 0, kSeen = 1, kFull = 2, kStall = 3 };

// Counters and sticky error kept in device memory per table.
struct DevStatus {
    uint32_t error;          // first device error (lhs_status), 0 = none
    uint32_t pad;
    unsigned long long wait_hits;
    unsigned long long cas_failures;
    unsigned long long lines;   // lines probed (only while counted, see TableView::flags)
    unsigned long long merged;  // successors merged into an equal one of their pass (counted)
};

// A batched find-or-put has up to a million wavefronts, and almost every one
// has a wait or a lost claim to report when a call's rows repeat.  On one
// address such additions are served one after the other, some tens of
// millions a second: they were most of the time of a call whose rows repeat.
// So find-or-put adds to one of kStripes lines behind the table's status, by
// workgroup, and read_status sums them; an expansion's workgroups add up in
// LDS first.  A call of 2^18 rows of 16 words, half of them repeats, into
// 2^20 slots: 98 us on one address, 42 us striped; 2^20 rows of 8 words into
// 2^22 slots 224 and 90 us.
struct alignas(128) CounterLine {
    unsigned long long waits, cas_failures, lines;
};
constexpr uint32_t kStripes = 64;
struct TableStatus {
    DevStatus st;
    CounterLine stripe[kStripes];
};

// TableView::flags: counters to keep, and how expansions merge equal
// successors of a pass (expand_tile)
enum : uint32_t { kCountLines = 1, kCountMerged = 2, kNoMerge = 4, kNarrowTags = 8 };

// Per-lane event counts, reduced per wavefront before touching DevStatus.
struct LaneCounters {
    uint32_t waits = 0;
    uint32_t cas_failures = 0;
    uint32_t lines = 0;
    uint32_t merged = 0;
};

// Probe sequence across lines (after the home line's walk).
enum : uint32_t { kProbeDouble = 0, kProbeLinear = 1, kProbeQuadratic = 2 };

struct TableView {
    uint64_t *bucket;
    uint32_t *data;
    uint64_t seed;
    uint32_t W;
    uint32_t line_mask;      // lines - 1
    uint32_t max_rounds;     // lines probed before EFULL
    uint32_t probe;          // kProbe*
    DevStatus *status;
    // BFS with predecessor records (else null): parent[slot] = the slot the
    // state was first generated from; dead_rec = [count, slots of the first
    // kDeadRecord deadlock states expanded]
    uint32_t *parent;
    uint32_t *dead_rec;
    uint32_t flags;          // kCount*, kNoMerge, kNarrowTags
};
constexpr uint32_t kDeadRecord = 1024;

// log2 of the line width in slots (8, 16 or 32).
template <uint32_t LS>
__host__ __device__ constexpr uint32_t line_shift() {
    static_assert(LS == 8 || LS == 16 || LS == 32, "line slots");
    return LS == 8 ? 3u : (LS == 16 ? 4u : 5u);
}

// Line-to-line step of a vector's probe sequence.  Double hashing: a
// constant odd step from the hash's high half; linear: the next line;
// quadratic: the k-th move goes k lines on (the lines visited are line0 +
// k(k+1)/2).  On 2^n lines each sequence visits every line once in its first
// 2^n rounds.
__device__ __forceinline__ uint32_t probe_step(uint64_t h, uint32_t probe) {
    return probe == kProbeLinear ? 1u : ((uint32_t)(h >> 32) | 1u);
}
__device__ __forceinline__ uint32_t next_line(uint32_t line, uint32_t rounds_done, uint32_t step,
                                              uint32_t probe, uint32_t line_mask) {
    return (line + (probe == kProbeQuadratic ? rounds_done : step)) & line_mask;
}

__device__ __forceinline__ uint32_t mbcnt(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// The lane number, recomputed where it is asked for: what is derived from it
// then lives where it is used, instead of being hoisted out of the loops
// around and spilled there.
__device__ __forceinline__ uint32_t fresh_lane() {
    uint32_t l = __lane_id();
    asm volatile("" : "+v"(l));
    return l;
}

// Inclusive prefix sum over the wavefront (all 64 lanes active): the lanes of
// a row of 16 by shifts, then the row sums carried on.  Moves between lanes
// inside the vector unit take a few cycles; through LDS (shuffles) each step
// costs about 130, and a tile has some twenty of them.
template <int Ctrl, int Rows>
__device__ __forceinline__ uint32_t lane_move(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, Ctrl, Rows, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t x) {
    x += lane_move<0x111, 0xF>(x);   // from 1, 2, 4 and 8 lanes below in the row
    x += lane_move<0x112, 0xF>(x);
    x += lane_move<0x114, 0xF>(x);
    x += lane_move<0x118, 0xF>(x);
    x += lane_move<0x142, 0xA>(x);   // lane 15 of the row below, into rows 1 and 3
    x += lane_move<0x143, 0xC>(x);   // lane 31, into rows 2 and 3
    return x;
}

// Sum over the wavefront (all 64 lanes active); lane-uniform result.
__device__ __forceinline__ uint32_t wave_sum(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_incl(x), 63);
}

// ---- coherent (agent-scope) accesses --------------------------------------
__device__ __forceinline__ uint64_t ld_coherent(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t ld_coherent(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld_coherent(const unsigned long long *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_coherent(unsigned long long *p, unsigned long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_coherent(uint64_t *p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_coherent(uint32_t *p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Wait until this wavefront's outstanding vector memory operations completed
// (s_waitcnt vmcnt(0)); the signal fences keep the compiler from moving
// memory accesses across it.
__device__ __forceinline__ void wait_vm_complete() {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}
// 16 bytes of a slot line: a plain load, or (CL) two coherent 8-byte loads,
// for callers whose tables may have been emptied while they run (another
// XCD's cache can still hold the line as it was before).
template <bool CL>
__device__ __forceinline__ uint4 ld_line16(const uint4 *p) {
    if constexpr (CL) {
        const uint64_t *q = reinterpret_cast<const uint64_t *>(p);
        const uint64_t a = ld_coherent(q), b = ld_coherent(q + 1);
        return make_uint4((uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32));
    } else {
        return *p;
    }
}

// Compiler-level acquire after observing DONE (the hardware already orders
// the dependent loads after the observed load).
__device__ __forceinline__ void after_done_observed() {
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

__device__ __forceinline__ uint64_t rotl64(uint64_t x, int r) {
    return (x << r) | (x >> (64 - r));
}

// Vectors that also give four words at a time as the bytes of one (get4).
template <class Vec>
constexpr bool kByteWords = false;

// 64-bit vector hash: MurmurHash3 x64 block mixing over 64-bit pairs of
// words, closed by its fmix64 finaliser (A. Appleby, MurmurHash3, public
// domain).  `Vec` provides get(i) for word i.
template <class Vec>
__device__ __forceinline__ uint64_t hash_vec(const Vec &v, uint32_t W, uint64_t seed) {
    const uint64_t c1 = 0x87c37b91114253d5ull, c2 = 0x4cf5ad432745937full;
    uint64_t h = seed;
    uint32_t i = 0;
    // four pairs at a time: their words are read and scrambled independently,
    // only the short mixing into h is a chain
    for (; i + 8 <= W; i += 8) {
        uint32_t w[8];
        uint64_t k[4];
        if constexpr (kByteWords<Vec>) {
            const uint32_t a = v.get4(i), b = v.get4(i + 4);
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                w[j] = (a >> (8 * j)) & 0xFFu;
                w[4 + j] = (b >> (8 * j)) & 0xFFu;
            }
        } else {
#pragma unroll
            for (uint32_t j = 0; j < 8; ++j)
                w[j] = v.get(i + j);
        }
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j)
            k[j] = rotl64(((uint64_t)w[2 * j] | ((uint64_t)w[2 * j + 1] << 32)) * c1, 31) * c2;
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
            h ^= k[j];
            h = rotl64(h, 27);
            h = h * 5 + 0x52dce729ull;
        }
    }
    for (; i + 1 < W; i += 2) {
        uint64_t k = (uint64_t)v.get(i) | ((uint64_t)v.get(i + 1) << 32);
        k *= c1;
        k = rotl64(k, 31);
        k *= c2;
        h ^= k;
        h = rotl64(h, 27);
        h = h * 5 + 0x52dce729ull;
    }
    if (i < W) {
        uint64_t k = v.get(i);
        k *= c1;
        k = rotl64(k, 31);
        k *= c2;
        h ^= k;
    }
    h ^= (uint64_t)W * 4u;
    h ^= h >> 33;
    h *= 0xff51afd7ed558ccdull;
    h ^= h >> 33;
    h *= 0xc4ceb9fe1a85ec53ull;
    h ^= h >> 33;
    return h;
}

// Clear a table's status and striped counters (a workgroup of at least
// kStripes threads).
__device__ __forceinline__ void zero_status(TableStatus *ts) {
    if (threadIdx.x == 0)
        ts->st = DevStatus{};
    if (threadIdx.x < kStripes)
        ts->stripe[threadIdx.x] = CounterLine{};
}

__device__ __forceinline__ void set_error(DevStatus *st, uint32_t code) {
    atomicCAS(&st->error, 0u, code);
}

// rotate an LS-bit mask right by r (bit k of the result = bit (k + r) mod LS)
template <uint32_t LS>
__device__ __forceinline__ uint32_t rotr_line(uint32_t m, uint32_t r) {
    if constexpr (LS == 32)
        return __builtin_rotateright32(m, r);
    else
        return ((m >> r) | (m << (LS - r))) & ((1u << LS) - 1u);
}

// Spread the low 16 bits of x so that bit i lands on bit 2i.
__device__ __forceinline__ uint32_t spread2(uint32_t x) {
    x = (x | (x << 8)) & 0x00FF00FFu;
    x = (x | (x << 4)) & 0x0F0F0F0Fu;
    x = (x | (x << 2)) & 0x33333333u;
    return (x | (x << 1)) & 0x55555555u;
}

// Lane geometry of a group of G consecutive lanes of a wavefront.
template <int G>
struct Group {
    uint32_t sub, gbase;
    __device__ __forceinline__ Group() {
        const uint32_t lane = __lane_id();
        sub = lane & (G - 1);
        gbase = lane - sub;
    }
    __device__ __forceinline__ bool leader() const { return sub == 0; }
    // this group's G bits of a wavefront ballot
    __device__ __forceinline__ uint32_t bits(uint64_t ballot) const {
        return (uint32_t)(ballot >> gbase) & (uint32_t)((1ull << G) - 1);
    }
    __device__ __forceinline__ bool all(bool x) const {
        if constexpr (G == 1)
            return x;
        return bits(__ballot(x)) == (uint32_t)((1ull << G) - 1);
    }
    __device__ __forceinline__ uint64_t from_leader(uint64_t v) const {
        if constexpr (G == 1)
            return v;
        const uint32_t lo = __shfl((uint32_t)v, (int)gbase, 64);
        const uint32_t hi = __shfl((uint32_t)(v >> 32), (int)gbase, 64);
        return ((uint64_t)hi << 32) | lo;
    }
};

// A lane's part of one line of LS slots, loaded by a group of G lanes.  The
// line is LS/2 16-byte chunks (two slots each); lane `sub` loads chunks sub,
// sub + G, ..., so every load instruction of the group covers one contiguous
// 16*G-byte segment of the line.  With G >= LS every lane below LS loads one
// slot and the others only take part in the ballots.
template <int G, uint32_t LS>
struct LinePart {
    static constexpr uint32_t SPL = LS / G;               // slots per lane
    static constexpr uint32_t Q = SPL <= 1 ? 1 : SPL / 2; // chunks per lane
    uint4 x[Q];
};

template <int G, uint32_t LS, bool CL = false>
__device__ __forceinline__ LinePart<G, LS> load_line(const Group<G> &g, const uint64_t *line_ptr) {
    using P = LinePart<G, LS>;
    P p;
    if constexpr (P::SPL <= 1) {
        const uint64_t *q = line_ptr + ((uint32_t)G == LS ? g.sub : min(g.sub, LS - 1));
        const uint64_t s0 = CL ? ld_coherent(q) : *q;
        p.x[0] = make_uint4((uint32_t)s0, (uint32_t)(s0 >> 32), 0u, 0u);
    } else {
#pragma unroll
        for (uint32_t q = 0; q < P::Q; ++q)
            p.x[q] = ld_line16<CL>(reinterpret_cast<const uint4 *>(line_ptr) + q * G + g.sub);
    }
    return p;
}

// Masks of a loaded line's empty slots, of slots whose memo equals `memo`
// (any status) and of done slots, bit i = slot i of the line.
template <int G, uint32_t LS>
__device__ __forceinline__ void line_masks(const Group<G> &g, const LinePart<G, LS> &p, uint64_t memo,
                                           uint32_t &empty, uint32_t &match, uint32_t &done) {
    using P = LinePart<G, LS>;
    uint32_t e = 0, m = 0, d = 0;
    if constexpr (P::SPL <= 1) {
        const bool own = (uint32_t)G == LS || g.sub < LS;
        const uint64_t s0 = ((uint64_t)p.x[0].y << 32) | p.x[0].x;
        constexpr uint32_t lm = LS == 32 ? 0xFFFFFFFFu : (1u << LS) - 1u;
        e = g.bits(__ballot(own && s0 == 0)) & lm;
        m = g.bits(__ballot(own && (s0 & ~kDone) == memo)) & lm;
        d = g.bits(__ballot(own && (s0 & kDone))) & lm;
    } else {
#pragma unroll
        for (uint32_t q = 0; q < P::Q; ++q) {
            const uint64_t s0 = ((uint64_t)p.x[q].y << 32) | p.x[q].x;
            const uint64_t s1 = ((uint64_t)p.x[q].w << 32) | p.x[q].z;
            if constexpr (G == 1) {
                e |= ((uint32_t)(s0 == 0) | ((uint32_t)(s1 == 0) << 1)) << (2 * q);
                m |= ((uint32_t)((s0 & ~kDone) == memo) | ((uint32_t)((s1 & ~kDone) == memo) << 1))
                     << (2 * q);
                d |= (((uint32_t)(s0 >> 62) & 1u) | (((uint32_t)(s1 >> 62) & 1u) << 1)) << (2 * q);
            } else {
                // chunk q*G + sub holds slots 2(q*G + sub) and 2(q*G + sub) + 1
                e |= spread2(g.bits(__ballot(s0 == 0))) << (2 * q * G);
                e |= spread2(g.bits(__ballot(s1 == 0))) << (2 * q * G + 1);
                m |= spread2(g.bits(__ballot((s0 & ~kDone) == memo))) << (2 * q * G);
                m |= spread2(g.bits(__ballot((s1 & ~kDone) == memo))) << (2 * q * G + 1);
                d |= spread2(g.bits(__ballot((s0 & kDone) != 0))) << (2 * q * G);
                d |= spread2(g.bits(__ballot((s1 & kDone) != 0))) << (2 * q * G + 1);
            }
        }
    }
    empty = e;
    match = m;
    done = d;
}

// The home line of a vector with hash h.
template <uint32_t LS>
__device__ __forceinline__ uint32_t home_line(const TableView &t, uint64_t h) {
    return (uint32_t)(h >> line_shift<LS>()) & t.line_mask;
}

// Row write by the group: 64-bit coherent stores when W is even (rows are
// 8-byte aligned), 32-bit otherwise; lane `sub` takes every G-th piece.
template <int G, class Vec>
__device__ __forceinline__ void write_row(const Group<G> &g, uint32_t *row, const Vec &v, uint32_t W) {
    if ((W & 1u) == 0) {
        uint64_t *r2 = reinterpret_cast<uint64_t *>(row);
        for (uint32_t j = g.sub; j < W / 2; j += G)
            st_coherent(r2 + j, (uint64_t)v.get(2 * j) | ((uint64_t)v.get(2 * j + 1) << 32));
    } else {
        for (uint32_t i = g.sub; i < W; i += G)
            st_coherent(row + i, v.get(i));
    }
}

// Row compare by the group, up to B pieces per lane in flight at once
// (pieces past the row's end are read as its last one).
template <int G, uint32_t B, class Vec>
__device__ __forceinline__ bool row_equals_by(const Group<G> &g, const uint32_t *row, const Vec &v, uint32_t W) {
    uint32_t diff = 0;
    if ((W & 1u) == 0) {
        const uint64_t *r2 = reinterpret_cast<const uint64_t *>(row);
        const uint32_t last = W / 2 - 1;
        for (uint32_t j0 = g.sub; j0 <= last; j0 += B * G) {
            uint64_t x[B];
#pragma unroll
            for (uint32_t k = 0; k < B; ++k)
                x[k] = ld_coherent(r2 + min(j0 + k * G, last));
#pragma unroll
            for (uint32_t k = 0; k < B; ++k) {
                const uint32_t j = min(j0 + k * G, last);
                diff |= ((uint32_t)x[k] ^ v.get(2 * j)) | ((uint32_t)(x[k] >> 32) ^ v.get(2 * j + 1));
            }
        }
    } else {
        const uint32_t last = W - 1;
        for (uint32_t j0 = g.sub; j0 <= last; j0 += B * G) {
            uint32_t x[B];
#pragma unroll
            for (uint32_t k = 0; k < B; ++k)
                x[k] = ld_coherent(row + min(j0 + k * G, last));
#pragma unroll
            for (uint32_t k = 0; k < B; ++k)
                diff |= x[k] ^ v.get(min(j0 + k * G, last));
        }
    }
    return g.all(diff == 0);
}
template <int G, class Vec>
__device__ __forceinline__ bool row_equals(const Group<G> &g, const uint32_t *row, const Vec &v, uint32_t W) {
    if constexpr (G == 1)
        return row_equals_by<G, 4>(g, row, v, W);
    else
        return ((W & 1u) ? W : W / 2) <= G ? row_equals_by<G, 1>(g, row, v, W) : row_equals_by<G, 2>(g, row, v, W);
}

// One find-or-put per group of G lanes (G = 1, 4, 8 or 16) on a table of
// LS-slot lines (LS = 8, 16 or 32: 64, 128 or 256 bytes).
//
// All lanes of the wavefront call this together; `active`, `v` and `h` are
// uniform within a group, and every decision below is taken from
// group-uniform values, so the G lanes of a group always run the same path.
//
// The probe sequence of a vector with hash h: home line
// (h >> log2 LS) & line_mask, start slot h & (LS-1) inside it; the line is
// examined in walk order start, start+1, ..., wrapping inside the line
// (Algorithm 4 with the start offset read as the line base); after a line,
// the next line follows the table's probe sequence (probe_step/next_line:
// double hashing by default), which visits distinct lines until every line
// was seen.  After max_rounds lines the operation reports EFULL.
//
// Per line one snapshot is taken.  Candidates are, in walk order, the
// snapshot's empty slots and the slots whose memo equals ours.  Slots that
// are claimed with another memo are skipped: they are immutable.
//  - empty candidate: the group leader CASes 0 -> OCC|memo.  Won: the group
//    writes the row, waits for the stores, and the leader stores
//    OCC|DONE|memo; result "new".  Lost: the CAS returned the slot's value;
//    if its memo is ours it becomes a match candidate, otherwise walk on.
//  - match candidate: unless the snapshot (or the failed CAS) already showed
//    DONE, load the slot until DONE (a bounded wait, the paper's write-busy
//    "lock"); then compare the stored row; equal means "seen", otherwise walk
//    on.  DONE never goes away, and the row loads are issued after it was
//    observed.
//
// SIMT forward progress: every loop iteration runs the claim phase (CAS,
// row write, publish) for all lanes before the wait phase of any lane, and
// nothing waits between a claim and its publish.  A group that waits on a
// slot claimed by a group of its own wavefront therefore finds it already
// published; a claim made by another wavefront is published without that
// wavefront waiting on anything first.
//
// `first` is the home line, loaded by the caller: a caller with several
// operations loads the next one's while this one runs.
template <int G, uint32_t LS, class Vec, bool CL = false>
__device__ __forceinline__ void find_or_put(const TableView &t, const Vec &v, uint64_t h, LinePart<G, LS> first,
                                            bool active, uint32_t &out_slot, uint32_t &out_code,
                                            LaneCounters &cnt) {
    const Group<G> g;
    const uint64_t memo = kOcc | (h & kMemoMask);
    const uint32_t start = (uint32_t)h & (LS - 1);
    const uint32_t step = probe_step(h, t.probe);
    uint32_t line = home_line<LS>(t, h);
    uint32_t rounds = 0;
    uint32_t cand = 0, empty = 0, donem = 0;  // walk-ordered: bit k <-> slot start+k (mod LS)
    bool have_line = false;
    out_slot = kNoSlot;
    out_code = kFull;
    if (!active)
        return;

    while (true) {
        if (!have_line) {
            if (rounds == t.max_rounds) {
                out_code = kFull;
                if (g.leader())
                    set_error(t.status, 3u /* LHS_EFULL */);
                break;
            }
            if (rounds)
                first = load_line<G, LS, CL>(g, t.bucket + (uint64_t)line * LS);
            uint32_t e, m, d;
            line_masks<G, LS>(g, first, memo, e, m, d);
            empty = rotr_line<LS>(e, start);
            cand = rotr_line<LS>(e | m, start);
            donem = rotr_line<LS>(d, start);
            have_line = true;
            cnt.lines += g.leader();
        }
        if (cand == 0) {
            have_line = false;
            ++rounds;
            line = next_line(line, rounds, step, t.probe, t.line_mask);
            continue;
        }
        const uint32_t k = __builtin_ctz(cand);
        cand &= cand - 1;
        const uint32_t slot = line * LS + ((start + k) & (LS - 1));
        uint64_t *bp = t.bucket + slot;
        uint32_t *row = t.data + (uint64_t)slot * t.W;
        bool match = ((empty >> k) & 1u) == 0;
        bool known_done = (donem >> k) & 1u;
        bool finished = false;

        // ---- claim phase ------------------------------------------------
        if (!match) {
            uint64_t old = 0;
            if (g.leader())
                __hip_atomic_compare_exchange_strong(bp, &old, memo, __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            old = g.from_leader(old);
            if (old == 0) {
                write_row<G>(g, row, v, t.W);
                wait_vm_complete();
                if (g.leader())
                    st_coherent(bp, memo | kDone);
                out_slot = slot;
                out_code = kNew;
                finished = true;
            } else {
                cnt.cas_failures += g.leader();
                match = (old & ~kDone) == memo;
                known_done = (old & kDone) != 0;
            }
        }
        // ---- wait + compare phase --------------------------------------
        if (match && !finished) {
            uint64_t cur = known_done ? kDone : ld_coherent(bp);
            if (!(cur & kDone)) {
                cnt.waits += g.leader();
                uint32_t spins = 0;
                while (!(cur & kDone) && ++spins < kSpinLimit) {
                    __builtin_amdgcn_s_sleep(2);
                    cur = ld_coherent(bp);
                }
            }
            if (!(cur & kDone)) {
                out_code = kStall;
                if (g.leader())
                    set_error(t.status, 4u /* LHS_ESTALL */);
                finished = true;
            } else {
                after_done_observed();
                if (row_equals<G>(g, row, v, t.W)) {
                    out_slot = slot;
                    out_code = kSeen;
                    finished = true;
                }
            }
        }
        if (finished)
            break;
    }
}

template <int G, uint32_t LS, class Vec, bool CL = false>
__device__ __forceinline__ void find_or_put(const TableView &t, const Vec &v, uint64_t h, bool active,
                                            uint32_t &out_slot, uint32_t &out_code, LaneCounters &cnt) {
    const Group<G> g;
    find_or_put<G, LS, Vec, CL>(t, v, h, load_line<G, LS, CL>(g, t.bucket + (uint64_t)home_line<LS>(t, h) * LS),
                                active, out_slot, out_code, cnt);
}

// ---------------------------------------------------------------------------
// One operation per lane with wavefront-cooperative memory accesses.
//
// Every lane owns one find-or-put (64 operations in flight per wavefront),
// but the random 128-byte slot lines and the vector rows are moved by the
// whole wavefront: the lanes that need a line (or a row) this iteration are
// compacted into a list in LDS, and LS/2 lanes serve each listed line (16
// bytes each, one coalesced access per line), eight lanes each row (8 bytes
// each).  Results
// come back through the same per-wavefront LDS area.  The helpers need the
// owner's vector: `Vec` has a two-word descriptor any lane can decode.

template <uint32_t LS>
struct WaveScratch {         // one per wavefront, in LDS
    uint64_t key[64];        // memo per rank (line snapshots)
    uint32_t idx[64];        // listed line / slot per rank
    uint32_t aux[64];        // second word (row descriptor y)
    uint32_t desc[64];       // row descriptor x per rank
    uint8_t res[64 * (LS / 2 > 8 ? LS / 2 : 8)];   // per (rank, helper lane) result bits
};

__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The three cooperative accesses below move up to 64 random lines or rows
// for a wavefront.  What bounds them is the latency of a random access, so
// each issues all its loads before it uses the first.  A lane without an
// entry of its own reads the list's last entry again (the same line, in
// cache) instead of branching around its load: a load under a divergent
// branch is waited for before the next one is issued, which made a snapshot
// of 64 lines four round trips and a compare of 64 rows eight.  Measured with
// the loads branched around and together: the 12-process search to 2^27
// states 24.6 and 22.6 ms, the 64-model batch 11.3 and 10.3 ms; a table of
// 2^28 slots built from 2^26 rows of 16 words, which HBM traffic bounds, 5.48
// and 5.40 ms.

// One part of a line snapshot: the lines of ranks [0, nn) by NQ load
// instructions of LPQ lines each.
template <uint32_t LS, bool CL, uint32_t NQ>
__device__ __forceinline__ void coop_line_part(WaveScratch<LS> *ws, const uint64_t *bucket, uint32_t nn) {
    constexpr uint32_t C = LS / 2, CS = line_shift<LS>() - 1, LPQ = 64 / C;
    const uint32_t lane = fresh_lane(), c = lane & (C - 1);
    uint4 x[NQ];
    uint32_t r[NQ];
#pragma unroll
    for (uint32_t q = 0; q < NQ; ++q) {
        r[q] = min(q * LPQ + (lane >> CS), nn - 1);
        x[q] = ld_line16<CL>(reinterpret_cast<const uint4 *>(bucket + (uint64_t)ws->idx[r[q]] * LS) + c);
    }
#pragma unroll
    for (uint32_t q = 0; q < NQ; ++q) {
        const uint64_t s0 = ((uint64_t)x[q].y << 32) | x[q].x;
        const uint64_t s1 = ((uint64_t)x[q].w << 32) | x[q].z;
        const uint64_t mk = ws->key[r[q]];
        const uint32_t b = (uint32_t)(s0 == 0) | ((uint32_t)(s1 == 0) << 1) |
                           ((uint32_t)((s0 & ~kDone) == mk) << 2) |
                           ((uint32_t)((s1 & ~kDone) == mk) << 3) |
                           ((uint32_t)(s0 >> 62) & 1u) << 4 | (((uint32_t)(s1 >> 62) & 1u) << 5);
        // lanes that repeat an entry may have read another state of its line;
        // either byte is a snapshot of the line's two slots
        ws->res[r[q] * C + c] = (uint8_t)b;
    }
}

// Masks (bit i = slot i of the line) of empty, memo-matching and done slots
// for every lane with `need`; other lanes only help.  Wavefront-uniform call
// with at least one such lane.  C = LS/2 helper lanes per line, 64/C lines
// per load instruction, C instructions (one when the lines fit it).
template <uint32_t LS, bool CL = false>
__device__ __forceinline__ void coop_line_masks(WaveScratch<LS> *ws, const uint64_t *bucket, bool need,
                                                uint32_t line, uint64_t memo, uint32_t &empty,
                                                uint32_t &match, uint32_t &done) {
    constexpr uint32_t C = LS / 2, LPQ = 64 / C;
    const uint64_t nmask = __ballot(need);
    const uint32_t nn = (uint32_t)__popcll(nmask);
    const uint32_t rank = mbcnt(nmask);
    if (need) {
        ws->idx[rank] = line;
        ws->key[rank] = memo;
    }
    wave_lds_sync();
    if (nn > LPQ)
        coop_line_part<LS, CL, C>(ws, bucket, nn);
    else
        coop_line_part<LS, CL, 1>(ws, bucket, nn);
    wave_lds_sync();
    if (need) {
        const uint32_t *r = reinterpret_cast<const uint32_t *>(ws->res) + rank * (C / 4);
        uint32_t e = 0, m = 0, d = 0;
#pragma unroll
        for (uint32_t k = 0; k < C; ++k) {
            const uint32_t b = (r[k >> 2] >> (8 * (k & 3))) & 0xFFu;
            e |= (b & 3u) << (2 * k);
            m |= ((b >> 2) & 3u) << (2 * k);
            d |= ((b >> 4) & 3u) << (2 * k);
        }
        empty = e;
        match = m;
        done = d;
    }
    wave_lds_sync();
}

// Write the rows of every lane with `go` (slot, descriptor); eight lanes per
// row, 64-bit coherent stores when W is even, 32-bit otherwise.
template <class Vec, class WS>
__device__ __forceinline__ void coop_write_rows(WS *ws, const uint32_t *smem, uint32_t *data,
                                                uint32_t W, bool go, uint32_t slot, uint2 d) {
    const uint32_t lane = fresh_lane();
    const uint64_t gm = __ballot(go);
    const uint32_t ng = (uint32_t)__popcll(gm);
    const uint32_t rank = mbcnt(gm);
    if (go) {
        ws->idx[rank] = slot;
        ws->desc[rank] = d.x;
        ws->aux[rank] = d.y;
    }
    wave_lds_sync();
    const uint32_t c = lane & 7u;
    // two rows per lane at a time: their reads from LDS overlap
    for (uint32_t i0 = 0; i0 < ng; i0 += 16) {
        uint32_t r[2], at[2];
        Vec v[2];
#pragma unroll
        for (uint32_t q = 0; q < 2; ++q) {
            r[q] = min(i0 + 8 * q + (lane >> 3), ng - 1);
            at[q] = ws->idx[r[q]];
            v[q] = Vec::decode(smem, make_uint2(ws->desc[r[q]], ws->aux[r[q]]));
        }
        if ((W & 1u) == 0) {
            for (uint32_t j = c; j < W / 2; j += 8) {
                uint64_t x[2];
#pragma unroll
                for (uint32_t q = 0; q < 2; ++q)
                    x[q] = (uint64_t)v[q].get(2 * j) | ((uint64_t)v[q].get(2 * j + 1) << 32);
#pragma unroll
                for (uint32_t q = 0; q < 2; ++q)
                    if (i0 + 8 * q + (lane >> 3) < ng)
                        st_coherent(reinterpret_cast<uint64_t *>(data + (uint64_t)at[q] * W) + j, x[q]);
            }
        } else {
            for (uint32_t j = c; j < W; j += 8) {
                uint32_t x[2];
#pragma unroll
                for (uint32_t q = 0; q < 2; ++q)
                    x[q] = v[q].get(j);
#pragma unroll
                for (uint32_t q = 0; q < 2; ++q)
                    if (i0 + 8 * q + (lane >> 3) < ng)
                        st_coherent(data + (uint64_t)at[q] * W + j, x[q]);
            }
        }
    }
    wave_lds_sync();
}

// One part of a row compare: ranks [i0, i0 + 8 * NB), eight lanes per row,
// NB loads in flight per lane; result byte 1 = this lane's pieces differ.
template <uint32_t NB, class Vec, class WS>
__device__ __forceinline__ void coop_rows_part(WS *ws, const uint32_t *smem, const uint32_t *data, uint32_t W,
                                               uint32_t i0, uint32_t ng) {
    const uint32_t lane = fresh_lane(), c = lane & 7u;
    uint32_t r[NB], slot[NB], diff[NB];
#pragma unroll
    for (uint32_t q = 0; q < NB; ++q) {
        r[q] = min(i0 + 8 * q + (lane >> 3), ng - 1);
        slot[q] = ws->idx[r[q]];
        diff[q] = 0;
    }
    if ((W & 1u) == 0) {
        for (uint32_t j0 = 0; j0 < W / 2; j0 += 8) {
            const uint32_t j = min(j0 + c, W / 2 - 1);   // past the end: the last piece again
            uint64_t x[NB];
#pragma unroll
            for (uint32_t q = 0; q < NB; ++q)
                x[q] = ld_coherent(reinterpret_cast<const uint64_t *>(data + (uint64_t)slot[q] * W) + j);
#pragma unroll
            for (uint32_t q = 0; q < NB; ++q) {
                const Vec v = Vec::decode(smem, make_uint2(ws->desc[r[q]], ws->aux[r[q]]));
                diff[q] |= ((uint32_t)x[q] ^ v.get(2 * j)) | ((uint32_t)(x[q] >> 32) ^ v.get(2 * j + 1));
            }
        }
    } else {
        for (uint32_t j0 = 0; j0 < W; j0 += 8) {
            const uint32_t j = min(j0 + c, W - 1);
            uint32_t x[NB];
#pragma unroll
            for (uint32_t q = 0; q < NB; ++q)
                x[q] = ld_coherent(data + (uint64_t)slot[q] * W + j);
#pragma unroll
            for (uint32_t q = 0; q < NB; ++q) {
                const Vec v = Vec::decode(smem, make_uint2(ws->desc[r[q]], ws->aux[r[q]]));
                diff[q] |= x[q] ^ v.get(j);
            }
        }
    }
#pragma unroll
    for (uint32_t q = 0; q < NB; ++q)
        ws->res[r[q] * 8 + c] = diff[q] != 0;   // lanes of one entry write the same byte
}

// Compare the stored rows of every lane with `go` against its vector;
// returns equality for those lanes.  Wavefront-uniform call with at least
// one such lane; same layout as coop_write_rows.
template <class Vec, class WS>
__device__ __forceinline__ bool coop_rows_equal(WS *ws, const uint32_t *smem,
                                                const uint32_t *data, uint32_t W, bool go,
                                                uint32_t slot, uint2 d) {
    const uint64_t gm = __ballot(go);
    const uint32_t ng = (uint32_t)__popcll(gm);
    const uint32_t rank = mbcnt(gm);
    if (go) {
        ws->idx[rank] = slot;
        ws->desc[rank] = d.x;
        ws->aux[rank] = d.y;
    }
    wave_lds_sync();
    for (uint32_t i0 = 0; i0 < ng; i0 += 32)
        coop_rows_part<4, Vec>(ws, smem, data, W, i0, ng);
    wave_lds_sync();
    bool eq = false;
    if (go) {
        const uint2 r = reinterpret_cast<const uint2 *>(ws->res)[rank];
        eq = (r.x | r.y) == 0;
    }
    wave_lds_sync();
    return eq;
}

// One find-or-put per lane, memory moved cooperatively (see above).  The
// probe sequence, walk order, claim/publish protocol and the SIMT
// forward-progress structure (claim phase, then publish, then waits, in every
// iteration) are those of the group variant.  Additionally a match candidate
// whose snapshot (or failed CAS) already showed DONE is compared without
// re-reading its slot: DONE never goes away, and the row loads are coherent
// and issued after that observation completed.
//
// All 64 lanes must call this together (inactive lanes only help).  `d` is
// the lane's vector descriptor (Vec::decode(smem, d) rebuilds it in any lane).
template <uint32_t LS, class Vec, bool CL = false>
__device__ __forceinline__ void find_or_put_wave(const TableView &t, WaveScratch<LS> *ws,
                                                 const uint32_t *smem, uint2 d, uint64_t h,
                                                 bool active, uint32_t &out_slot,
                                                 uint32_t &out_code, LaneCounters &cnt) {
    const uint64_t memo = kOcc | (h & kMemoMask);
    const uint32_t start = (uint32_t)h & (LS - 1);
    const uint32_t step = probe_step(h, t.probe);
    uint32_t line = home_line<LS>(t, h);
    uint32_t rounds = 0, cand = 0, empty = 0, donem = 0, slot = 0;
    bool have_line = false, finished = !active;
    bool matched = false;   // `slot` holds a done match whose row is still to be compared
    out_slot = kNoSlot;
    out_code = kFull;

    while (__ballot(!finished)) {
        // ---- line snapshots for the lanes that need one -------------------
        if (!finished && !have_line && rounds == t.max_rounds) {
            out_code = kFull;
            set_error(t.status, 3u /* LHS_EFULL */);
            finished = true;
        }
        const bool need = !finished && !have_line;
        if (__ballot(need)) {
            uint32_t e = 0, m = 0, dn = 0;
            coop_line_masks<LS, CL>(ws, t.bucket, need, line, memo, e, m, dn);
            if (need) {
                empty = rotr_line<LS>(e, start);
                cand = rotr_line<LS>(e | m, start);
                donem = rotr_line<LS>(dn, start);
                have_line = true;
                ++cnt.lines;
            }
        }
        // ---- next candidate in walk order ---------------------------------
        uint32_t kind = 0;     // 0 none, 1 empty, 2 match
        bool known_done = matched;
        if (!finished) {
            if (matched) {
                kind = 2;
                matched = false;
            } else if (cand == 0) {
                have_line = false;
                ++rounds;
                line = next_line(line, rounds, step, t.probe, t.line_mask);
            } else {
                const uint32_t k = __builtin_ctz(cand);
                cand &= cand - 1;
                slot = line * LS + ((start + k) & (LS - 1));
                kind = ((empty >> k) & 1u) ? 1u : 2u;
                known_done = (donem >> k) & 1u;
            }
        }
        // ---- claim phase, with the compare of matches already seen DONE ----
        // Rows of slots seen DONE (in the snapshot, or by the last
        // iteration's claim or wait) are compared while the claims are in
        // flight: their loads are issued after that observation completed,
        // behind the acquire below, and DONE never goes away.
        const bool early = kind == 2 && known_done;
        const uint64_t em = __ballot(early);
        if (em)
            after_done_observed();
        bool won = false;
        uint64_t old = 0;
        if (kind == 1)
            __hip_atomic_compare_exchange_strong(t.bucket + slot, &old, memo, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (em) {
            const bool eq = coop_rows_equal<Vec>(ws, smem, t.data, t.W, early, slot, d);
            if (early) {
                if (eq) {
                    out_slot = slot;
                    out_code = kSeen;
                    finished = true;
                }
                kind = 0;   // a different row: the walk goes on
            }
        }
        if (kind == 1) {
            if (old == 0) {
                won = true;
            } else {
                ++cnt.cas_failures;
                kind = (old & ~kDone) == memo ? 2u : 0u;
                known_done = (old & kDone) != 0;
            }
        }
        if (__ballot(won)) {
            coop_write_rows<Vec>(ws, smem, t.data, t.W, won, slot, d);
            wait_vm_complete();
            if (won) {
                st_coherent(t.bucket + slot, memo | kDone);
                out_slot = slot;
                out_code = kNew;
                finished = true;
                kind = 0;
            }
        }
        // ---- wait phase (only slots not yet seen done); a match then goes
        // to the next iteration's compare -------------------------------------
        if (kind == 2) {
            matched = true;
            if (!known_done) {
                uint64_t cur = ld_coherent(t.bucket + slot);
                if (!(cur & kDone)) {
                    ++cnt.waits;
                    uint32_t spins = 0;
                    while (!(cur & kDone) && ++spins < kSpinLimit) {
                        __builtin_amdgcn_s_sleep(2);
                        cur = ld_coherent(t.bucket + slot);
                    }
                }
                if (!(cur & kDone)) {
                    out_code = kStall;
                    set_error(t.status, 4u /* LHS_ESTALL */);
                    finished = true;
                }
            }
        }
    }
}

// Add a wavefront's lane counters to the table's striped counters; t.status
// is a table's own (the first member of its TableStatus).  Must be called by
// all 64 lanes of the wavefront.  Lines probed are added only when the table
// counts them (on by request: see lhs_set_counters).
__device__ __forceinline__ void flush_counters_striped(const TableView &t, const LaneCounters &c) {
    if (!__ballot((c.waits | c.cas_failures) != 0) && !(t.flags & kCountLines))
        return;
    const uint32_t w = wave_sum(c.waits), f = wave_sum(c.cas_failures);
    const uint32_t l = (t.flags & kCountLines) ? wave_sum(c.lines) : 0u;
    if (__lane_id() == 0) {
        CounterLine &o = reinterpret_cast<TableStatus *>(t.status)->stripe[blockIdx.x & (kStripes - 1)];
        if (w)
            atomicAdd(&o.waits, (unsigned long long)w);
        if (f)
            atomicAdd(&o.cas_failures, (unsigned long long)f);
        if (l)
            atomicAdd(&o.lines, (unsigned long long)l);
    }
}

}  // namespace lhs
