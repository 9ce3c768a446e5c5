"""Performance cases of the library: what a program does through its public entry points, small to large.

Four kinds of work:
  build    an empty table takes a stream of rows in a few find-or-put calls (each call's rows are
           distinct; of the later calls' rows a share is stored already);
  lookup   one find-or-put call of rows that are all stored;
  explore  reach_explore of a guarded model, by the host's level loop, graph-captured levels, without
           levels, with predecessor records, or through the entry point that allocates nothing;
  batch    reach_explore_batch over models of the mix;  serve  a burst of queries to the server.

A table's slot numbers depend on which of two competing rows came first, so a build returns its seen
flags; a lookup returns them with the slots where the table was filled one row at a time, else with
the value that the program keeps for each stored state, read through the slot.
"""
import random

import numpy as np
import torch

import paper_1004_2772_amd as lhs

NONE = 0xFFFFFFFF
M64 = (1 << 64) - 1

# The 64-model mix of the batch and the served workloads (K = 3):
# (seed, P, L, S, D, reachable states, edges).
MIX = [
    (0xb0ef305750c553c2, 12, 32, 9, 14, 8023, 19525), (0x20fc121b7d59a932, 15, 16, 15, 10, 8122, 25531),
    (0x365179065f460029, 15, 25, 12, 10, 1776, 5305), (0x2a695c3bc7d57ca9, 3, 17, 2, 6, 5787, 8629),
    (0x2c149ade04becb05, 15, 21, 15, 8, 1776, 4919), (0xb9a2d1c40737eea9, 3, 24, 9, 5, 4040, 7156),
    (0xaaf55d29c0973b42, 13, 8, 15, 6, 33545, 110272), (0xe11eac1ce8c8a436, 14, 9, 8, 11, 2437, 4582),
    (0x3444281485e3db3b, 10, 31, 15, 8, 4485, 12195), (0x3b8d25caf17a9c55, 16, 7, 8, 8, 17621, 57888),
    (0x3f5d79553a79f169, 12, 14, 4, 15, 8045, 14556), (0x1516028f9202029b, 12, 27, 8, 12, 1104, 2331),
    (0x2ff774369e7b03ba, 15, 11, 16, 9, 15646, 58191), (0xef9bd7e5efd0b829, 12, 13, 11, 11, 1204, 3435),
    (0x8ab00e56fb0defc8, 8, 4, 2, 5, 580557, 2802979), (0xc80763a76da73163, 13, 24, 10, 9, 5398, 13114),
    (0x93df382f23aa1734, 7, 7, 12, 6, 15848, 66267), (0xf2df6fb56bad789b, 14, 9, 7, 14, 75559, 217339),
    (0xbadac311b63b1f85, 3, 12, 4, 3, 57414, 173647), (0x449e8e54ccb22c4c, 3, 16, 8, 2, 764224, 3421255),
    (0x7959f74fc0c5f0c7, 3, 22, 7, 2, 872076, 3906135), (0x67f0f5970e99f6bf, 3, 13, 7, 3, 969387, 2979694),
    (0x3864c47bd701e7d2, 7, 25, 3, 13, 2780, 4789), (0x29aedd51f42b1700, 4, 4, 3, 3, 5717, 23596),
    (0xff8068375f973dac, 6, 18, 4, 10, 10248, 16826), (0x4752a9a891ff29f2, 6, 32, 14, 5, 9307, 17799),
    (0x87bb4a9576f10c1c, 7, 18, 14, 4, 1798, 5829), (0x1a255235bc3651a7, 16, 27, 15, 10, 45799, 106575),
    (0x59e8a257089ee681, 11, 32, 15, 13, 1768, 6038), (0x2e61c2a1e2d20c4f, 10, 5, 12, 5, 69730, 363466),
    (0xd4ae2ddb56f8b6be, 2, 19, 4, 2, 3490, 10440), (0x3858d8a29a4d458f, 12, 23, 16, 9, 4616, 13816),
    (0x9a427beeda34aa34, 10, 19, 5, 14, 2147, 4171), (0xa5ec8a8d13acfb5, 3, 14, 4, 4, 32749, 73076),
    (0xfbbd4c9ac3dc3e20, 6, 4, 8, 2, 595088, 5334818), (0x9fb9ba0e43a085cc, 9, 12, 14, 5, 21200, 66978),
    (0x6f2ae02f25a7ae82, 2, 10, 5, 3, 3422, 7726), (0x634907d2a4f11326, 3, 32, 2, 3, 185943, 560773),
    (0x48548ddd8c821dba, 13, 29, 13, 7, 17492, 42896), (0x737152820136629f, 3, 32, 2, 4, 206157, 471651),
    (0x6453fec238ae67fe, 14, 21, 16, 7, 27945, 98168), (0x3c2394052ff04773, 3, 7, 7, 2, 21728, 98849),
    (0xccde02257c85cd9b, 5, 8, 3, 3, 477917, 2365751), (0x5f08300d2ac762db, 4, 8, 2, 4, 34310, 105394),
    (0xa7d6a0564c023e07, 4, 5, 13, 2, 753602, 4334513), (0x250844996fa304d0, 5, 5, 2, 3, 26282, 131554),
    (0xf15455504ef7bd10, 7, 4, 4, 6, 566498, 2212187), (0x9c9e0149b24dc4ae, 3, 21, 2, 2, 13101, 58378),
    (0x54bda2cbc8cde1fc, 15, 23, 13, 10, 17614, 43659), (0xa66b15cea0d812ff, 4, 13, 3, 4, 416697, 1168706),
    (0xb65bb1eb85244ac2, 5, 4, 15, 3, 20817, 86781), (0xee9c12e79eca2f4e, 16, 14, 12, 10, 22536, 67842),
    (0xc2682af9a1460dee, 13, 27, 10, 10, 18339, 57985), (0xeab2958ffdbfbe0d, 3, 32, 4, 2, 345971, 1548540),
    (0xb0a7f9e44a3c9407, 3, 29, 3, 3, 284721, 852535), (0xb79771617303059, 13, 19, 8, 11, 229090, 538707),
    (0x261af3419b25c3aa, 15, 19, 8, 15, 117211, 312746), (0x19eb2836f45cbfeb, 3, 30, 3, 5, 143008, 266258),
    (0x630776c99db1ee66, 5, 5, 12, 2, 786664, 5692557), (0xb8b31a5a986e10f6, 12, 7, 11, 8, 106465, 401350),
    (0x1b9c4068fafbb635, 2, 28, 11, 2, 484957, 1471625), (0x2dc18e6672668c2e, 4, 19, 3, 6, 758720, 1485707),
    (0x582dec4ce47590f7, 3, 25, 6, 2, 627398, 2816764), (0x86cf709dd9ac93ac, 2, 17, 10, 2, 133110, 399760),
]
# Single models: (seed, P, L, S, D, K, states, edges); the first is explored up to a cap of states
# (its space exceeds 2^27), the others to the end.
BIG = (0x2, 12, 16, 4, 10, 3, 123057326, 230333042)
WIDE = (78, 8, 6, 4, 4, 2, 32518299, 129457763)
MIDDLE = (77, 7, 6, 3, 4, 2, 1078377, 3999223)
DEEP = (0x2dc18e6672668c2e, 4, 19, 3, 6, 3, 758720, 1485707)
SMALL = (0x29aedd51f42b1700, 4, 4, 3, 3, 3, 5717, 23596)
WORDY = (0x630776c99db1ee66, 5, 5, 12, 2, 3, 786664, 5692557)
MODELS = {"big": BIG, "wide": WIDE, "middle": MIDDLE, "deep": DEEP, "small": SMALL, "wordy": WORDY}

FLAGS = {"host": 0, "graph": lhs.REACH_F_GRAPH, "async": lhs.REACH_F_ASYNC, "parents": lhs.REACH_F_PARENTS,
         "noalloc": 0}


def listed():
    return [
        # a few rows looked up in a small table: the latency of one call
        {"name": "lookup_few", "kind": "lookup", "W": 16, "n": 64, "log2": 14, "fill": 0.25, "tuned": True, "slots": True},
        # an ordinary call on the default table shape, an odd number of odd-width rows
        {"name": "lookup_odd", "kind": "lookup", "W": 5, "n": 30011, "log2": 18, "fill": 0.5, "tuned": False, "slots": False},
        # a nearly full table of the widest rows, read
        {"name": "lookup_full", "kind": "lookup", "W": 32, "n": 1000003, "log2": 22, "fill": 0.9, "tuned": True, "slots": False},
        # a small table built in a few calls
        {"name": "build_small", "kind": "build", "W": 8, "n": 120000, "log2": 20, "calls": 4, "seen": 0.5, "tuned": True},
        # an ordinary one, of odd width
        {"name": "build_middle", "kind": "build", "W": 13, "n": 4000001, "log2": 24, "calls": 3, "seen": 0.4, "tuned": True},
        # the benchmark's stream: 2^26 rows, nearly half of them repeats, into 2^28 slots
        {"name": "build_stream", "kind": "build", "W": 16, "n": 1 << 26, "log2": 28, "calls": 2, "seen": 0.9, "tuned": True},
        # a model of a few thousand states: the latency of a level
        {"name": "explore_small", "kind": "explore", "model": "small", "mode": "host", "cap": 0, "log2": 16},
        # a million states, the host's level loop
        {"name": "explore_middle", "kind": "explore", "model": "middle", "mode": "host", "cap": 0, "log2": 22},
        # the benchmark's search of the 12-process model up to 2^27 states
        {"name": "explore_big", "kind": "explore", "model": "big", "mode": "host", "cap": 1 << 27, "log2": 28},
        # exploration without level barriers, to the end
        {"name": "explore_async", "kind": "explore", "model": "wide", "mode": "async", "cap": 0, "log2": 26},
        # the 64-model mix in one call
        {"name": "batch_mix", "kind": "batch", "models": 64, "log2": 21},
        # a burst of queries at the server, all waited for
        {"name": "serve_burst", "kind": "serve", "queries": 96},
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["lookup", "lookup", "build", "build", "build", "explore", "explore", "explore", "batch", "serve"])
    if kind == "lookup":
        log2 = rng.randint(14, 25)
        W = rng.randint(1, 32)
        fill = rng.choice([0.125, 0.3, 0.5, 0.8, 0.95])
        return {"kind": kind, "W": W, "n": _log(rng, 16, min(1 << 22, int(fill * (1 << log2)))), "log2": log2,
                "fill": fill, "tuned": rng.random() < 0.7, "slots": False}
    if kind == "build":
        log2 = rng.randint(15, 26)
        calls = rng.randint(2, 6)
        n = _log(rng, 256, (1 << log2) // 2)
        return {"kind": kind, "W": rng.randint(1, 32), "n": n, "log2": log2, "calls": calls,
                "seen": rng.choice([0.1, 0.25, 0.5, 0.9]), "tuned": rng.random() < 0.7}
    if kind == "explore":
        mode = rng.choice(["host", "host", "graph", "async", "parents", "noalloc"])
        capped = ["big", "big", "wide", "wide"] if mode != "async" else []   # without levels a cap cuts anywhere
        model = rng.choice(capped + ["middle", "deep", "small", "wordy"])
        if model in ("big", "wide"):
            cap = _log(rng, 3000, 1 << (18 if mode == "noalloc" else 24))
            log2 = max(16, (4 * cap - 1).bit_length())
        else:
            cap = 0
            log2 = (16 if model == "small" else 21) + (0 if mode == "noalloc" else rng.randint(0, 2))
        return {"kind": kind, "model": model, "mode": mode, "cap": cap, "log2": log2}
    if kind == "batch":
        return {"kind": kind, "models": _log(rng, 2, 63), "log2": 21}
    return {"kind": kind, "queries": _log(rng, 1, 95)}


# ---- inputs -----------------------------------------------------------------

class Model:
    """P processes of L local states, S shared variables; trans [P, L, K, 5]."""

    def __init__(self, P, L, S, K, trans, init):
        self.P, self.L, self.S, self.K, self.trans, self.init, self.cap = P, L, S, K, trans, init, 0


def _guarded(seed, P, L, S, D, K):
    """The guarded model of a seed: per (process, local state, transition) five xorshift64 (13, 7, 17) words
    give target, guard variable and value, effect variable and value."""
    x, out = seed, np.empty((P * L * K, 5), dtype=np.uint32)
    for i in range(P * L * K):
        for j, m in enumerate((L, S, D, S, D)):
            x ^= (x << 13) & M64
            x ^= x >> 7
            x ^= (x << 17) & M64
            out[i, j] = x % m
    return Model(P, L, S, K, out.reshape(P, L, K, 5), np.zeros(P + S, dtype=np.uint32))


def _relabelled(m, rng):
    """The same model with the values of every process's local states renamed (the initial ones too)."""
    perm = np.array([rng.sample(range(m.L), m.L) for _ in range(m.P)], dtype=np.uint32)
    trans = np.empty_like(m.trans)
    for p in range(m.P):
        trans[p, perm[p]] = m.trans[p]
        trans[p, :, :, 0] = perm[p][trans[p, :, :, 0]]
    init = m.init.copy()
    init[:m.P] = [perm[p][m.init[p]] for p in range(m.P)]
    return Model(m.P, m.L, m.S, m.K, trans, init)


def _variant(m, cap, states, rng, table):
    """The model with some transitions' targets and guards drawn anew, such that it is another search of about
    the same size (with a cap: one that exceeds the cap, or 2^18 states)."""
    values = int(m.trans[..., 2].max()) + 1
    some = 4 if cap else 1
    base = lhs.reach_explore(m, cap=min(cap, 1 << 18), table=table)
    for _ in range(200):
        got = Model(m.P, m.L, m.S, m.K, m.trans.copy(), m.init)
        for _ in range(some):
            got.trans[rng.randrange(m.P), rng.randrange(m.L), rng.randrange(m.K), 0] = rng.randrange(m.L)
            got.trans[rng.randrange(m.P), rng.randrange(m.L), rng.randrange(m.K), 2] = rng.randrange(values)
        r = lhs.reach_explore(got, cap=min(cap, 1 << 18), table=table)
        if r.edges != base.edges and (r.capped or (not cap and 0.8 * states <= r.total <= 1.25 * states)):
            return got
    return m


def _rows(first, n, W, g):
    """n distinct random rows: word 0 is an odd multiple of the row's number."""
    out = torch.randint(-(1 << 31), (1 << 31) - 1, (n, W), dtype=torch.int32, device="cuda", generator=g)
    i = torch.arange(first, first + n, dtype=torch.int64, device="cuda")
    out[:, 0] = (((i * 0x9E3779B1 + 0x7F4A7C15) & 0xFFFFFFFF) - (1 << 31)).to(torch.int32)
    return out


def _table(case):
    if case["tuned"]:
        lhs.tune_load_default()
        return lhs.Table(1 << case["log2"], case["W"])
    return lhs.Table(1 << case["log2"], case["W"], lhs.config())


def _sizes(case):
    """(rows, new rows) of each call of a build."""
    n, k = case["n"], case["calls"]
    out = []
    for c in range(k):
        rows = n // k + (1 if c < n % k else 0)
        old = 0 if c == 0 else min(int(rows * case["seen"]), sum(x[1] for x in out))
        out.append((rows, rows - old))
    return out


def _stream(case, seed):
    """The rows of every call of a build, [n, W]: new ones, and some of the earlier calls', shuffled."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    sizes = _sizes(case)
    total = sum(x[1] for x in sizes)
    distinct = _rows(seed & 0xFFFFF, total, case["W"], g)
    out = torch.empty((case["n"], case["W"]), dtype=torch.int32, device="cuda")
    at = have = 0
    for rows, new in sizes:
        old = torch.randperm(have, device="cuda", generator=g)[:rows - new] if rows > new else torch.empty(0, dtype=torch.int64, device="cuda")
        pick = torch.cat([torch.arange(have, have + new, device="cuda"), old])
        pick = pick[torch.randperm(rows, device="cuda", generator=g)]
        torch.index_select(distinct, 0, pick, out=out[at:at + rows])
        at += rows
        have += new
    return out


_server = None


def _the_server():
    """The process's server (a program has one)."""
    global _server
    if _server is None:
        lhs.tune_load_default()
        _server = lhs.Server(budget_bytes=32 << 30, capacity=1 << 21)
    return _server


def prepare(case, seed):
    kind = case["kind"]
    rng = random.Random(seed)
    if kind == "build":
        states = _stream(case, seed)
        seen = torch.empty(case["n"], dtype=torch.uint8, device="cuda")
        cuts, at = [], 0
        for rows, _ in _sizes(case):
            cuts.append((states[at:at + rows], seen[at:at + rows]))
            at += rows
        return {"kind": kind, "table": _table(case), "cuts": cuts, "seen": seen}
    if kind == "lookup":
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        stored = int(case["fill"] * (1 << case["log2"]))
        rows = _rows(seed & 0xFFFFF, stored, case["W"], g)
        table = _table(case)
        seen = torch.empty(stored, dtype=torch.uint8, device="cuda")
        slot = torch.empty(stored, dtype=torch.int32, device="cuda")
        step = 1 if case["slots"] else max(1, stored // 64)
        for at in range(0, stored, step):
            table.find_or_put(rows[at:at + step], seen[at:at + step], slot[at:at + step])
        value = None
        if not case["slots"]:
            value = torch.zeros(1 << case["log2"], dtype=torch.int32, device="cuda")
            value[slot.long()] = torch.arange(stored, dtype=torch.int32, device="cuda")
        n = case["n"]
        ask = rows.index_select(0, torch.randint(0, stored, (n,), device="cuda", generator=g))
        return {"kind": kind, "table": table, "rows": ask, "value": value,
                "seen": torch.empty(n, dtype=torch.uint8, device="cuda"),
                "slot": torch.empty(n, dtype=torch.int32, device="cuda")}
    lhs.tune_load_default()
    if kind == "explore":
        m = MODELS[case["model"]]
        model = _guarded(*m[:6])
        table = lhs.Table(1 << case["log2"], model.P + model.S)
        model = _variant(model, case["cap"], m[6], rng, table)
        return {"kind": kind, "table": table, "model": model, "cap": case["cap"], "mode": case["mode"]}
    if kind == "batch":
        models = [_relabelled(_guarded(*x[:5], 3), rng) for x in rng.sample(_mix(case["models"]), case["models"])]
        tables = [lhs.Table(1 << case["log2"], m.P + m.S, lhs.config(8, "double", 0, 1)) for m in models]
        return {"kind": kind, "models": models, "tables": tables}
    mix = [_guarded(*x[:5], 3) for x in rng.sample(MIX, 16)]
    return {"kind": kind, "server": _the_server(), "models": [rng.choice(mix) for _ in range(case["queries"])]}


def _mix(n):
    """n models of the mix, spread over it."""
    return [MIX[(i * 64) // n] for i in range(n)]


# ---- one pass -----------------------------------------------------------------

LEVELS = 512   # more than any of these models has


def _levels(counts):
    return np.pad(np.array(counts, dtype=np.int64), (0, LEVELS - len(counts)))


def _counts(r):
    return {"states": r.total, "edges": r.edges, "deadlocks": r.deadlocks, "capped": r.capped,
            "levels": _levels(r.level_counts)}


def run(state):
    kind = state["kind"]
    if kind == "build":
        state["table"].clear()
        for rows, seen in state["cuts"]:
            state["table"].find_or_put(rows, seen)
        return {"seen": state["seen"]}
    if kind == "lookup":
        state["table"].find_or_put(state["rows"], state["seen"], state["slot"])
        if state["value"] is None:
            return {"seen": state["seen"], "slot": state["slot"]}
        return {"seen": state["seen"], "value": torch.index_select(state["value"], 0, state["slot"])}
    if kind == "explore":
        if state["mode"] == "noalloc":
            return _counts(lhs.reach_explore_noalloc(state["model"], state["table"], cap=state["cap"]))
        return _counts(lhs.reach_explore(state["model"], cap=state["cap"], table=state["table"],
                                         flags=FLAGS[state["mode"]]))
    if kind == "batch":
        got = lhs.reach_explore_batch(state["models"], tables=state["tables"])
    else:
        tickets = [state["server"].submit(m) for m in state["models"]]
        got = [state["server"].wait(t)[0] for t in tickets]
    return {"states": np.array([r.total for r in got], dtype=np.int64),
            "edges": np.array([r.edges for r in got], dtype=np.int64),
            "deadlocks": np.array([r.deadlocks for r in got], dtype=np.int64),
            "levels": np.stack([_levels(r.level_counts) for r in got])}


def work(case):
    """Bytes: inputs and outputs once, the cleared slots, one slot and one row per operation, and per
    expanded state its row read."""
    kind = case["kind"]
    if kind in ("build", "lookup"):
        n, row = case["n"], 4 * case["W"]
        per = row + 1 + 8 + row
        if kind == "build":
            return {"bytes": 8 * (1 << case["log2"]) + n * per, "flops": 0}
        return {"bytes": n * (per + (4 if case["slots"] else 12)), "flops": 0}
    if kind == "explore":
        m = MODELS[case["model"]]
        share = 1.0 if not case["cap"] else min(1.0, 0.6 * case["cap"] / m[6])
        n, e, row = m[6] * share, m[7] * share, 4 * (m[1] + m[3])
        return {"bytes": 8 * (1 << case["log2"]) + n * (2 * row + 8) + e * 8, "flops": 0}
    if kind == "batch":
        mix, slots = _mix(case["models"]), 8 * (1 << case["log2"])
    else:
        mix, slots = [MIX[(i * 64) // case["queries"] % 64] for i in range(case["queries"])], 8 * (1 << 21)
    return {"bytes": sum(slots + x[5] * (8 * (x[1] + x[3]) + 8) + x[6] * 8 for x in mix), "flops": 0}


# ---- the same, in plain torch and numpy ------------------------------------------

def _search(m, cap):
    """Breadth-first search over numbered rows, a level at a time."""
    base = [m.L] * m.P + [int(max(m.trans[..., 4].max(), m.init[m.P:].max(initial=0))) + 1] * m.S
    scale = [1]
    for b in base[:-1]:
        scale.append(scale[-1] * b)
    if scale[-1] * base[-1] >= 1 << 63:
        return None
    scale = np.array(scale, dtype=np.int64)
    known = np.array([int((m.init.astype(np.int64) * scale).sum())], dtype=np.int64)
    front, levels, edges, dead, capped = m.init.astype(np.int64)[None, :], [1], 0, 0, False
    while True:
        found, degree = [], np.zeros(len(front), dtype=np.int64)
        for p in range(m.P):
            for k in range(m.K):
                t = m.trans[p, front[:, p], k].astype(np.int64)
                on = front[np.arange(len(front)), m.P + t[:, 1]] == t[:, 2]
                degree += on
                nxt = front[on].copy()
                nxt[:, p] = t[on, 0]
                nxt[np.arange(len(nxt)), m.P + t[on, 3]] = t[on, 4]
                found.append(nxt)
        rows = np.concatenate(found)
        keys, first = np.unique(rows @ scale, return_index=True)
        at = np.minimum(np.searchsorted(known, keys), len(known) - 1)
        first = first[known[at] != keys]
        if cap and sum(levels) + len(first) > cap:
            capped = True
            break
        edges += int(degree.sum())
        dead += int((degree == 0).sum())
        if not len(first):
            break
        front = rows[first]
        known = np.union1d(known, front @ scale)
        levels.append(len(front))
    return {"states": sum(levels), "edges": edges, "deadlocks": dead, "capped": capped,
            "levels": _levels(levels)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "build":
        seen, at = torch.zeros(case["n"], dtype=torch.uint8), 0
        key = _stream(case, seed)[:, 0].long().cpu().numpy()    # word 0 tells rows apart
        order = np.argsort(key, kind="stable")
        again = np.concatenate([[False], key[order][1:] == key[order][:-1]])
        seen[torch.from_numpy(order[again])] = 1
        return {"seen": seen}
    if kind == "lookup":
        return {"seen": torch.ones(case["n"], dtype=torch.uint8), "slot" if case["slots"] else "value": None}
    if kind != "explore" or case["mode"] == "async" or (case["cap"] or MODELS[case["model"]][6]) > 200000:
        return None
    state = prepare(case, seed)
    return _search(state["model"], case["cap"])
