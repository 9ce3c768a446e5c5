"""How long an idle workgroup of a persistent launch waits for the others: the
bound is on the time without progress, so neither a slow error nor a long chain
of levels ends as a stall."""
import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lhs():
    import torch
    assert torch.cuda.is_available()
    import paper_1004_2772_amd as m
    return m


def box_model(dims):
    """One process per dimension that counts up to its end: prod(dims) states."""
    P, L = len(dims), max(dims)
    trans = np.zeros((P, L, 1, 5), dtype=np.uint32)
    for p, n in enumerate(dims):
        for l in range(L):
            trans[p, l, 0] = (l + 1, gen.NONE, 0, gen.NONE, 0) if l + 1 < n else (l, 0, 1, gen.NONE, 0)
    return gen.Model(P, L, 1, 1, 1, trans, np.zeros(P + 1, dtype=np.uint32), 0, f"box{dims}")


def counter_model(digits, top):
    """A counter of base-16 digits (shared variables) whose highest starts at
    `top`; the process is at the digit to increment: a chain of states."""
    L = digits + 1
    trans = np.zeros((1, L, 16, 5), dtype=np.uint32)
    for d in range(digits):
        for k in range(16):
            trans[0, d, k] = (0, d, k, d, k + 1) if k < 15 else (d + 1, d, 15, d, 0)
    trans[0, digits] = (digits, 0, 16, 0, 0)     # no value reaches 16: the end
    init = np.zeros(1 + digits, dtype=np.uint32)
    init[digits] = top
    return gen.Model(1, L, digits, 17, 16, trans, init, 0, f"counter{digits}:{top}")


def chain_length(digits, top):
    """States of counter_model: values from top * 16^(digits-1) on, and the
    process's steps to a higher digit, the last of which ends it."""
    n = top * 16 ** (digits - 1)
    end = 16 ** digits
    carries = sum(end // 16 ** d - n // 16 ** d for d in range(1, digits + 1))
    return end - n + carries


def test_served_overflow_of_a_large_table_ends_alone(lhs):
    """A query that overflows a table of 2^24 slots while few workgroups have
    work: its last operations probe 2^21 lines one after the other, seconds
    without a level finished.  It ends with LHS_EFULL, and the query beside it
    and the next one are served."""
    dims = (126, 269, 495)
    assert 0 < np.prod(dims) - (1 << 24) < 1000
    print(f"\n[idle] overflow of 2^24 slots by {np.prod(dims)} states", flush=True)
    with lhs.Server(capacity=1 << 24, cfg=lhs.config(8, "double", 0, 1)) as srv:
        bad = srv.submit(box_model(dims))
        good = srv.submit(counter_model(3, 0))
        with pytest.raises(lhs.LhsError) as e:
            srv.wait(bad)
        assert e.value.name == "LHS_EFULL"
        assert srv.wait(good)[0].total == chain_length(3, 0)
        assert srv.wait(srv.submit(gen.cyclic_model(2, 8)))[0].total == 64


def test_batch_long_chain(lhs):
    """A chain of 1.1 million one-state levels (about 9 s) stays with one
    workgroup, and all others are idle until its end."""
    m = counter_model(6, 15)
    n = chain_length(6, 15)
    print(f"\n[idle] chain of {n} levels", flush=True)
    r = lhs.reach_explore_batch([m], capacity=1 << 22, max_levels=1 << 22)[0]
    assert (r.total, r.n_levels, r.edges, r.deadlocks) == (n, n, n - 1, 1)
    assert r.level_counts == [1] * n


def test_served_overflow_costs_one_walk(lhs):
    """A query that overflows its table in a level that one workgroup runs
    alone.  The level is 78 states, four of which find no slot; the next would
    be 66 states, none of which does.  Each of those costs a probe of all 2^17
    lines, so the query has to end with the first level."""
    cap, dims = 1 << 20, (51, 91, 226)
    # the last levels of a box: 1, 3, 6, ... states from its far corner
    last = [k * (k + 1) // 2 for k in range(1, 13)]
    assert last[-2:] == [66, 78] and sum(last) - (np.prod(dims) - cap) == 74
    with lhs.Server(cfg=lhs.config(8, "double", 0, 1)) as srv, \
            lhs.Table(cap, 4, lhs.config(8, "double", 0, 1)) as t:
        t.set_counters(1)
        with pytest.raises(lhs.LhsError) as e:
            srv.wait(srv.submit(box_model(dims), table=t))
        assert e.value.name == "LHS_EFULL"
        lines = t.info()["lines_probed"]
    print(f"\n[idle] overflow of 2^20 slots: {lines} lines probed", flush=True)
    assert lines < 66 * (cap // 8)
