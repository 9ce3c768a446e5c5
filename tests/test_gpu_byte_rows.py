"""Explorations whose LDS rows are bytes (every word of every reachable state
below 256) and those one value above, vs the CPU oracle.  The models are
small ones of the mix with their values and local states spread up to the
limit, so that the state space stays the same size."""
import numpy as np
import pytest

import gen
import oracle

from conftest import result_fields
from gpu_util import assert_same_set

pytestmark = pytest.mark.gpu

#: (seed, P, L, S, D): state widths 5, 6, 7 and 12 (every remainder of the words of a packed word)
SHAPES = {5: (0x2a695c3bc7d57ca9, 3, 17, 2, 6), 6: (0xd4ae2ddb56f8b6be, 2, 19, 4, 2),
          7: (0x29aedd51f42b1700, 4, 4, 3, 3), 12: (0xb9a2d1c40737eea9, 3, 24, 9, 5)}


@pytest.fixture(scope="module")
def lhs():
    import torch
    assert torch.cuda.is_available()
    import paper_1004_2772_amd
    return paper_1004_2772_amd


def spread(W, value_top, local_top):
    """The width-W model with its largest shared value renamed to value_top and
    its largest local state to local_top (0: left as they are)."""
    seed, P, L, S, D = SHAPES[W]
    m = gen.guarded_model(seed, P, L, S, D)
    trans, init = m.trans.copy(), m.init.copy()
    if value_top:
        for i in (2, 4):
            trans[..., i] = np.where(trans[..., i] == D - 1, value_top, trans[..., i])
        init[P:] = np.where(init[P:] == D - 1, value_top, init[P:])
    if local_top:
        wide = np.full((P, local_top + 1, m.K, 5), 0, dtype=np.uint32)
        wide[:, :L] = trans
        wide[:, local_top] = trans[:, L - 1]
        wide[..., 0] = np.where(wide[..., 0] == L - 1, local_top, wide[..., 0])
        init[:P] = np.where(init[:P] == L - 1, local_top, init[:P])
        trans, L = wide, local_top + 1
    return gen.Model(P, L, S, value_top + 1 if value_top else D, m.K, trans, init, 0,
                     f"spread({W},{value_top},{local_top})", seed)


CASES = [(W, v, l) for W in SHAPES for v, l in ((0, 0), (255, 0), (256, 0), (0, 255), (0, 256), (65535, 0))]


@pytest.mark.parametrize("W,value_top,local_top", CASES)
def test_explorations(lhs, W, value_top, local_top):
    m = spread(W, value_top, local_top)
    want = oracle.reach(m, keep_states=True)
    assert want.total > 1000
    print(f"\n[rows] {m.name}: {want.total} states", flush=True)
    for flags in (0, lhs.REACH_F_GRAPH, lhs.REACH_F_ASYNC):
        print(f"[rows] flags {flags}", flush=True)
        with lhs.Table(1 << 15, W) as t:
            got = lhs.reach_explore(m, table=t, flags=flags)
            if flags == lhs.REACH_F_ASYNC:
                assert (got.total, got.edges, got.deadlocks) == (want.total, want.edges, want.deadlocks)
            else:
                assert result_fields(got) == result_fields(want)
            assert_same_set(t.dump()[0], want.states, m.name)
    with lhs.Table(1 << 15, W) as t:
        assert result_fields(lhs.reach_explore_noalloc(m, t)) == result_fields(want)
        assert_same_set(t.dump()[0], want.states, m.name)


def test_initial_word(lhs):
    """The initial state's own words decide too."""
    for top in (255, 256, 0xFFFFFFFF):
        m = spread(6, 0, 0)
        m.init = m.init.copy()
        m.init[m.P + m.S - 1] = top
        want = oracle.reach(m, keep_states=True)
        print(f"\n[rows] initial word {top}: {want.total} states", flush=True)
        with lhs.Table(1 << 15, m.W) as t:
            assert result_fields(lhs.reach_explore(m, table=t)) == result_fields(want)
            assert_same_set(t.dump()[0], want.states, str(top))


@pytest.mark.parametrize("tops", [(0, 255), (255, 256), (256, 65535)])
def test_batch_and_server(lhs, tops):
    """Models of both kinds in one batch, and one after the other on a server
    whose launch has rows of bytes only."""
    models = [spread(W, v, 0) for W in SHAPES for v in tops]
    want = [oracle.reach(m) for m in models]
    print(f"\n[rows] batch and server, values up to {tops}", flush=True)
    for got, w in zip(lhs.reach_explore_batch(models, capacity=1 << 15), want):
        assert result_fields(got) == result_fields(w)
    with lhs.Server(capacity=1 << 15) as srv:
        order = [0, 2, 1, 3, 5, 4, 6, 7]
        tickets = [srv.submit(models[k]) for k in order]
        for k, t in zip(order, tickets):
            got, _ = srv.wait(t)
            assert result_fields(got) == result_fields(want[k]), models[k].name
