"""Levels run by the persistent level driver at the sizes where it changes
its ways: a level that stays with its workgroup or is handed out in tiles, a
buffer of new states that fills up in such a level, the room it needs below
the cap, more levels than one launch counts, levels too wide for it and back,
and more models than one poll sees."""
import numpy as np
import pytest

import gen
import oracle

from conftest import result_fields
from gpu_util import assert_same_set

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lhs():
    import torch
    assert torch.cuda.is_available()
    import paper_1004_2772_amd
    return paper_1004_2772_amd


def layered(sizes, K=16):
    """One process whose BFS levels have the given sizes: every state of a
    layer has K transitions into the next one, which cover it."""
    first = np.concatenate([[0], np.cumsum(sizes)])
    L = int(first[-1])
    trans = np.full((1, L, K, 5), gen.NONE, dtype=np.uint32)
    trans[..., 2] = 0
    trans[..., 4] = 0
    for d, n in enumerate(sizes):
        nxt, n_next = (first[d + 1], sizes[d + 1]) if d + 1 < len(sizes) else (first[d], n)
        assert n_next <= n * K
        j = np.arange(n * K).reshape(n, K)
        trans[0, first[d]:first[d] + n, :, 0] = nxt + j % n_next
    return gen.Model(1, L, 0, 1, K, trans, np.zeros(1, dtype=np.uint32), 0, f"layered{tuple(sizes)}", 0)


SIZES = {
    "around_solo": [1, 16, 95, 96, 97, 96, 98, 95, 1, 2, 32, 96, 97, 1],
    "around_tiles": [1, 16, 255, 256, 257, 512, 513, 31, 32, 33, 64, 65, 1],
    "spill": [1, 16, 96, 1536, 96, 1024, 64, 1024, 1025, 96, 1280, 90, 1440, 3],
    "wide_and_back": [1, 16, 200, 3000, 30000, 200, 9, 9, 9, 144, 2000, 12000, 70, 1],
}


@pytest.mark.parametrize("name", sorted(SIZES))
def test_level_sizes(lhs, name):
    m = layered(SIZES[name])
    want = oracle.reach(m, keep_states=True)
    assert want.level_counts == SIZES[name]
    print(f"\n[levels] {name}: {want.total} states", flush=True)
    with lhs.Table(1 << 18, 1) as t:
        assert result_fields(lhs.reach_explore(m, table=t)) == result_fields(want)
        assert_same_set(t.dump()[0], want.states, name)
    for r in lhs.reach_explore_batch([m, m], capacity=1 << 18):
        assert result_fields(r) == result_fields(want)


@pytest.mark.parametrize("over", [0, 1 << 17])
@pytest.mark.parametrize("name", ["around_solo", "spill"])
def test_caps(lhs, name, over):
    """Caps that end the search inside it, or 2^17 above one of its sums: a
    level stays with its workgroup only with that much room below the cap."""
    m = layered(SIZES[name])
    sums = np.cumsum(SIZES[name])
    with lhs.Table(1 << 18, 1) as t:
        for cap in sorted({int(s) + d + over for s in sums[2:] for d in (-1, 0, 1)}):
            want = oracle.reach(m, cap=cap, keep_states=True)
            print(f"[levels] {name} cap {cap}: {want.total} states", flush=True)
            assert result_fields(lhs.reach_explore(m, cap=cap, table=t)) == result_fields(want)
            assert_same_set(t.dump()[0], want.states, f"{name} {cap}")


def test_more_levels_than_a_launch(lhs):
    for n in (4095, 4096, 4097, 9000):
        m = gen.chain_model(n)
        print(f"\n[levels] chain of {n}", flush=True)
        with lhs.Table(1 << 15, 1) as t:
            got = lhs.reach_explore(m, table=t)
            assert (got.total, got.n_levels, got.edges, got.deadlocks) == (n, n, n, 0)
            assert got.level_counts == [1] * n


def test_wide_levels_and_back(lhs):
    """Levels above 2^16 states in the middle of narrow ones."""
    m = gen.guarded_model(77, 7, 6, 3, 4, 2)
    want = oracle.reach(m)
    assert max(want.level_counts) > 1 << 16 and want.level_counts[-1] < 100
    print(f"\n[levels] {m.name}: {want.total} states in {want.n_levels} levels", flush=True)
    with lhs.Table(1 << 22, m.W) as t:
        for flags in (0, lhs.REACH_F_PARENTS):
            assert result_fields(lhs.reach_explore(m, table=t, flags=flags)) == result_fields(want)


def test_many_models(lhs):
    """More models than one poll of the tickets reads."""
    models = [layered([1] + [1 + (i * 7 + k) % 16 for k in range(3 + i % 5)]) for i in range(150)]
    want = [oracle.reach(m) for m in models]
    print(f"\n[levels] {len(models)} models", flush=True)
    for r, w in zip(lhs.reach_explore_batch(models, capacity=1 << 12), want):
        assert result_fields(r) == result_fields(w)
