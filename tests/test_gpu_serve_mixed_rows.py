"""Queries whose words do not fit a byte beside queries whose words do: they
join the running launch, whatever the widths."""
import numpy as np
import pytest

import gen
import oracle
from conftest import result_fields
from test_gpu_idle_bound import chain_length, counter_model

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lhs():
    import torch
    assert torch.cuda.is_available()
    import paper_1004_2772_amd as m
    return m


def padded(m, W, L):
    """The model with variables and local states added that nothing uses."""
    trans = np.concatenate([m.trans, np.repeat(m.trans[:, -1:], L - m.L, axis=1)], axis=1)
    return gen.Model(m.P, L, W - m.P, m.D, m.K, np.ascontiguousarray(trans),
                     np.concatenate([m.init, np.zeros(W - m.W, dtype=np.uint32)]), m.cap, m.name)


def word_model(P, S, cap=0):
    """P processes that walk among 300 local states, and set one of S
    variables to 65535 and back: levels of one to some thousand states."""
    L = 300
    rng = np.random.default_rng(100 * P + S)
    trans = np.zeros((P, L, 3, 5), dtype=np.uint32)
    trans[..., 1] = trans[..., 3] = gen.NONE
    for p in range(P):
        for l in range(L):
            trans[p, l, 0, 0] = (l + 1 + (l * l) % (5 + p)) % L
            trans[p, l, 1, 0] = L - 1 - l
            trans[p, l, 2, 0] = l // 2
            if l % 50 == 0:
                v = S - 1 - rng.integers(0, min(S, 2))
                trans[p, l, 1, 1:] = (v, 0, v, 65535)
                trans[p, l, 2, 1:] = (v, 65535, v, 0)
    return gen.Model(P, L, S, 65536, 3, trans, np.zeros(P + S, dtype=np.uint32), cap, f"word{P}+{S}")


# (widest vector of the byte launch, P, S of the word query): tiles of 256,
# 128, 64 and 32 of its rows fit the launch; some queries are cut off by a cap.
# The launch has room in LDS for the transitions of its own byte query, L * 16:
# with 120 local states also for the word query's 1800.  23 processes have more
# than 64 pairs of process and transition, which are found in another way.
@pytest.mark.parametrize("wmax,P,S,cap,L", [(5, 2, 1, 0, 5), (5, 2, 3, 0, 120), (31, 2, 29, 0, 5),
                                            (31, 3, 13, 30000, 5), (20, 2, 18, 0, 120), (12, 3, 9, 30000, 5),
                                            (31, 23, 8, 30000, 5), (24, 23, 1, 30000, 120)])
def test_word_query_joins_byte_launch(lhs, wmax, P, S, cap, L):
    m = word_model(P, S, cap)
    want = result_fields(oracle.reach(m))
    print(f"\n[serve] word query W={P + S} in a byte launch of W={wmax}: {want['total']} states in "
          f"levels of at most {max(want['level_counts'])}", flush=True)
    with lhs.Server(capacity=1 << 21, cfg=lhs.config(8, "double", 0, 1)) as srv:
        # some 0.2 s of one-state levels, in rows of bytes
        first = srv.submit(padded(counter_model(4, 9), wmax, L))
        while srv.stats()["steps"] == 0:
            pass
        byte, word, again = srv.submit(gen.cyclic_model(1, 100)), srv.submit(m), srv.submit(m)
        got = srv.wait(word)
        assert result_fields(got[0]) == want
        assert result_fields(srv.wait(again)[0]) == want
        assert srv.wait(byte)[0].total == 100
        r, times = srv.wait(first)
        assert r.total == chain_length(4, 9)
        assert got[1][2] < times[2], "the query waited for the launch's end"
        assert srv.stats()["steps"] == 1, "another launch"
