"""The server's levels at the sizes where its level driver changes its ways:
levels that stay with their workgroup or are handed out in tiles, caps that
end a query or leave a level less room than it needs there, more queries than
one poll of the tickets sees, and tables made while a launch runs."""
import numpy as np
import pytest

import oracle

from conftest import result_fields
from gpu_util import assert_same_set
from test_gpu_levels import SIZES, layered, lhs  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", sorted(SIZES))
def test_level_sizes(lhs, name):  # noqa: F811
    m = layered(SIZES[name])
    want = oracle.reach(m, keep_states=True)
    print(f"\n[serve] {name}: {want.total} states", flush=True)
    with lhs.Server(capacity=1 << 18) as s, lhs.Table(1 << 18, 1) as t:
        mine = s.submit(m, table=t)
        # the tables of the second and third are made while the first runs
        others = [s.submit(m) for _ in range(2)]
        for k in [mine] + others:
            assert result_fields(s.wait(k)[0]) == result_fields(want)
        assert_same_set(t.dump()[0], want.states, name)


@pytest.mark.parametrize("over", [0, 1 << 17, 1 << 18])
def test_caps(lhs, over):  # noqa: F811
    """Caps inside the search, and 2^17 and 2^18 above one of its sums: a
    level (and a query's first) stays with its workgroup only with room below
    the cap."""
    m = layered(SIZES["around_solo"])
    sums = np.cumsum(SIZES["around_solo"])
    caps = sorted({int(s) + d + over for s in sums[1:] for d in (-1, 0, 1)})
    print(f"\n[serve] caps {caps[0]}..{caps[-1]}", flush=True)
    with lhs.Server(capacity=1 << 20) as s:
        got = [(c, s.submit(m, cap=c)) for c in caps]
        for c, k in got:
            assert result_fields(s.wait(k)[0]) == result_fields(oracle.reach(m, cap=c)), c


def test_many_queries(lhs):  # noqa: F811
    """More queries on the GPU than one poll of the tickets reads."""
    models = [layered([1] + [1 + (i * 7 + k) % 16 for k in range(3 + i % 5)]) for i in range(150)]
    want = [oracle.reach(m) for m in models]
    print(f"\n[serve] {len(models)} queries", flush=True)
    with lhs.Server(capacity=1 << 12) as s:
        for _ in range(2):
            ks = [s.submit(m) for m in models]
            for k, w in zip(ks, want):
                assert result_fields(s.wait(k)[0]) == result_fields(w)
