"""Models with many transitions at the server: they reach the GPU whole, and
as fast as by a copy."""
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


def path_model(L, K):
    """One process on a path through all L local states in a mixed order: each
    of its L * K transitions leads on, and is taken."""
    trans = np.zeros((1, L, K, 5), dtype=np.uint32)
    trans[..., 1] = trans[..., 3] = gen.NONE
    order = np.concatenate([[0], 1 + np.random.default_rng(L).permutation(L - 1)])
    trans[0, order[:-1], :, 0] = order[1:, None]
    trans[0, order[-1], :, 0] = order[-1]
    return gen.Model(1, L, 0, 1, K, trans, np.zeros(1, dtype=np.uint32), 0, f"path{L}x{K}")


# around one workgroup's 256 transitions, a launch's 64 x 256, and one more each
@pytest.mark.parametrize("L,K", [(16, 16), (257, 1), (1024, 16), (16385, 1), (5000, 7)])
def test_transitions_arrive(lhs, L, K):
    print(f"\n[serve] {L * K} transitions", flush=True)
    with lhs.Server(capacity=1 << 16) as srv:
        for _ in range(2):      # a buffer of its own, and a reused one
            a, b = srv.submit(path_model(L, K)), srv.submit(gen.cyclic_model(2, 8))
            r, _ = srv.wait(a)
            assert (r.total, r.n_levels, r.edges, r.deadlocks) == (L, L, L * K, 0)
            assert srv.wait(b)[0].total == 64


def test_many_transitions_are_copied_fast(lhs):
    """3.8 million transitions (31 MB), of which the exploration uses 40: the
    admission takes no more than twice as long as in the server that uploads
    each query by a copy."""
    L, K = 60000, 16
    trans = np.zeros((4, L, K, 5), dtype=np.uint32)
    trans[..., 1] = trans[..., 3] = gen.NONE
    trans[0, :, :, 0] = np.minimum(np.arange(L) + 1, 39)[:, None]
    m = gen.Model(4, L, 0, 1, K, trans, np.zeros(4, dtype=np.uint32), 0, "wide table")
    best = {}
    for rounds in (False, True):
        with lhs.Server(capacity=1 << 16, rounds=rounds) as srv:
            times = []
            for _ in range(8):
                r, t = srv.wait(srv.submit(m))
                assert r.total == 40
                times.append(t[2] - t[1])
        best[rounds] = min(times)
    print(f"\n[serve] {4 * L * K} transitions: {best[False] * 1e3:.2f} ms, by copies {best[True] * 1e3:.2f} ms",
          flush=True)
    assert best[False] < 2 * best[True]
