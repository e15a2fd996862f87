"""Forward lists beyond rank 16384, the hub kernels' further passes: lists of
256 (16 classes) and 512 entries (64 codes) to a table, on both sides of
one, two and three tables, next to each other and far apart.  Against the census
over the dyad records, which the parity tests pin to the oracle; smaller ones
against the oracle itself (integers, tolerance 0)."""
import time

import numpy as np
import pytest

from paper_1603_02655_amd import tc
from tests.test_gpu_forward import _check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = tc.Context(0)
    yield c
    c.close()


def _circulant(n, steps, seed):
    """Equal degrees, so the ranks follow the ids: N+(y) is y + step, where that has the larger id."""
    rng = np.random.default_rng(seed)
    a = np.repeat(np.arange(n, dtype=np.int32), len(steps))
    b = (a + np.tile(np.asarray(steps, np.int32), n)) % n
    f = rng.integers(1, 4, a.size, dtype=np.uint8)
    return n, np.concatenate([a[f & 1 > 0], b[f & 2 > 0]]), np.concatenate([b[f & 1 > 0], a[f & 2 > 0]])


def _against_dyads(ctx, x, name):
    n, src, dst = x
    default = ctx.get_tuning()
    g = ctx.build_graph(n, src.astype(np.int32), dst.astype(np.int32))
    try:
        print(f"[gpu] tail {name} n={n} arcs={src.size} stream={g.info['tri_stream']}", flush=True)
        got, got64 = ctx.census(g).tolist(), ctx.census64(g).tolist()
        batch = ctx.census_batch([g, g]).tolist()
        with np.errstate(over="ignore"):
            parts = np.sum([ctx.census_shard(g, k, 3) for k in range(3)], axis=0, dtype=np.uint64).tolist()
        ctx.set_tuning(tri=0)
        want = ctx.census(g).tolist()
        assert got == want and batch == [want, want] and parts[1:] == want[1:]
        assert got64 == ctx.census64(g).tolist()
    finally:
        ctx.set_tuning(**default)
        g.release()


@pytest.mark.parametrize("k", [255, 256, 257, 511, 512, 513, 1025])
def test_lists_around_the_table_size(ctx, k):
    _against_dyads(ctx, _circulant(16384 + 2 * k + 50, range(1, k + 1), k), f"ring {k}")


def test_long_lists_far_apart(ctx):
    n = 30_000
    steps = np.random.default_rng(5).choice(np.arange(1, n // 2), 1150, replace=False)
    _against_dyads(ctx, _circulant(n, np.sort(steps), 6), "scattered")


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 33, 70])
def test_short_lists(ctx, k):
    n = 16384 + 700
    a = np.repeat(np.arange(n), k)
    pairs = np.stack([a, (a + np.tile(np.arange(1, k + 1), n)) % n], 1)
    _check(ctx, n, pairs, k, f"ring {k}")


def test_groups_beyond_the_table_cost_as_much_as_below(ctx):
    """Complete groups of 300: 50 of them below rank 16384, 200 for the most part beyond."""
    i, j = np.triu_indices(300, 1)

    def groups(c):
        a, b = (np.arange(c)[:, None] * 300 + i).ravel(), (np.arange(c)[:, None] * 300 + j).ravel()
        return ctx.build_graph(300 * c, a.astype(np.int32), b.astype(np.int32))

    def median(g):
        t = []
        for _ in range(9):
            t0 = time.perf_counter()
            ctx.census(g)
            t.append(time.perf_counter() - t0)
        return sorted(t)[4]

    few, many = groups(50), groups(200)
    a, b = median(few), median(many)
    few.release()
    many.release()
    print(f"[gpu] tail: 50 groups {a * 1e6:.0f} us, 200 groups {b * 1e6:.0f}", flush=True)
    assert b < 10 * a
