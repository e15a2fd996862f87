"""Hub edges found at either end: graphs whose popular vertices have few
neighbours of smaller rank, so that an edge (x, y) streams N+(y) against N+(x)
instead of the prefix of N+(x) against N+(y).  Sizes on both sides of the rule
(blocks of 16), ranks on both sides of the table's 16384, keys with and without
room for an edge's place; 16 and 64 classes, alone, in shards and in a batch,
against the oracle (integers, tolerance 0)."""
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


def _bipartite(users, items, tops):
    """Users joined to all items, everything to `tops` vertices: N+(item) = tops, N+(user) = tops and items."""
    u, i = np.meshgrid(np.arange(users), users + np.arange(items), indexing="ij")
    pairs = [np.stack([u.ravel(), i.ravel()], 1)]
    for k in range(tops):
        pairs.append(np.stack([np.arange(users + items), np.full(users + items, users + items + k)], 1))
    return users + items + tops, np.concatenate(pairs)


# prefixes of 1, 2, 3, ... blocks against lists of 1, 2 and 3: the edges change
# ends past 32, 64 and 96 entries
@pytest.mark.parametrize("users,items,tops", [(90, 34, 1), (150, 100, 1), (150, 100, 16), (150, 100, 17), (300, 200, 3),
                                              (600, 520, 40), (70, 40, 40)])
def test_few_neighbours_of_smaller_rank(ctx, users, items, tops):
    n, pairs = _bipartite(users, items, tops)
    _check(ctx, n, pairs, users + tops, "bipartite")


def test_changed_ends_are_used(ctx):
    n, pairs = _bipartite(400, 300, 1)
    g = ctx.build_graph(n, pairs[:, 0].astype(np.int32), pairs[:, 1].astype(np.int32))
    assert g.info["tri_stream"] < 20 * g.info["tri_bucket_edges"][3]    # (prefixes: 150 entries on average)
    g.release()


def test_items_with_links(ctx):
    # random items per user, random links among the items: both kinds of edges at one vertex
    rng = np.random.default_rng(5)
    users, items, per, links = 700, 150, 60, 4
    u, i = np.repeat(np.arange(users), per), users + rng.integers(0, items, users * per)
    a = users + np.repeat(np.arange(items), links)
    b = users + rng.integers(0, items, a.size)
    pairs = np.unique(np.sort(np.concatenate([np.stack([u, i], 1), np.stack([a, b], 1)[a != b]]), 1), axis=0)
    _check(ctx, users + items, pairs, 6, "links")


@pytest.mark.parametrize("pad", [0, 16384 - 60, 16384 + 5, 40000])
def test_ranks_beyond_the_table(ctx, pad):
    """`pad` vertices in cliques of 40 rank before everything else, so the lists of
    the bipartite part stand below, around and beyond rank 16384."""
    n0, pairs = _bipartite(36, 34, 1)
    cliques = [pairs]
    n = n0
    a, b = np.triu_indices(80, 1)
    left = pad
    while left > 0:
        k = min(left, 80)
        keep = b < k
        cliques.append(np.stack([a[keep], b[keep]], 1) + n)
        n += k
        left -= k
    # a few cliques reach into the items, so that their lists hold ranks of both sides
    rng = np.random.default_rng(pad)
    if pad:
        cliques.append(np.stack([36 + rng.integers(0, 34, 60), n0 + rng.integers(0, pad, 60)], 1))
    _check(ctx, n, np.unique(np.sort(np.concatenate(cliques), 1), axis=0), pad, f"pad {pad}")


def test_wide_keys(ctx):
    """Keys without room for an edge's place, edges found at both ends; against the
    census over the dyad records."""
    rng = np.random.default_rng(8)
    n, m = 4_800_000, 17_500_000
    src, dst = rng.integers(0, n, m, dtype=np.int32), rng.integers(0, n, m, dtype=np.int32)
    users, items = 2000, 400
    k = users * 200
    src[:k] = np.repeat(np.arange(users), 200)
    dst[:k] = users + rng.integers(0, items, k)
    src[k : k + users + items] = n - 1                    # joined to all of them
    dst[k : k + users + items] = np.arange(users + items)
    default = ctx.get_tuning()
    try:
        ctx.set_tuning(t_hub=6)
        g = ctx.build_graph(n, src, dst)
        try:
            print(f"[gpu] wide keys edges={g.info['tri_bucket_edges']} stream={g.info['tri_stream']}", flush=True)
            assert g.info["fwd_entries"] > 1 << 24
            got = ctx.census(g).tolist()
            ctx.set_tuning(**dict(default, tri=0))
            assert ctx.census(g).tolist() == got
        finally:
            g.release()
    finally:
        ctx.set_tuning(**default)
