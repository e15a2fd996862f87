"""Forward-list kernels at the edges of what they tell apart: ranks around the
hub table's 16384 (and rows whose ranks collide modulo it), runs of hub records
around a step (64), a slice and a task (256, 512), prefixes around a block of
16 entries, and enough of them to pass a segment of 1024 blocks and the packed
counts' 63 steps.  Each through the default thresholds, with every edge in the
hub mode and with every edge in the lane mode, 16 and 64 classes, alone and in a
batch, against the oracle (integers, tolerance 0)."""
import numpy as np
import pytest

import oracle
from paper_1603_02655_amd import tc

pytestmark = pytest.mark.gpu

BIG = 0xFFFFFFFF
MODES = {"default": {}, "hub": dict(t_hub=0), "lane": dict(t0=BIG, t1=BIG, t_hub=BIG)}


@pytest.fixture(scope="module")
def ctx():
    c = tc.Context(0)
    yield c
    c.close()


def _directed(pairs, rng):
    """Arcs of the joined pairs (k, 2): one way, the other or both."""
    f = rng.integers(1, 4, len(pairs))
    a, b = pairs[:, 0], pairs[:, 1]
    return (np.concatenate([a[f & 1 > 0], b[f & 2 > 0]]).astype(np.int32),
            np.concatenate([b[f & 1 > 0], a[f & 2 > 0]]).astype(np.int32))


def _check(ctx, n, pairs, seed, name):
    rng = np.random.default_rng(seed)
    src, dst = _directed(np.asarray(pairs, np.int64), rng)
    want, want64 = oracle.census(n, src, dst).tolist(), oracle.census64(n, src, dst).tolist()
    default = ctx.get_tuning()
    for mode, tuning in MODES.items():
        print(f"[gpu] forward {name} n={n} arcs={src.size} mode={mode}", flush=True)
        try:
            ctx.set_tuning(**tuning)
            g = ctx.build_graph(n, src, dst)
            try:
                assert ctx.census(g).tolist() == want, mode
                assert ctx.census64(g).tolist() == want64, mode
                assert ctx.census_batch([g, g]).tolist() == [want, want], mode
                with np.errstate(over="ignore"):
                    parts = np.sum([ctx.census_shard(g, k, 3) for k in range(3)], axis=0, dtype=np.uint64)
                assert parts.tolist()[1:] == want[1:], mode
            finally:
                g.release()
        finally:
            ctx.set_tuning(**default)


@pytest.mark.parametrize("n", [16383, 16385, 16390, 33000, 50021])
def test_ranks_around_the_table(ctx, n):
    # a circulant graph (equal degrees: ranks follow the ids) with steps that
    # close triangles near a vertex and 16384 and 32768 ranks away
    steps = [d for d in (1, 2, 3, 16383, 16384, 16385, 32768, 32769) if d < n]
    i = np.arange(n)
    pairs = np.concatenate([np.stack([i, (i + d) % n], 1) for d in steps])
    _check(ctx, n, pairs, n, "circulant")


@pytest.mark.parametrize("k", [1, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1025])
def test_runs_of_hub_records(ctx, k):
    # k vertices joined to both ends of an edge, and a little noise
    x = np.arange(2, k + 2)
    pairs = np.concatenate([[[0, 1]], np.stack([x * 0, x], 1), np.stack([x * 0 + 1, x], 1),
                            np.stack([x[:-1:3], x[:-1:3] + 1], 1)])
    _check(ctx, k + 2, pairs, k, "book")


@pytest.mark.parametrize("m", [15, 16, 17, 18, 33, 49, 130, 400])
def test_prefix_blocks(ctx, m):
    a, b = np.triu_indices(m, 1)
    _check(ctx, m + 3, np.stack([a, b], 1), m, "clique")


def test_hub_keys_wider_than_a_word(ctx):
    # so many vertices and pairs that a hub edge's key cannot hold its place in
    # the row: the records gather it; against the census over the dyad records
    rng = np.random.default_rng(7)
    n, m = 4_800_000, 17_500_000
    src, dst = rng.integers(0, n, m, dtype=np.int32), rng.integers(0, n, m, dtype=np.int32)
    dst[: m // 8] = dst[: m // 8] % 3000        # popular vertices, and triangles among them
    src[: m // 16] = src[: m // 16] % 60000
    default = ctx.get_tuning()
    try:
        ctx.set_tuning(t_hub=6)
        g = ctx.build_graph(n, src, dst)
        try:
            print(f"[gpu] forward wide keys edges={g.info['tri_bucket_edges']}", flush=True)
            assert g.info["tri_bucket_edges"][3] > 1 << 20 and g.info["fwd_entries"] > 1 << 24
            got = ctx.census(g).tolist()
            ctx.set_tuning(**dict(default, tri=0))
            assert ctx.census(g).tolist() == got
            assert got[8] + got[9] > 1000
        finally:
            g.release()
    finally:
        ctx.set_tuning(**default)


@pytest.mark.parametrize("blocks", [1, 3, 7, 8, 64, 65])
def test_small_grids(ctx, blocks):
    # grids of fewer workgroups than there are work counters (8), and about
    # 4 x 258 hub tasks: on either side of 16 per wavefront of the grid
    n = 33000
    i = np.arange(n)
    pairs = np.concatenate([np.stack([i, (i + d) % n], 1) for d in (1, 2, 3, 4, 5, 6, 7, 8)])
    default = ctx.get_tuning()
    grids = {k: blocks for k in default if k.endswith("_blocks")}
    try:
        ctx.set_tuning(**grids)
        _check(ctx, n, pairs, blocks, "grid")
        ctx.set_tuning(t0=4, t1=20, t_hub=BIG)    # wave and group records
        _check(ctx, n, pairs, blocks, "grid, wave and group modes")
    finally:
        ctx.set_tuning(**default)


@pytest.mark.parametrize("blocks", [1, 7])
def test_small_grids_over_dyads(ctx, blocks):
    n = 2000
    i = np.arange(n)
    pairs = np.concatenate([np.stack([i, (i + d) % n], 1) for d in (1, 2, 3, 4, 5, 6, 7, 8)])
    default = ctx.get_tuning()
    try:
        ctx.set_tuning(tri=0, **{k: blocks for k in default if k.endswith("_blocks")})
        _check(ctx, n, pairs, blocks, "grid over dyads")
        ctx.set_tuning(t0=4, t1=20, t_hub=BIG)
        _check(ctx, n, pairs, blocks, "grid over dyads, wave and group modes")
    finally:
        ctx.set_tuning(**default)
