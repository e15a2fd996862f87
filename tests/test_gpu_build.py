"""Device build at the edges of its kernels: key counts around a sort tile
(4096 keys, two per arc) and an entry tile (2048 keys), vertex counts around
the powers of two that set the number of sort bits and digits, long gaps of
vertices without arcs, and repeated arcs across tile borders.  Counts and build
statistics against the oracle and numpy (integers, tolerance 0)."""
import numpy as np
import pytest

import oracle
from paper_1603_02655_amd import tc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = tc.Context(0)
    yield c
    c.close()


def _stats(n, src, dst):
    s, d = src.astype(np.int64), dst.astype(np.int64)
    loops = int((s == d).sum())
    k = np.unique((s * n + d)[s != d])
    pairs, times = np.unique(np.minimum(k // n, k % n) * n + np.maximum(k // n, k % n), return_counts=True)
    deg = np.bincount(pairs // n, minlength=n) + np.bincount(pairs % n, minlength=n)
    return dict(arcs_in=s.size, arcs_kept=k.size, self_loops_dropped=loops, duplicates_dropped=s.size - loops - k.size,
                asym_dyads=int((times == 1).sum()), mutual_dyads=int((times == 2).sum()),
                max_degree=int(deg.max()), sum_d2=int((deg * deg).sum()))


def _check(ctx, n, src, dst, device=False):
    src, dst = np.asarray(src, np.int32), np.asarray(dst, np.int32)
    print(f"[gpu] build n={n} m={src.size} device={device}", flush=True)
    a, b = (tc.DeviceArray(src), tc.DeviceArray(dst)) if device else (src, dst)
    g = ctx.build_graph(n, a, b)
    try:
        want = _stats(n, src, dst)
        assert {k: g.info[k] for k in want} == want
        full = oracle.census(n, src, dst).tolist()
        assert ctx.census(g).tolist() == full
        # the dyad view: the whole range, and a range that starts inside the ids
        assert ctx.census_range(g, 0, n).tolist()[1:] == full[1:]
        assert (ctx.census_range(g, 0, n // 3) + ctx.census_range(g, n // 3, n)).tolist()[1:] == full[1:]
    finally:
        g.release()


@pytest.mark.parametrize("m", [1, 2, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4097, 70001])
def test_tile_edges(ctx, m):
    rng = np.random.default_rng(m)
    n = 300
    _check(ctx, n, rng.integers(0, n, m), rng.integers(0, n, m), device=m % 2 == 0)


@pytest.mark.parametrize("n", [2, 3, 4, 5, 255, 256, 257, 511, 512, 513, 65535, 65536, 65537, 262145])
def test_id_bits(ctx, n):
    rng = np.random.default_rng(n)
    m = 3000
    src, dst = rng.integers(0, n, m), rng.integers(0, n, m)
    src[:4], dst[:4] = [n - 1, 0, n - 1, n - 1], [0, n - 1, n - 2, n - 1]   # the largest id, and its loop
    _check(ctx, n, src, dst)


def test_gaps_between_rows(ctx):
    # few vertices with arcs, far apart, none at the first and last ids
    n = 40000
    rng = np.random.default_rng(9)
    ids = np.sort(rng.choice(np.arange(500, n - 500), 60, replace=False))
    ids[10:19] = ids[10] + np.arange(9)          # a run of neighbouring ids
    pick = rng.integers(0, ids.size, (2, 900))
    _check(ctx, n, ids[pick[0]], ids[pick[1]])


@pytest.mark.parametrize("times", [2, 700, 5000])
def test_repeated_arcs(ctx, times):
    # runs of equal keys longer than a wavefront's 64, a round and a whole tile
    src = np.concatenate([np.full(times, 3), np.full(times, 7), [1, 7, 2]])
    dst = np.concatenate([np.full(times, 7), np.full(times, 3), [3, 1, 2]])
    order = np.random.default_rng(times).permutation(src.size)
    _check(ctx, 9, src[order], dst[order])
