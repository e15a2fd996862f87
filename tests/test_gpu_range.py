"""Census of a vertex range: its terms come from all entries of the graph where
the range's rows hold a sixteenth of them or more, else from look-ups.  Ranges on
both sides of that line, single vertices, empty ranges and whole graphs, over
every bucket, against the oracle's range census (integers, tolerance 0)."""
import time

import numpy as np
import pytest

import oracle
from paper_1603_02655_amd import synth, tc

pytestmark = pytest.mark.gpu

BIG = 0xFFFFFFFF


@pytest.fixture(scope="module")
def ctx():
    c = tc.Context(0)
    yield c
    c.close()


def _random(n, m, seed):
    rng = np.random.default_rng(seed)
    return n, rng.integers(0, n, m, dtype=np.int32), rng.integers(0, n, m, dtype=np.int32)


def _rmat(seed):
    g = synth.rmat_digraph(1 << 11, 1 << 14, synth.rng_for(81, seed), reciprocity=0.3)
    return g.n, g.src, g.dst


GRAPHS = {"random": lambda: _random(1600, 9000, 1), "rmat": lambda: _rmat(2), "pairs": lambda: _random(7, 30, 3),
          "few": lambda: (900, np.array([899, 0, 450], np.int32), np.array([0, 899, 3], np.int32))}
MODES = {"default": {}, "hub": dict(t_hub=0), "lane": dict(t0=BIG, t1=BIG, t_hub=BIG), "wave": dict(t0=0, t1=BIG, t_hub=BIG),
         "group": dict(t0=0, t1=0, t_hub=BIG), "mixed": dict(t0=8, t1=24, t_hub=60)}


@pytest.mark.parametrize("mode", sorted(MODES))
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_ranges_on_both_sides_of_the_line(ctx, name, mode):
    n, src, dst = GRAPHS[name]()
    default = ctx.get_tuning()
    try:
        ctx.set_tuning(**MODES[mode])
        g = ctx.build_graph(n, src, dst)
    finally:
        ctx.set_tuning(**default)
    try:
        ranges = [(0, n), (n - 1, n), (0, 1), (n // 2, n // 2), (n // 3, n // 3 + 1)]
        # rows that hold just less and just more than a sixteenth of the entries
        keep = src != dst
        a, b = src[keep].astype(np.int64), dst[keep].astype(np.int64)
        pairs = np.unique(np.minimum(a, b) * n + np.maximum(a, b))
        deg = np.bincount(np.concatenate([pairs // n, pairs % n]), minlength=n)
        ends = np.concatenate([[0], np.cumsum(deg)])
        for u0 in (0, n // 4):
            u1 = int(np.searchsorted(ends, ends[u0] + -(-int(ends[-1]) // 16)))
            ranges += [(u0, min(n, u1 + d)) for d in (-1, 0, 1) if u1 + d > u0]
        print(f"[gpu] range {name} {mode} {ranges}", flush=True)
        og = oracle.OracleGraph(n, src, dst)
        for u0, u1 in ranges:
            want = og.census_range(u0, u1).tolist()
            assert ctx.census_range(g, u0, u1).tolist()[1:] == want[1:], (u0, u1)
    finally:
        g.release()


def test_whole_range_costs_about_a_census(ctx):
    n = 50_000
    g = ctx.build_graph(*_random(n, 50 * n, 4))
    default = ctx.get_tuning()

    def median(f):
        t = []
        for _ in range(11):
            t0 = time.perf_counter()
            f()
            t.append(time.perf_counter() - t0)
        return sorted(t)[5]

    try:
        ctx.set_tuning(tri=0)
        whole, ranged = median(lambda: ctx.census(g)), median(lambda: ctx.census_range(g, 0, n))
        print(f"[gpu] census over dyad records {whole * 1e6:.0f} us, range of all vertices {ranged * 1e6:.0f}", flush=True)
        assert ranged < 1.35 * whole    # (1.6 times with two look-ups per dyad in the bucket kernels)
    finally:
        ctx.set_tuning(**default)
        g.release()
