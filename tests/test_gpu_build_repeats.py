"""Arcs repeated 10^4 to 10^6 times, as in edge lists of events: counts and
statistics as for the distinct arcs, in about the time of a list without
repeats.  Oracle and numpy, integers, tolerance 0."""
import time

import numpy as np
import pytest

from paper_1603_02655_amd import tc
from tests.test_gpu_build import _check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = tc.Context(0)
    yield c
    c.close()


# the last key of a run is what tells: the mirrored arc once, often, never; runs
# of 2^k - 1, 2^k and 2^k + 1 keys end the doubling steps on, before and after it
@pytest.mark.parametrize("times,mirrored", [(1, 1), (2, 1), (3, 0), (3, 1), (4, 1), (7, 1), (8, 1), (9, 2), (16383, 1),
                                            (16384, 1), (16385, 0), (40000, 40000), (1_000_000, 0), (1_000_000, 1),
                                            (1, 1_000_000)])
def test_runs_of_one_pair(ctx, times, mirrored):
    rng = np.random.default_rng(times + mirrored)
    n, more = 50, 400
    src = np.concatenate([np.full(times, 11), np.full(mirrored, 30), rng.integers(0, n, more)])
    dst = np.concatenate([np.full(times, 30), np.full(mirrored, 11), rng.integers(0, n, more)])
    order = rng.permutation(src.size)
    _check(ctx, n, src[order], dst[order], device=times % 2 == 0)


def test_every_pair_repeated(ctx):
    rng = np.random.default_rng(3)
    n = 40
    src, dst = rng.integers(0, n, 100_000), rng.integers(0, n, 100_000)
    _check(ctx, n, src, dst)


def test_repeats_cost_no_serial_walk(ctx):
    """A build is bound by its number of arcs (the walk of one lane along 10^6
    equal keys took a hundred times as long as the rest)."""
    m, n = 1_000_000, 100_000
    rng = np.random.default_rng(4)
    src, dst = rng.integers(0, n, 2 * m, dtype=np.int32), rng.integers(0, n, 2 * m, dtype=np.int32)
    rep_s, rep_d = src.copy(), dst.copy()
    at = rng.permutation(2 * m)[:m]
    rep_s[at], rep_d[at] = 17, 4711

    def best(s, d):
        t = []
        for _ in range(4):
            t0 = time.perf_counter()
            ctx.build_graph(n, s, d).release()
            t.append(time.perf_counter() - t0)
        return min(t)

    plain, repeated = best(src, dst), best(rep_s, rep_d)
    print(f"[gpu] build without repeats {plain * 1e3:.2f} ms, with {repeated * 1e3:.2f}", flush=True)
    assert repeated < 10 * plain
