"""The lane kernels' grid cap (lane_blocks) in the launch that runs a whole
census: fewer workgroups than 256-record blocks take several each.  Counts
against the oracle (integers, tolerance 0), and the cap's effect on the time."""
import time

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


def _random(n, m, seed):
    rng = np.random.default_rng(seed)
    return n, rng.integers(0, n, m, dtype=np.int32), rng.integers(0, n, m, dtype=np.int32)


@pytest.mark.parametrize("spare", [-2, -1, 0, 1])
def test_caps_around_the_number_of_blocks(ctx, spare):
    x = _random(1500, 8000, 3)
    want, want64 = oracle.census(*x).tolist(), oracle.census64(*x).tolist()
    g = ctx.build_graph(*x)
    default = ctx.get_tuning()
    try:
        blocks = -(-g.info["tri_bucket_edges"][0] // 256)
        assert blocks > 3 and g.info["tri_bucket_edges"][1:3] == [0, 0]
        for cap in {1, 3, blocks + spare, -(-blocks // 2) + spare}:
            ctx.set_tuning(lane_blocks=cap)
            print(f"[gpu] lane grid {cap} of {blocks}", flush=True)
            assert ctx.census(g).tolist() == want
            assert ctx.census64(g).tolist() == want64
            assert ctx.census_each_noalloc([g, g]).tolist() == [want, want]
    finally:
        ctx.set_tuning(**default)
        g.release()


def test_cap_has_an_effect(ctx):
    g = ctx.build_graph(*_random(200_000, 800_000, 4))
    default = ctx.get_tuning()

    def median():
        t = []
        for _ in range(9):
            t0 = time.perf_counter()
            ctx.census(g)
            t.append(time.perf_counter() - t0)
        return sorted(t)[4]

    try:
        full = median()
        ctx.set_tuning(lane_blocks=2)    # of 2200 blocks of records
        two = median()
        print(f"[gpu] lane grid: default {full * 1e6:.0f} us, two workgroups {two * 1e6:.0f}", flush=True)
        assert two > 4 * full
    finally:
        ctx.set_tuning(**default)
        g.release()
