"""Censuses of several launches: hub edges that stream more than the graph has
entries run beside the terms and the lane bucket, which have a second stream and
its joins; a small lane bucket comes before the hub kernel, a large one (more
than two workgroups per CU) after.  Reached with edges of every mode, and with
kernel timing; 16 and 64 classes, shards and sequences against the oracle
(integers, tolerance 0)."""
import numpy as np
import pytest

import oracle
from paper_1603_02655_amd import tc

pytestmark = pytest.mark.gpu

ALL_MODES = dict(t0=40, t1=500, t_hub=450)


@pytest.fixture(scope="module")
def ctx():
    c = tc.Context(0)
    yield c
    c.close()


def _graph(sparse):
    """A complete part of 600 vertices, whose edges reach every mode, and `sparse` vertices of 8 neighbours."""
    rng = np.random.default_rng(sparse)
    a, b = np.triu_indices(600, 1)
    f = rng.integers(1, 4, a.size)
    n = 600 + sparse
    s, d = rng.integers(0, n, 4 * sparse), rng.integers(600, n, 4 * sparse)
    src = np.concatenate([a[f & 1 > 0], b[f & 2 > 0], s])
    dst = np.concatenate([b[f & 1 > 0], a[f & 2 > 0], d])
    names = rng.permutation(n)
    return n, names[src].astype(np.int32), names[dst].astype(np.int32)


@pytest.mark.parametrize("timing", [False, True])
@pytest.mark.parametrize("thresholds", ["all", "default"])
@pytest.mark.parametrize("sparse", [3000, 120_000])
def test_terms_and_lanes_beside_the_hub_kernel(ctx, sparse, thresholds, timing):
    x = _graph(sparse)
    og = oracle.OracleGraph(*x)
    want, want64 = og.census().tolist(), og.census64().tolist()
    default = ctx.get_tuning()
    try:
        if thresholds == "all":
            ctx.set_tuning(**ALL_MODES)
        g = ctx.build_graph(*x)
        try:
            edges = g.info["tri_bucket_edges"]
            print(f"[gpu] beside sparse={sparse} {thresholds} timing={timing} edges={edges}", flush=True)
            assert g.info["tri_stream"] > 2 * g.info["fwd_entries"]
            if thresholds == "all":
                assert min(edges) > 0
            # either side of two workgroups of 256 records per CU (256 CUs)
            assert (edges[0] > 2 * 256 * 256) == (sparse > 100_000)
            ctx.set_timing(timing)
            for _ in range(3):      # (each run leaves its counters clear for the next)
                assert ctx.census(g).tolist() == want
                assert ctx.census64(g).tolist() == want64
            with np.errstate(over="ignore"):
                parts = np.sum([ctx.census_shard(g, k, 3) for k in range(3)], axis=0, dtype=np.uint64)
            assert parts.tolist()[1:] == want[1:]
            assert ctx.census_each([g, g]).tolist() == [want, want]
            assert ctx.census_each_noalloc([g, g, g]).tolist() == [want, want, want]
        finally:
            ctx.set_timing(False)
            g.release()
    finally:
        ctx.set_tuning(**default)
