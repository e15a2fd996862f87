"""A batch of one large dense graph fills the chip: its hub tasks are handed out
in items small enough that the launch is not bound by a few workgroups.  Counts
against the single census (which the parity tests pin to the oracle), and the
time against it; items that end on, before and after a graph's last task."""
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


def _complete(n, seed):
    a, b = np.triu_indices(n, 1)
    f = np.random.default_rng(seed).integers(1, 4, a.size)
    return (n, np.concatenate([a[f & 1 > 0], b[f & 2 > 0]]).astype(np.int32),
            np.concatenate([b[f & 1 > 0], a[f & 2 > 0]]).astype(np.int32))


def _median(f, reps=9):
    t = []
    for _ in range(reps):
        t0 = time.perf_counter()
        f()
        t.append(time.perf_counter() - t0)
    return sorted(t)[reps // 2]


@pytest.mark.parametrize("n", [1451, 1452, 1453, 1454, 1455])
def test_dense_graph_alone_and_twice(ctx, n):
    # from 2^20 hub edges on, tasks of 256 records: some of these counts leave a rest of 4
    x = _complete(n, n)
    g = ctx.build_graph(*x)
    try:
        print(f"[gpu] batch items n={n} tasks={g.info['tri_tasks']} of {g.info['tri_chunk']}", flush=True)
        assert g.info["tri_chunk"] == 256
        want = ctx.census(g).tolist()
        if n == 1451:
            assert want == oracle.census(*x).tolist()
        assert ctx.census_batch([g, g]).tolist() == [want, want]
        assert ctx.census_batch([g]).tolist() == [want]
        if n == 1451:
            # (items of 32 tasks took three times the census)
            one, batch = _median(lambda: ctx.census(g)), _median(lambda: ctx.census_batch([g]))
            print(f"[gpu] census {one * 1e6:.0f} us, batch of one {batch * 1e6:.0f}", flush=True)
            assert batch < 2 * one
    finally:
        g.release()
