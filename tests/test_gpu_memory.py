"""Device memory that runs out, and memory that is kept for reuse.

Each test runs its scenario in a process of its own, in which hipMalloc and
hipFree go through tests/native/alloc_shim.c: it refuses calls on demand, or
once the live bytes would pass a limit, as a smaller GPU would.  Whatever is
refused, a call returns the right counts or TC_ERR_NOMEM."""
import ctypes
import os
import subprocess
import sys
import threading

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

from paper_1603_02655_amd import synth, tc  # noqa: E402

pytestmark = pytest.mark.gpu


def _run(tmp_path, scenario):
    shim = str(tmp_path / "alloc_shim.so")
    subprocess.run(["gcc", "-O1", "-Wall", "-shared", "-fPIC", os.path.join(ROOT, "tests", "native", "alloc_shim.c"),
                    "-o", shim, "-ldl", "-lpthread"], check=True)
    r = subprocess.run([sys.executable, "-u", os.path.abspath(__file__), scenario, shim], capture_output=True, text=True,
                       cwd=ROOT, timeout=100)
    print(r.stdout[-4000:], r.stderr[-4000:], flush=True)
    assert r.returncode == 0 and "scenario passed" in r.stdout


def _graph():
    g = synth.rmat_digraph(1 << 12, 1 << 16, synth.rng_for(71, 0), reciprocity=0.2)
    return g.n, g.src, g.dst


def _poll(c, t):
    while True:
        r = c.poll(t)
        if r is not None:
            return r


def _results(c, g):
    """Every census of g on the current path, as the 16 counts."""
    n, k = g.n, 5
    cuts = [n * i // k for i in range(k + 1)]

    def parts(fs):
        s = np.zeros(16, np.uint64)
        for f in fs:
            s += f()
        s[0] = 0
        return s

    table = tc.tc_class_table()
    return {
        "census": lambda: c.census(g),
        "census64": lambda: np.array([c.census64(g)[table == q].sum() for q in range(16)], np.uint64),
        "range": lambda: parts([lambda i=i: c.census_range(g, cuts[i], cuts[i + 1]) for i in range(k)]),
        "shard": lambda: parts([lambda i=i: c.census_shard(g, i, k) for i in range(k)]),
        "each": lambda: c.census_each([g])[0],
        "noalloc": lambda: c.census_each_noalloc([g])[0],
        "batch": lambda: c.census_batch([g])[0],
        "submit": lambda: _poll(c, c.submit(g)),
    }


def _check_all(c, g, want, may_fail):
    """Every call returns the right counts, or (may_fail) TC_ERR_NOMEM; the calls that failed."""
    failed = []
    for tri in (1, 0):
        c.set_tuning(tri=tri)
        for name, f in _results(c, g).items():
            try:
                got = f()
            except tc.TcError as e:
                assert may_fail and e.code == tc.TC_ERR_NOMEM, (name, tri, e)
                failed.append((name, tri))
                continue
            w = want.copy()
            if name in ("range", "shard"):
                w[0] = 0
            assert got.tolist() == w.tolist(), (name, tri)
    return failed


# ---------------------------------------------------------------- scenarios --

NEW = dict(t0=16, t1=256, t_hub=64, hub_tile=512)


def scenario_rebucket(shim):
    """A rebucket that fails at its k-th allocation, for every k; the next one mends the graph."""
    n, src, dst = _graph()
    lost, k = set(), 0
    while True:
        # (a budget of one byte: nothing is kept, so that every allocation is a hipMalloc)
        with tc.Context(0, hbm_budget_bytes=1) as c:
            g = c.build_graph(n, src, dst)
            want = c.census(g)
            old = c.get_tuning()
            c.set_tuning(**NEW)
            shim.shim_fail_from(k)
            try:
                c.rebucket(g)
                ok = True
            except tc.TcError as e:
                assert e.code == tc.TC_ERR_NOMEM
                ok = False
            refused = shim.shim_refused()
            shim.shim_fail_from(-1)
            assert ok == (refused == 0)
            print("allocation", k, "ok" if ok else "failed", flush=True)
            # (with a budget of one byte a served request never fits)
            failed = [f for f in _check_all(c, g, want, True) if f[0] != "submit"]
            lost.update(failed)
            if ok:
                assert not failed
                break
            c.set_tuning(**dict(old, **NEW, tri=1))
            c.rebucket(g)
            assert not [f for f in _check_all(c, g, want, True) if f[0] != "submit"]
            c.set_tuning(**dict(old, **NEW, tri=1))
            fresh = c.build_graph(n, src, dst)
            same = [q for q in g.info if not q.startswith(("arcs", "self", "dup"))]
            assert {q: g.info[q] for q in same} == {q: fresh.info[q] for q in same}
        k += 1
    assert k >= 6                    # scratch, records, tasks, lists, edge records, edge tasks
    assert ("census", 0) in lost     # (the dyad records were refused)


def test_failed_rebucket_leaves_no_dangling_records(tmp_path):
    _run(tmp_path, "rebucket")


def scenario_threads(shim):
    """Every thread that makes streams or allocates has chosen the context's device."""
    n, src, dst = _graph()
    with tc.Context(0) as c:
        g = c.build_graph(n, src, dst)
        want, got = c.census(g), []

        def requests():     # (a thread of the caller's that has made no HIP call)
            tickets = [c.submit(g)] + [c.submit_arcs(n, src, dst) for _ in range(4)]
            got.extend(_poll(c, t) for t in tickets)

        th = threading.Thread(target=requests)
        th.start()
        th.join()
        assert len(got) == 5 and all(r.tolist() == want.tolist() for r in got)
    assert shim.shim_unchosen() == 0


def test_serving_threads_choose_the_device(tmp_path):
    _run(tmp_path, "threads")


def _er(n, m, seed):
    rng = synth.rng_for(72, seed)
    return n, rng.integers(0, n, m, dtype=np.int32), rng.integers(0, n, m, dtype=np.int32)


def _released(c, count=5):
    """Builds `count` graphs of 2^18 arcs and releases them all: their memory is kept."""
    gs = [c.build_graph(*_er(1 << 14, 1 << 18, i)) for i in range(count)]
    for g in gs:
        g.release()


def scenario_kept(shim):
    """Kept memory goes back when an allocation of any kind needs it, and on trim."""
    big = _er(1 << 15, 1 << 19, 9)
    n, src, dst = _graph()

    def full(slack=0):
        shim.shim_set_limit(shim.shim_live() + slack)

    def free():
        assert shim.shim_refused() > 0, "the limit was not reached"
        shim.shim_set_limit(2**63)

    with tc.Context(0) as c:
        empty = shim.shim_live()
        g = c.build_graph(n, src, dst)
        want = c.census(g)
        wb = tc.Context(0)
        want_big = wb.census(wb.build_graph(*big))
        wb.close()

        _released(c)
        full(64 << 10)                  # scratch and graph of a larger build
        b = c.build_graph(*big)
        free()
        assert c.census(b).tolist() == want_big.tolist()
        b.release()

        other = tc.Context(0)           # another context's allocations
        o = None
        try:
            full(64 << 10)
            o = other.build_graph(*big)
            free()
            assert other.census(o).tolist() == want_big.tolist()
        finally:
            other.close()

        tiny = dict(batch=lambda: c.census_batch([g])[0].tolist() == want.tolist(),
                    submit=lambda: _poll(c, c.submit(g)).tolist() == want.tolist(),
                    context=lambda: tc.Context(0).close() is None)
        for name, f in tiny.items():    # buffers of the calls
            print(name, flush=True)
            _released(c)
            full()
            assert f(), name
            free()

        t = [c.submit_arcs(*big) for _ in range(3)]     # the serving slots' scratch
        for x in t:
            assert _poll(c, x).tolist() == want_big.tolist()
        _released(c)
        full(64 << 10)
        b = c.build_graph(*_er(1 << 16, 1 << 20, 10))
        free()
        b.release()
        g.release()
        before = shim.shim_live()
        c.trim()
        # left: the batch plan's and the slots' small buffers
        assert before - empty > (32 << 20) and shim.shim_live() - empty < (4 << 20)
        h = c.build_graph(n, src, dst)
        assert c.census(h).tolist() == want.tolist()
        h.release()


def test_kept_memory_goes_back(tmp_path):
    _run(tmp_path, "kept")


def scenario_rounding(shim):
    """A block that fits only in its exact size is allocated so."""
    big = _er(1 << 15, 1 << 19, 9)
    with tc.Context(0, hbm_budget_bytes=1) as c:     # nothing kept: exact sizes
        at = shim.shim_live()
        g = c.build_graph(*big)
        want, exact = c.census(g), shim.shim_live() - at
        g.release()
        assert shim.shim_live() == at
    with tc.Context(0) as c:
        g = c.build_graph(*_er(1 << 15, 1 << 19, 11))   # (the scratch)
        g.release()
        c.trim()
        at = shim.shim_live()
        g = c.build_graph(*big)
        rounded = shim.shim_live() - at
        g.release()
        c.trim()
        scratch = rounded - exact
        assert scratch > 0
        shim.shim_set_limit(shim.shim_live() + rounded - (64 << 10))
        g = c.build_graph(*big)
        assert shim.shim_refused() > 0
        shim.shim_set_limit(2**63)
        assert c.census(g).tolist() == want.tolist()


def test_blocks_that_fit_only_exactly(tmp_path):
    _run(tmp_path, "rounding")


def scenario_budget(shim):
    """Served requests that bring their arcs, few of them beside many vertices or
    the other way round, hold no more than the budget, kept memory included."""
    budget = 200 << 20
    few = [(1_000_000, np.array([k, 3], np.int32), np.array([999_999, k + 5], np.int32)) for k in range(6)]
    many = [_er(1 << 15, 1 << 19, 20 + k) for k in range(6)]
    with tc.Context(0) as c:
        want = [c.census(c.build_graph(*x)) for x in few + many]
    with tc.Context(0, hbm_budget_bytes=budget) as c:
        c.submit_arcs(3, [0], [1])
        base = shim.shim_live()
        shim.shim_peak()
        for order in (range(12), range(11, -1, -1), (0, 6, 1, 7, 2, 8, 3, 9, 4, 10, 5, 11)):
            x = few + many
            tickets = {k: c.submit_arcs(*x[k]) for k in order}
            for k, t in tickets.items():
                assert _poll(c, t).tolist() == want[k].tolist()
            peak = shim.shim_peak() - base
            print("peak", peak >> 20, "MB", flush=True)
            assert peak <= budget + (4 << 20)    # (the slots' own small buffers)


def test_served_builds_hold_the_budget(tmp_path):
    _run(tmp_path, "budget")


def scenario_batches(shim):
    """Sets of every kind (with hub tasks over forward lists, over dyad records,
    both or neither) alternate on one batch plan without a new allocation, and
    each replay is right."""
    with tc.Context(0) as c:
        ring = np.arange(500, dtype=np.int32)
        flat = [c.build_graph(500, ring, (ring + k) % 500) for k in (1, 2, 3)]
        hubs = [c.build_graph(*_graph()), c.build_graph(*_er(300, 9000, 30))]
        c.set_tuning(tri=0)
        dyads = [c.build_graph(*_er(300, 9000, 31))]       # (no forward lists)
        c.set_tuning(tri=1)
        sets = [flat, hubs, dyads, hubs + dyads + flat]
        want = [c.census_each(s) for s in sets]
        for s in reversed(sets):
            c.census_batch(s)
        shim.shim_fail_from(-1)
        for r in range(3):
            for s, w in zip(sets, want):
                for _ in range(1 + r):
                    assert c.census_batch(s).tolist() == w.tolist()
        assert shim.shim_calls() == 0


def test_alternating_batches_keep_their_buffers(tmp_path):
    _run(tmp_path, "batches")


def scenario_events(shim):
    """A fork or join of the side stream that fails: the call returns once both
    streams have ended what was launched, and the next one is right."""
    a, b = np.triu_indices(500, 1)
    n, src, dst = 500, a.astype(np.int32), b.astype(np.int32)
    with tc.Context(0) as c:
        c.set_tuning(t0=40, t1=300, t_hub=350)        # edges of every mode: several launches
        g = c.build_graph(n, src, dst)
        assert min(g.info["tri_bucket_edges"]) > 0
        want, want64 = c.census(g), c.census64(g)
        calls = dict(census=(lambda: c.census(g), want), census64=(lambda: c.census64(g), want64),
                     noalloc=(lambda: c.census_each_noalloc([g])[0], want))
        for name, (f, w) in calls.items():
            k = 0
            while True:
                shim.shim_fail_events(k)
                try:
                    got = f()
                except tc.TcError as e:
                    assert e.code == tc.TC_ERR_DEVICE
                    got = None
                failed, syncs = shim.shim_events_failed(), shim.shim_syncs()
                shim.shim_fail_events(-1)
                print(name, "event", k, "failed" if failed else "ok", syncs, flush=True)
                assert (got is None) == (failed > 0)
                assert f().tolist() == w.tolist()
                if not failed:
                    assert got.tolist() == w.tolist()
                    break
                assert syncs >= 2
                k += 1
            assert k == 4                             # fork and join, a record and a wait each


def test_failed_forks_and_joins(tmp_path):
    _run(tmp_path, "events")


if __name__ == "__main__":
    so = ctypes.CDLL(sys.argv[2], mode=ctypes.RTLD_GLOBAL)   # before libtc.so
    so.shim_fail_from.argtypes = [ctypes.c_long]
    so.shim_set_limit.argtypes = [ctypes.c_uint64]
    so.shim_live.restype = ctypes.c_uint64
    so.shim_peak.restype = ctypes.c_uint64
    so.shim_fail_events.argtypes = [ctypes.c_long]
    so.shim_events_failed.restype = so.shim_syncs.restype = ctypes.c_long
    so.shim_calls.restype = ctypes.c_long
    so.shim_refused.restype = ctypes.c_long
    so.shim_unchosen.restype = ctypes.c_long
    globals()["scenario_" + sys.argv[1]](so)
    print("scenario passed", flush=True)
