"""A build of 2^31 arcs: 2^32 keys, which the sort addresses with 64-bit
positions.  The arcs are a small list over and over, so the oracle's census of
the list is the answer (integers, tolerance 0).  17 GB of host memory, 70 GB on
the device."""
import numpy as np
import pytest

import oracle
from paper_1603_02655_amd import tc

pytestmark = pytest.mark.gpu


def test_keys_beyond_32_bits():
    n, base, m = 3000, 20011, (1 << 31) + 77
    rng = np.random.default_rng(31)
    one = rng.integers(0, n, (2, base), dtype=np.int32)
    arcs = []
    for row in one:
        a = np.empty(m, np.int32)
        done = 1 << 20
        a[:done] = np.resize(row, done)
        while done < m:                       # whole copies of the list: doubling keeps the order
            whole = done // base * base
            k = min(whole, m - done)
            at = done % base
            a[done : done + k] = a[at : at + k]
            done += k
        arcs.append(a)
        print(f"[gpu] wide build: {m} ids ready", flush=True)
    loops = int((arcs[0] == arcs[1]).sum())
    kept = np.unique(one[0].astype(np.int64) * n + one[1])
    kept = kept[kept // n != kept % n].size
    with tc.Context(0) as c:
        g = c.build_graph(n, *arcs)
        print("[gpu] wide build: built", flush=True)
        assert (g.info["arcs_in"], g.info["arcs_kept"], g.info["self_loops_dropped"]) == (m, kept, loops)
        assert g.info["duplicates_dropped"] == m - loops - kept
        want = oracle.census(n, one[0], one[1]).tolist()
        assert c.census(g).tolist() == want
        assert c.census_range(g, 0, n).tolist()[1:] == want[1:]
        g.release()
