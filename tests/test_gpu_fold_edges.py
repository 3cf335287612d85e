"""Fingerprints of graphs whose nodes end at the edges of a lane's, a row's, a wave's and a workgroup's share."""
import numpy as np
import pytest

import oracle as orc
from synth import layout as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 33, 63, 64, 65, 127, 448, 449, 511, 512, 513, 1023, 1025, 2632, 5000])
def test_node_counts(n):
    from tests.support import session

    rng = np.random.default_rng(n)
    nodes = np.zeros(3 * n + 1, L.NODE)
    nodes["kernel_id"] = rng.integers(0, 1 << 63, len(nodes), dtype=np.uint64)
    nodes["blob_len"] = rng.integers(0, 1 << 20, len(nodes))
    nodes[n:2 * n] = nodes[:n]  # the second graph repeats the first, the third begins a node late
    off = np.array([0, n, 2 * n, 3 * n + 1], np.uint64)
    keys, tid, tg = orc.fingerprint(nodes, off, L.FP_ALL)
    got = session.fingerprint(nodes, off, L.FP_ALL)
    assert np.array_equal(got[0], keys) and np.array_equal(got[1], tid) and np.array_equal(got[2], tg)
    assert list(tid) == [0, 0, 1]
