"""Launch dimensions: grid-override lists of every length around the eight-way search's steps, and
graph counts around the 256 that the per-graph sums take at a time."""
import numpy as np
import pytest

import oracle as orc
from synth import MatProblem
from synth import layout as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graphs", [1, 255, 256, 257, 600, 1000, 1001, 1024])
def test_grid_overrides(graphs):
    from tests.support import session
    from tests.test_gpu_parity import check_mat, problem, replicate_outputs, small

    rng = np.random.default_rng(graphs)
    mp = problem(orc, small(2))
    mp = replicate_outputs(mp, -(-graphs // mp.G))
    kw = {n: getattr(mp, n) for n in MatProblem.ARRAYS}
    kw["graph_tmpl"] = mp.graph_tmpl[:graphs]
    kw["ovr_off"] = mp.ovr_off[:graphs + 1]
    kw["ovr"] = mp.ovr[:int(kw["ovr_off"][-1])]
    nodes = np.diff(mp.src_node_off.astype(np.int64))[mp.tmpl_graph[kw["graph_tmpl"]]]
    lists = []
    for g, n in enumerate(nodes):
        k = min(int(n), [0, 1, 2, 7, 8, 9, 63, 64, 65, int(n)][g % 10])
        e = np.zeros(k, L.GRID_OVR)
        e["node"] = np.sort(rng.choice(int(n), k, replace=False))
        e["grid"] = rng.integers(1, 1 << 31, (k, 3))
        lists.append(e)
    kw["govr"] = np.concatenate(lists)
    kw["govr_off"] = np.cumsum([0] + [len(e) for e in lists]).astype(np.uint64)
    check_mat(session, orc, MatProblem(n_ranks=mp.n_ranks, **kw), tag=f"{graphs} graphs")
