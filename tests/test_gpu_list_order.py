"""Disorder in the short lists at every place of the check: as many lists as its offsets in LDS hold, one more and many
more, so that kinds are searched in LDS and in memory; in the prep launch and where main resolves its own tiles."""
import numpy as np
import pytest

import oracle as orc
from synth import MatProblem
from synth import layout as L

pytestmark = pytest.mark.gpu


def problem_of(graphs, each, ranks):
    """One template of 64 words and 8 nodes, `graphs` graphs with `each` overrides and grids, a few without any."""
    rng = np.random.default_rng(graphs + each + ranks)
    n = np.where(np.arange(graphs) % 5 == 3, 0, each)
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.uint64)
    ovr, govr = np.zeros(int(off[-1]), L.OVR32), np.zeros(int(off[-1]), L.GRID_OVR)
    at = np.arange(int(off[-1])) - np.repeat(off[:-1].astype(np.int64), n)
    ovr["byte_off"], ovr["value"] = at * 4, rng.integers(0, 1 << 32, len(at))
    govr["node"], govr["grid"] = at, 7
    patch = np.zeros(ranks * each, L.PATCH)
    patch["word"] = np.tile(np.arange(each), ranks)
    nodes = np.zeros(8, L.NODE)
    return MatProblem(
        src_words=rng.integers(0, 1 << 63, 64, dtype=np.uint64), src_word_off=[0, 64], src_nodes=nodes, src_node_off=[0, 8],
        relocs=np.zeros(0, L.RELOC), src_reloc_off=[0, 0], tmpl_graph=[0], graph_tmpl=np.zeros(graphs), ovr=ovr, ovr_off=off,
        govr=govr, govr_off=off, new_base=np.zeros((2, 1)), map_rank=[0, ranks - 1], n_ranks=ranks, patch=patch,
        patch_off=np.arange(ranks + 1) * each)


@pytest.mark.parametrize("graphs,ranks", [(1, 1), (300, 3), (683, 682), (1000, 47), (1000, 49), (1024, 2), (2047, 1), (2049, 9),
                                          (40, 2100), (20000, 2)])
def test_disorder_anywhere_is_flagged(graphs, ranks):
    from tests.support import session

    each = 8
    p = problem_of(graphs, each, ranks)
    base = {n: getattr(p, n) for n in MatProblem.ARRAYS}
    ref, rdims = orc.materialize(p)
    out, dims, status = session.materialize(p)
    assert status == 0 and np.array_equal(out, ref) and np.array_equal(dims, rdims)
    for name, key in (("ovr", "byte_off"), ("govr", "node"), ("patch", "word")):
        lists = getattr(p, name)
        for i in sorted({1, each - 1, len(lists) // 2 // each * each + 3, len(lists) - 1}):
            bad = lists.copy()
            bad[key][i] = bad[key][i - 1]
            _, _, status = session.materialize(MatProblem(n_ranks=ranks, **{**base, name: bad}))
            assert status & L.ST_BAD_ORDER, (name, i)
