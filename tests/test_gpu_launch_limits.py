"""Materializations of more tiles, patch slices or launch dimensions than one grid holds (2^32 threads, beyond which the
runtime cuts a grid without an error): the same in several launches and rounds, with the number of blocks from which
that happens set low."""
import numpy as np
import pytest

import oracle as orc
from synth import MatProblem, make_config
from synth import layout as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("most", [1, 2, 7, 41, 42, 43])
def test_tiles_and_patch_slices_in_pieces(most):
    """41 tiles and one that is reserved; 33,600 slices, which a thread each looks for."""
    import paper_2604_06664_amd as fdy
    from tests.support import session
    from tests.test_gpu_parity import check_mat
    from tests.test_gpu_tile_slices import places, problem

    rng = np.random.default_rng(most)
    n, ranks = 41 * 2032 - 5, 800
    lens = rng.integers(0, 6, ranks)
    patch = np.zeros(int(lens.sum()), L.PATCH)
    patch["word"] = np.concatenate([places(rng, n, k) for k in lens])
    patch["value"] = rng.integers(0, 1 << 63, len(patch))
    r = np.zeros(n // 3, L.RELOC)
    r["word"], r["region"] = np.arange(n // 3) * 3, rng.integers(0, 50, n // 3)
    mp = problem(n, r, [0, len(r)], 50, rng, ranks, map_rank=[ranks - 1, 0, ranks // 2], patch=patch,
                 patch_off=np.cumsum(np.r_[0, lens]).astype(np.uint64))
    old = fdy.tune_set(fdy.TUNE_MAT_MOST_BLOCKS, most)
    assert old == 1 << 23
    try:
        check_mat(session, orc, mp, tag=f"{most} blocks")
    finally:
        fdy.tune_set(fdy.TUNE_MAT_MOST_BLOCKS, old)


@pytest.mark.parametrize("most", [1, 2, 3, 5])
def test_launch_dimensions_in_rounds(most):
    import paper_2604_06664_amd as fdy
    from tests.support import session
    from tests.test_gpu_parity import check_mat

    ar = make_config(2, layers=8, batch_sizes=[1, 2, 4, 8, 16]) if most % 2 else make_config(1)
    relocs, _ = orc.scan(ar.words, ar.table)
    _, tid, tg = orc.fingerprint(ar.nodes, ar.node_off, ar.fp_mask)
    mp = MatProblem.from_archive(ar, relocs, orc.reloc_segment(relocs, ar.word_off), graph_tmpl=tid, tmpl_graph=tg)
    old = fdy.tune_set(fdy.TUNE_MAT_MOST_BLOCKS, most)
    try:
        check_mat(session, orc, mp, tag=f"{most} blocks")
    finally:
        fdy.tune_set(fdy.TUNE_MAT_MOST_BLOCKS, old)
