"""The slices of relocations, overrides and rank patches that fall into an output tile: lists of lengths
around the steps of a search by four or eight lanes, and tile counts on both sides of the one (2,048, one of them in
reserve) from which a thread looks for a tile's ends alone."""
import numpy as np
import pytest

import oracle as orc
from synth import MatProblem
from synth import layout as L

pytestmark = pytest.mark.gpu
TILE = 2032  # (test_gpu_mat_routes.py fails where this is not the kernel's)


def problem(n, relocs, src_reloc_off, regions, rng, ranks=0, **lists):
    """One graph of n words that is its own template, three base maps."""
    kw = dict(src_words=rng.integers(0, 1 << 63, n, dtype=np.uint64), src_word_off=[0, n], src_nodes=np.zeros(0, L.NODE),
              src_node_off=[0, 0], relocs=relocs, src_reloc_off=src_reloc_off, tmpl_graph=[0], graph_tmpl=[0],
              ovr=np.zeros(0, L.OVR32), ovr_off=[0, 0], govr=np.zeros(0, L.GRID_OVR), govr_off=[0, 0],
              new_base=rng.integers(0, 1 << 63, (3, regions), dtype=np.uint64), map_rank=None, n_ranks=ranks,
              patch=np.zeros(0, L.PATCH), patch_off=[0])
    return MatProblem(**(kw | lists))


def places(rng, n, k):
    return np.sort(rng.choice(n, min(n, k), replace=False))


@pytest.mark.parametrize("tiles", [1, 2, 9, 300, 2046, 2047, 2049])
@pytest.mark.parametrize("entries", [0, 1, 8, 9, 65, 4097, 200_000])
def test_slices(tiles, entries):
    from tests.support import session
    from tests.test_gpu_parity import check_mat

    rng = np.random.default_rng(tiles * 7 + entries)
    n, regions, ranks = tiles * TILE - 5, 100, 3
    r = np.zeros(min(n, entries), L.RELOC)
    r["word"], r["region"], r["offset"] = places(rng, n, entries), rng.integers(0, regions, len(r)), rng.integers(0, 1 << 40, len(r))
    ovr = np.zeros(min(2 * n, entries), L.OVR32)
    ovr["byte_off"], ovr["value"] = places(rng, 2 * n, entries) * 4, rng.integers(0, 1 << 32, len(ovr))
    lists = []
    for k in (entries, entries // 3, 5):
        e = np.zeros(min(n, k), L.PATCH)
        e["word"], e["value"] = places(rng, n, k), rng.integers(0, 1 << 63, len(e))
        lists.append(e)
    mp = problem(n, r, [0, len(r)], regions, rng, ranks, ovr=ovr, ovr_off=[0, len(ovr)], map_rank=[1, 0, 2],
                 patch=np.concatenate(lists), patch_off=np.cumsum([0] + [len(e) for e in lists]).astype(np.uint64))
    check_mat(session, orc, mp, tag=f"{tiles} tiles, {entries} entries")


@pytest.mark.parametrize("tiles", [1, 9, 2047, 2049])  # (with 9 also resolved by the main kernel itself)
def test_offsets_that_decrease_are_reported(tiles):
    """A relocation list that ends before it begins: no entry applies, and the status says so."""
    from tests.support import session

    rng = np.random.default_rng(tiles)
    n = tiles * TILE - 5
    r = np.zeros(n, L.RELOC)
    r["word"] = np.arange(n)
    for lo, hi in ((n // 2, 7), (n // 2, n // 2 - 1), (1, 0)):
        _, _, status = session.materialize(problem(n, r, [lo, hi], 1, rng))
        assert status & L.ST_BAD_ORDER, (lo, hi)
    _, _, status = session.materialize(problem(n, r, [0, n], 1, rng))
    assert status == 0


@pytest.mark.parametrize("ranks", [1, 799, 800, 1599])  # 41 tiles with the one in reserve: beyond 32,768 pairs (799 and 800 ranks) a thread searches alone
@pytest.mark.parametrize("entries", [1, 9, 700])
def test_slices_of_many_ranks(ranks, entries):
    from tests.support import session
    from tests.test_gpu_parity import check_mat

    rng = np.random.default_rng(ranks + entries)
    n = 40 * TILE - 5
    lens = rng.integers(0, 3, ranks)
    lens[[0, ranks // 2, ranks - 1]] = entries
    patch = np.zeros(int(lens.sum()), L.PATCH)
    patch["word"] = np.concatenate([places(rng, n, k) for k in lens])
    patch["value"] = rng.integers(0, 1 << 63, len(patch))
    r = np.zeros(n // 3, L.RELOC)
    r["word"], r["region"] = np.arange(n // 3) * 3, rng.integers(0, 50, n // 3)
    mp = problem(n, r, [0, len(r)], 50, rng, ranks, map_rank=[ranks - 1, 0, ranks // 2], patch=patch,
                 patch_off=np.cumsum(np.r_[0, lens]).astype(np.uint64))
    check_mat(session, orc, mp, tag=f"{ranks} ranks, {entries} entries")
