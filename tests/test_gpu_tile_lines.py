"""Output tiles against the 128-byte lines that they are stored by: template lengths around a tile, an output
that begins at each 16-byte place of a line, and maps of an odd number of words, so that tiles begin everywhere."""
import numpy as np
import pytest

import oracle as orc
from synth import MatProblem
from synth import layout as L

pytestmark = pytest.mark.gpu
TILE = 2032


@pytest.mark.parametrize("place", range(8))
def test_tiles_at_every_place_of_a_line(place):
    import paper_2604_06664_amd as fdy
    from tests.support import session

    rng = np.random.default_rng(place)
    lens = [1, 2, 15, 16, 17, TILE - 1, TILE, TILE + 1, TILE + 15, TILE + 16, TILE + 17, 2 * TILE, 2 * TILE + 1, 2 * TILE + 9,
            2 * TILE + 16, 2 * TILE + 17, 3 * TILE + 15, 0]  # (a last tile has up to 2,048 words)
    off = np.cumsum([0] + lens).astype(np.uint64)
    W, regions = int(off[-1]), 50
    words = np.sort(rng.choice(W, W // 2, replace=False))
    r = np.zeros(len(words), L.RELOC)
    r["word"], r["region"], r["offset"] = words, rng.integers(0, regions, len(r)), rng.integers(0, 1 << 40, len(r))
    tmpl = rng.permutation(np.r_[np.arange(len(lens)), np.arange(len(lens)), 0]).astype(np.uint32)
    ovr, ovr_off = [], [0]
    for t in tmpl:  # the first and the last half of each tile
        at = sorted({b for k in range(0, lens[t], TILE) for b in (2 * k, 2 * min(k + TILE, lens[t]) - 1)})
        o = np.zeros(len(at), L.OVR32)
        o["byte_off"], o["value"] = np.array(at, np.uint32) * 4, rng.integers(0, 1 << 32, len(at))
        ovr.append(o)
        ovr_off.append(ovr_off[-1] + len(o))
    mp = MatProblem(
        src_words=rng.integers(0, 1 << 63, W, dtype=np.uint64), src_word_off=off, src_nodes=np.zeros(0, L.NODE),
        src_node_off=np.zeros(len(lens) + 1), relocs=r, src_reloc_off=np.searchsorted(words, off.astype(np.int64)),
        tmpl_graph=np.arange(len(lens)), graph_tmpl=tmpl, ovr=np.concatenate(ovr), ovr_off=ovr_off,
        govr=np.zeros(0, L.GRID_OVR), govr_off=np.zeros(len(tmpl) + 1),
        new_base=rng.integers(0, 1 << 63, (17, regions), dtype=np.uint64), map_rank=None, n_ranks=0,
        patch=np.zeros(0, L.PATCH), patch_off=[0])
    wpm = mp.out_words_per_map()
    assert wpm % 2 == 1
    want, _ = orc.materialize(mp)
    default = fdy.tune_get(fdy.TUNE_MAT_SELF_WGS)
    try:
        for self_wgs in (0, default):  # tiles resolved by a launch ahead / by the workgroups themselves
            fdy.tune_set(fdy.TUNE_MAT_SELF_WGS, self_wgs)
            n = 17 * wpm * 8
            room = fdy.device_bytes(n + 512, fill=0xCD)
            lo = (-room.data_ptr()) % 128 + 128 + 16 * place
            run = session.MatRun(mp, want_dims=False, out=room[lo:lo + n])
            run.launch()
            got, _, status = run.result()
            assert status == 0 and np.array_equal(got, want)
            host = room.cpu().numpy()
            assert (host[:lo] == 0xCD).all() and (host[lo + n:] == 0xCD).all()
    finally:
        fdy.tune_set(fdy.TUNE_MAT_SELF_WGS, default)


@pytest.mark.parametrize("n", [1023 * 2048, 1023 * 2048 + 1, 2047 * TILE, 2047 * TILE + 1])
def test_slices_at_the_lines_between_launch_forms(n):
    """1,023 times 2,048 words (and a tile in reserve) are the last that a launch resolves by itself, 2,048 tiles with
    the one in reserve the last whose ends several lanes look for."""
    from tests.support import session
    from tests.test_gpu_parity import check_mat
    from tests.test_gpu_tile_slices import places, problem

    rng = np.random.default_rng(n)
    r = np.zeros(n // 4, L.RELOC)
    r["word"], r["region"], r["offset"] = places(rng, n, n // 4), rng.integers(0, 100, len(r)), rng.integers(0, 1 << 40, len(r))
    ovr = np.zeros(5000, L.OVR32)
    ovr["byte_off"], ovr["value"] = places(rng, 2 * n, 5000) * 4, rng.integers(0, 1 << 32, len(ovr))
    mp = problem(n, r, [0, len(r)], 100, rng, ovr=ovr, ovr_off=[0, len(ovr)])
    mp.new_base = mp.new_base[:1].copy()
    check_mat(session, orc, mp, tag=f"{n} words")


@pytest.mark.parametrize("ranks", [0, 3])
@pytest.mark.parametrize("maps,group", [(1, 0), (2, 0), (16, 0), (17, 0), (63, 64), (64, 64), (65, 64), (130, 64)])
def test_maps_around_the_lines_of_a_group(maps, group, ranks):
    """Two maps to a workgroup by themselves, 64 at most; from nine groups on fewer workgroups to a compute unit (the
    others' launches are resolved by the workgroups themselves as well, up to eight maps each)."""
    import paper_2604_06664_amd as fdy
    from tests.support import session
    from tests.test_gpu_parity import check_mat
    from tests.test_gpu_tile_slices import places, problem

    rng = np.random.default_rng(maps * 5 + ranks)
    n = 3 * TILE + 77
    r = np.zeros(n // 2, L.RELOC)  # up to six registers of entries per thread, none in the second tile
    r["word"] = np.sort(np.r_[places(rng, TILE, 1500), 2 * TILE + places(rng, TILE + 77, len(r) - 1500)])
    r["region"], r["offset"] = rng.integers(0, 100, len(r)), rng.integers(0, 1 << 40, len(r))
    ovr = np.zeros(1100, L.OVR32)  # more than two to a thread in one tile
    ovr["byte_off"], ovr["value"] = places(rng, 2 * TILE, len(ovr)) * 4, rng.integers(0, 1 << 32, len(ovr))
    lists = []
    for k in range(ranks):
        e = np.zeros((5, 600, 0)[k], L.PATCH)  # none, a few, more than one to a thread
        e["word"], e["value"] = places(rng, TILE, len(e)), rng.integers(0, 1 << 63, len(e))
        lists.append(e)
    mp = problem(n, r, [0, len(r)], 100, rng, ranks, ovr=ovr, ovr_off=[0, len(ovr)],
                 **(dict(map_rank=rng.integers(0, ranks, maps).astype(np.uint32), patch=np.concatenate(lists),
                         patch_off=np.cumsum([0] + [len(e) for e in lists]).astype(np.uint64)) if ranks else {}))
    mp.new_base = rng.integers(0, 1 << 63, (maps, 100), dtype=np.uint64)
    try:
        assert fdy.tune_set(fdy.TUNE_MAT_MAP_GROUP, group) == 0
        check_mat(session, orc, mp, tag=f"{maps} maps by {group}, {ranks} ranks")
    finally:
        fdy.tune_set(fdy.TUNE_MAT_MAP_GROUP, 0)


@pytest.mark.parametrize("how", ["swap", "equal"])
def test_disorder_at_every_seam(how):
    """One relocation for every word of three tiles and a bit: neighbours out of order where one lane, wave, register or
    tile of the check ends and the next begins (the one in front is read by another lane, or from memory)."""
    from tests.support import session
    from tests.test_gpu_tile_slices import problem

    rng = np.random.default_rng(3)
    n = 3 * TILE + 300
    r = np.zeros(n, L.RELOC)
    r["word"] = np.arange(n)
    new_base = rng.integers(0, 1 << 63, (3, 1), dtype=np.uint64)
    mp = problem(n, r, [0, n], 1, rng)
    mp.new_base = new_base
    out, _, status = session.materialize(mp, want_dims=False)
    assert status == 0 and np.array_equal(out, np.repeat(new_base, n, axis=1))
    seams = [1, 2, 63, 64, 65, 128, 192, 255, 257] + [256 * i for i in range(1, 8)] + [256 * i + 64 for i in range(1, 8)] + [TILE - 1]
    for tile in range(4):
        for at in [tile * TILE + s for s in seams] + [(tile + 1) * TILE]:
            if at >= n:
                continue
            bad = r.copy()
            if how == "swap":
                bad[[at - 1, at]] = bad[[at, at - 1]]
            else:
                bad["word"][at] = bad["word"][at - 1]
            mp = problem(n, bad, [0, n], 1, rng)
            _, _, status = session.materialize(mp, want_dims=False)
            assert status & L.ST_BAD_ORDER, at
