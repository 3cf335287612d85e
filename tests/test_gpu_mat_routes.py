"""How many base maps a workgroup takes under rank patches, and so whether a launch resolves its own tiles, on both sides
of each line of the rule; and the most groups of maps with which one does.  Results against the oracle."""
import numpy as np
import pytest

import oracle as orc
from synth import layout as L

pytestmark = pytest.mark.gpu
TILE = 2032


# tiles (one more is reserved), maps, launches
@pytest.mark.parametrize("tiles,maps,launches", [
    (448, 4, 1), (448, 5, 1), (448, 6, 1), (448, 8, 1), (448, 9, 1), (448, 10, 1), (448, 11, 2),  # 449 * 11 > 4,608
    (866, 3, 1), (866, 5, 1), (866, 6, 2),
    (1000, 3, 1), (1031, 4, 1), (1032, 3, 2), (1032, 5, 2), (1032, 6, 2),  # 1,031 * 2,032 words are 1,023 * 2,048
    (266, 16, 1), (270, 17, 2), (198, 25, 2), (199, 25, 2),  # 199 + 1: groups of four
    (159, 23, 1), (159, 32, 2),
    (23, 84, 1), (23, 96, 2), (23, 112, 1), (40, 62, 2), (40, 64, 1), (10, 256, 1), (10, 257, 2)])
def test_launches_under_patches(tiles, maps, launches):
    import paper_2604_06664_amd as fdy
    from tests.support import session
    from tests.test_gpu_tile_slices import places, problem

    rng = np.random.default_rng(tiles * maps)
    n, ranks = tiles * TILE - 7, 3
    r = np.zeros(n // 50, L.RELOC)
    r["word"], r["region"], r["offset"] = places(rng, n, n // 50), rng.integers(0, 60, len(r)), rng.integers(0, 1 << 40, len(r))
    ovr = np.zeros(300, L.OVR32)
    ovr["byte_off"], ovr["value"] = places(rng, 2 * n, 300) * 4, rng.integers(0, 1 << 32, 300)
    lists = []
    for k in (700, 3, 260):
        e = np.zeros(k, L.PATCH)
        e["word"], e["value"] = places(rng, min(n, 4 * TILE), k), rng.integers(0, 1 << 63, k)
        lists.append(e)
    mp = problem(n, r, [0, len(r)], 60, rng, ranks, ovr=ovr, ovr_off=[0, len(ovr)],
                 map_rank=rng.integers(0, ranks, maps).astype(np.uint32), patch=np.concatenate(lists),
                 patch_off=np.cumsum([0] + [len(e) for e in lists]).astype(np.uint64))
    mp.new_base = rng.integers(0, 1 << 63, (maps, 60), dtype=np.uint64)
    run = session.MatRun(mp, want_dims=False)
    fdy.prof_enable(8)
    try:
        run.launch()
        timed = fdy.prof_read()
    finally:
        fdy.prof_enable(0)
    out, _, status = run.result()
    assert status == 0 and np.array_equal(out, orc.materialize(mp, False)[0])
    assert sum(v["n"] for v in timed.values()) == launches, timed


# tiles by groups of two maps: 64 groups are the most that resolve their own tiles; between 1,000 and 1,230 workgroups
# five share a compute unit, on either side four
@pytest.mark.parametrize("tiles,maps,launches", [(4, 127, 1), (4, 128, 1), (4, 129, 2), (4, 300, 2), (10, 200, 2), (10, 201, 2),
                                                 (10, 246, 2), (10, 247, 2)])
def test_launches_by_groups_of_maps(tiles, maps, launches):
    import paper_2604_06664_amd as fdy
    from tests.support import session
    from tests.test_gpu_tile_slices import places, problem

    rng = np.random.default_rng(maps)
    n = tiles * TILE - 100
    r = np.zeros(n // 3, L.RELOC)
    r["word"], r["region"], r["offset"] = places(rng, n, n // 3), rng.integers(0, 60, len(r)), rng.integers(0, 1 << 40, len(r))
    mp = problem(n, r, [0, len(r)], 60, rng)
    mp.new_base = rng.integers(0, 1 << 63, (maps, 60), dtype=np.uint64)
    run = session.MatRun(mp, want_dims=False)
    fdy.prof_enable(8)
    try:
        run.launch()
        timed = fdy.prof_read()
    finally:
        fdy.prof_enable(0)
    out, _, status = run.result()
    assert status == 0 and np.array_equal(out, orc.materialize(mp, False)[0])
    assert sum(v["n"] for v in timed.values()) == launches, timed


@pytest.mark.parametrize("tiles", [*range(38, 49), *range(78, 89), 160])  # (and one in reserve)
def test_launches_of_whole_rounds(tiles):
    """Rounded up to a multiple of eight from 40 tiles on, and from 80 where the workgroups resolve them."""
    from tests.support import session
    from tests.test_gpu_parity import check_mat
    from tests.test_gpu_tile_slices import places, problem

    rng = np.random.default_rng(tiles)
    n = tiles * TILE - 1
    r = np.zeros(n // 20, L.RELOC)
    r["word"], r["region"], r["offset"] = places(rng, n, n // 20), rng.integers(0, 60, len(r)), rng.integers(0, 1 << 40, len(r))
    mp = problem(n, r, [0, len(r)], 60, rng)  # three maps, two groups; resolved both ways
    check_mat(session, orc, mp, tag=f"{tiles} tiles", want_dims=False)


@pytest.mark.parametrize("tiles", range(40, 49))
def test_entries_of_no_tile_are_marked(tiles):
    """A table that held a tile of one word in each of its entries, the graph's first."""
    import paper_2604_06664_amd as fdy
    from tests.support import session
    from tests.test_gpu_tile_slices import problem

    rng = np.random.default_rng(tiles)
    n = tiles * TILE
    r = np.zeros(1, L.RELOC)
    mp = problem(n, r, [0, 1], 60, rng)
    old = fdy.tune_set(fdy.TUNE_MAT_SELF_WGS, 0)
    try:
        run = session.MatRun(mp, want_dims=False)
        ws = np.zeros(run.ws_bytes, np.uint8)
        table = ws[1024:1024 + 48 * (tiles + 8)].view(np.uint32).reshape(-1, 12)  # behind the header and three offset lists
        table[:, 4] = 1
        run.d_ws.copy_(fdy.to_device(ws))
        run.launch()
    finally:
        fdy.tune_set(fdy.TUNE_MAT_SELF_WGS, old)
    out, _, status = run.result()
    assert status == 0 and np.array_equal(out, orc.materialize(mp, False)[0])
    after = fdy.to_host(run.d_ws, np.uint32, run.ws_bytes // 4)[256:][:12 * (tiles + 8)].reshape(-1, 12)[:, 4]
    entries = (tiles + 1 + 7) // 8 * 8
    assert (after[:tiles] == TILE).all() and not after[tiles:entries].any() and (after[entries:] == 1).all()


@pytest.mark.parametrize("n", [1, TILE - 1, TILE, TILE + 1, 2 * TILE, 2 * TILE + 1])
def test_tiles_have_2032_words(n):
    """One launch of main to each tile (and the one in reserve): what the other tests call a tile is one."""
    import paper_2604_06664_amd as fdy
    from tests.support import session
    from tests.test_gpu_tile_slices import problem

    mp = problem(n, np.zeros(0, L.RELOC), [0, 0], 1, np.random.default_rng(n))
    run = session.MatRun(mp, want_dims=False)
    old = fdy.tune_set(fdy.TUNE_MAT_MOST_BLOCKS, 1)
    fdy.prof_enable(8)
    try:
        run.launch()
        timed = fdy.prof_read()
    finally:
        fdy.prof_enable(0)
        fdy.tune_set(fdy.TUNE_MAT_MOST_BLOCKS, old)
    assert timed["mat_main_kernel"]["n"] == -(-n // TILE) + 1
    out, _, status = run.result()
    assert status == 0 and np.array_equal(out, orc.materialize(mp, False)[0])
