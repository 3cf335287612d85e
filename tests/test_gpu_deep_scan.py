"""Scans of tables that level 0 does not hold whole: where level 0 samples the lines (up to 131,072
allocations) and where nodes lie between, for every kind of layout, with words just below, at and
behind the regions (truncated keys lead those a line too far), at the edges of sub-tiles and
chunks; offsets too large for a packed result; base maps whose values have no code."""
import numpy as np
import pytest

import oracle as orc
from synth import layout as L
from tests.test_gpu_flat_scan import SUB, check_all_forms

pytestmark = pytest.mark.gpu


def table_of(rng, n, shape):
    if shape == "granule":  # whole 2 MiB granules
        size = np.exp(rng.uniform(np.log(4096), np.log(64 << 20), n)).astype(np.uint64) // np.uint64(512) * np.uint64(512)
        step = (size + np.uint64((2 << 20) - 1)) >> np.uint64(21) << np.uint64(21)
        step += rng.integers(0, 4, n).astype(np.uint64) << np.uint64(21)
    elif shape == "huge":  # the same, some of gigabytes
        size = rng.integers(8, 1 << 16, n).astype(np.uint64) * np.uint64(512)
        size[::37] = np.uint64(8 << 30)
        size[5::370] = np.uint64((1 << 40) + 4096)
        step = (size + np.uint64((2 << 20) - 1)) >> np.uint64(21) << np.uint64(21)
    elif shape == "bytes":  # touching or nearly
        size = rng.integers(1, 1 << 22, n).astype(np.uint64)
        step = size + rng.choice([0, 0, 1, 16, 900], n).astype(np.uint64)
    else:  # "run": far fewer level-0 keys than bases
        size = np.full(n, 16, np.uint64)
        step = np.full(n, 16, np.uint64)
        step[n // 2] = np.uint64(1 << 45)
    base = np.uint64(0x10000000) + np.cumsum(step) - step
    t = np.zeros(n, L.ALLOC)
    t["base"], t["size"] = base, size
    assert orc.table_validate(t)[0] == 0
    return t


def words_of(rng, n, t, density):
    w = rng.integers(0, 1 << 16, n, dtype=np.uint64)
    at = np.flatnonzero(rng.random(n) < density)
    r = rng.integers(0, len(t), len(at))
    some = rng.random(len(at)) < 0.3
    r[some] = r[some] // 8 * 8  # the first entries of lines
    off = (rng.random(len(at)) * t["size"][r]).astype(np.uint64)
    kind = rng.integers(0, 6, len(at))
    off = np.where(kind == 0, np.uint64(0), off)
    off = np.where(kind == 1, ~np.uint64(0), off)  # one below
    off = np.where(kind == 2, t["size"][r], off)   # one behind
    w[at] = t["base"][r] + off
    return w


@pytest.mark.parametrize("n_alloc", [16385, 131072, 131073])
@pytest.mark.parametrize("shape", ["granule", "huge", "bytes", "run"])
def test_layouts(n_alloc, shape):
    rng = np.random.default_rng(n_alloc)
    t = table_of(rng, n_alloc, shape)
    check_all_forms(words_of(rng, 60 * SUB + 5, t, 0.3), t, rng)


@pytest.mark.parametrize("n_words", [1, SUB + 1, 7 * SUB + 1, 1535 * SUB + 3, 1536 * SUB - 511, 1536 * SUB + 1, 4096 * SUB + 77])
@pytest.mark.parametrize("n_alloc", [20000, 140000])
def test_edges(n_alloc, n_words):
    rng = np.random.default_rng(n_words)
    t = table_of(rng, n_alloc, "huge")
    check_all_forms(words_of(rng, n_words, t, 0.2), t, rng)


@pytest.mark.parametrize("density", [0.0, 0.1, 0.17, 0.2, 0.49, 1.0])  # one, two, more rounds of candidates
def test_rounds(density):
    rng = np.random.default_rng(17)
    t = table_of(rng, 135000, "bytes")
    check_all_forms(words_of(rng, 90 * SUB + 300, t, density), t, rng)


def pools_of(rng, n, largest):
    """Pools of small blocks, 2^43 bytes and more apart: lines and nodes share level-0 keys, in some pools by the
    hundred; between them regions of their own."""
    size = rng.integers(1, largest // 16 + 1, n).astype(np.uint64) * np.uint64(16)
    step = size + rng.choice([0, 0, 16], n).astype(np.uint64)
    step[[n // 3, n // 3 + 1, n // 2]] += np.uint64(1 << 43)
    step[-2] += np.uint64(1 << 46)
    t = np.zeros(n, L.ALLOC)
    t["base"], t["size"] = np.uint64(0x10000000) + np.cumsum(step) - step, size
    assert orc.table_validate(t)[0] == 0
    return t


# one level and two, runs of two and four nodes to a key, three levels
@pytest.mark.parametrize("top_log2,n_alloc", [(14, 16385), (14, 131072), (14, 131073), (14, 300007), (5, 150), (5, 1500), (5, 3000),
                                              (5, 5000), (5, 20000)])
@pytest.mark.parametrize("largest", [16, 512, 8192])
def test_pools_of_small_blocks(top_log2, n_alloc, largest):
    import paper_2604_06664_amd as fdy

    rng = np.random.default_rng(n_alloc + largest)
    t = pools_of(rng, n_alloc, largest)
    old = fdy.tune_set(fdy.TUNE_SCAN_TOP_LOG2, top_log2)
    try:
        check_all_forms(words_of(rng, 60 * SUB + 5, t, 0.4), t, rng)
    finally:
        fdy.tune_set(fdy.TUNE_SCAN_TOP_LOG2, old)


@pytest.mark.parametrize("top_log2,n_alloc", [(14, 5), (2, 40), (1, 40)])
def test_offsets_beyond_a_packed_result(top_log2, n_alloc):
    import paper_2604_06664_amd as fdy

    rng = np.random.default_rng(3)
    t = np.zeros(n_alloc, L.ALLOC)
    t["base"] = np.uint64(1 << 20) + np.arange(n_alloc, dtype=np.uint64) * np.uint64(1 << 58 if n_alloc == 5 else 1 << 55)
    t["size"] = np.where(np.arange(n_alloc) % 3 == 0, (1 << 55) - 7, 1 << 30).astype(np.uint64)
    old = fdy.tune_set(fdy.TUNE_SCAN_TOP_LOG2, top_log2)
    try:
        check_all_forms(words_of(rng, 40 * SUB + 9, t, 0.5), t, rng)
    finally:
        fdy.tune_set(fdy.TUNE_SCAN_TOP_LOG2, old)


@pytest.mark.parametrize("bases,n_alloc,subs", [("moved", 131073, 24577), ("random", 131073, 24577), ("some odd", 131073, 24577),
                                                ("some odd", 131073, 24575), ("some odd", (1 << 20) + 9, 24576)])
def test_base_map_beside_the_lines(bases, n_alloc, subs):
    """From 24,576 sub-tiles on, with nodes (and, beyond 2^20 allocations, two of them to a key): codes, and new bases
    that have none."""
    from tests.support import session
    from tests.test_gpu_parity import oracle_rebase

    rng = np.random.default_rng(24)
    t = table_of(rng, n_alloc, "granule")
    n = (subs - 1) * SUB + 1
    words = np.tile(words_of(rng, 1 << 18, t, 0.2), 49)[:n]
    nb = t["base"] + np.uint64(0x5000_0000_0000)
    if bases == "random":
        nb = rng.integers(0, 1 << 64, len(t), dtype=np.uint64)
    elif bases == "some odd":
        odd = np.arange(3, len(t), 7)  # (the 64 regions looked at are others)
        nb[odd] += rng.choice([1, 1 << 62], len(odd)).astype(np.uint64)
        nb[1::9] -= np.uint64(0x4fff_0000_0000)  # far below those looked at
    ref, cnt = orc.scan(words, t)
    want, _ = oracle_rebase(orc, words, t, nb)
    run = session.ScanPointersRebaseRun(words, t, nb, prepared=True, staging=False)
    run.launch()
    got, have, status, out = run.result()
    assert status == 0 and have == cnt and np.array_equal(got, ref) and np.array_equal(out, want)
    run = session.ScanRebaseRun(words, t, nb, in_place=True, prepared=False)
    run.launch()
    out, have, status = run.result()
    assert status == 0 and have == cnt and np.array_equal(out, want)
