"""Scans of tables that fit the LDS level whole (up to 2^14 allocations): edges of sub-tiles and
chunks, every share of candidates, runs of blocks that share a truncated key, and a prepared table
whose two sets of chunk states are used in turn by calls of different sizes."""
import numpy as np
import pytest

import oracle as orc
from synth import layout as L

pytestmark = pytest.mark.gpu

SUB = 512
CHUNK_EDGES = [1, SUB - 1, SUB, SUB + 1, 7 * SUB, 7 * SUB + 1, 15 * SUB - 1, 1535 * SUB + 3, 1536 * SUB - 511,
               1536 * SUB + 1, 4096 * SUB + 77]


def table_of(rng, n, shape):
    if shape == "run":  # a run of 16-byte blocks inside one key of a span of 2^46 bytes
        base = np.uint64(0x10000) + np.arange(n, dtype=np.uint64) * np.uint64(16)
        size = np.full(n, 16, np.uint64)
        if n > 1:
            base[-1] = np.uint64(1 << 46)
    else:
        step = rng.integers(8, 1 << 22, n).astype(np.uint64)
        base = np.uint64(0x7F0000000000) + np.cumsum(step) - step
        size = np.maximum(np.uint64(1), (step * rng.random(n)).astype(np.uint64))
    t = np.zeros(n, L.ALLOC)
    t["base"], t["size"] = base, size
    return t


def words_of(rng, n, t, density):
    w = rng.integers(0, 1 << 16, n, dtype=np.uint64)
    at = np.flatnonzero(rng.random(n) < density)
    r = rng.integers(0, len(t), len(at))
    off = (rng.random(len(at)) * t["size"][r]).astype(np.int64)
    off += rng.choice([0, 0, 0, -1, 1], len(at))  # some just outside
    w[at] = (t["base"][r].astype(np.int64) + off).astype(np.uint64)
    return w


def check_all_forms(words, table, rng):
    from tests.support import session
    from tests.test_gpu_parity import oracle_rebase

    ref, n = orc.scan(words, table)
    for prepared in (False, True):
        got, cnt, status = session.scan(words, table, prepared=prepared, staging=False)
        assert status == 0 and cnt == n and np.array_equal(got, ref)
    units = words.view(np.uint32)[1:]
    ref4, n4 = orc.scan_stride4(units, table)
    got, cnt, status = session.scan_stride4(units, table, prepared=True)
    assert status == 0 and cnt == n4 and np.array_equal(got, ref4)
    new_base = rng.integers(0, 1 << 64, len(table), dtype=np.uint64)
    want, _ = oracle_rebase(orc, words, table, new_base)
    for in_place in (False, True):
        run = session.ScanRebaseRun(words, table, new_base, in_place=in_place, prepared=in_place)
        run.launch()
        out, cnt, status = run.result()
        assert status == 0 and cnt == n and np.array_equal(out, want)
    run = session.ScanPointersRebaseRun(words, table, new_base, prepared=True, staging=False)
    run.launch()
    got, cnt, status, out = run.result()
    assert status == 0 and cnt == n and np.array_equal(got, ref) and np.array_equal(out, want)


@pytest.mark.parametrize("n_words", CHUNK_EDGES)
def test_edges(n_words):
    rng = np.random.default_rng(n_words)
    check_all_forms(words_of(rng, n_words, t := table_of(rng, 1000, "spread"), 0.3), t, rng)


@pytest.mark.parametrize("density", [0.0, 0.02, 0.49, 0.51, 1.0])
@pytest.mark.parametrize("n_alloc,shape", [(1, "spread"), (2, "run"), (5, "spread"), (16383, "spread"), (16384, "run")])
def test_candidates_and_tables(n_alloc, shape, density):
    rng = np.random.default_rng(n_alloc)
    t = table_of(rng, n_alloc, shape)
    check_all_forms(words_of(rng, 20 * SUB + 5, t, density), t, rng)


@pytest.mark.parametrize("each", [1, 64, 65, 96, 97, 128, 192, 193, 256, 257, 320, 384, 385, 448, 449, 511, 512])
@pytest.mark.parametrize("top_log2,n_alloc", [(14, 1), (14, 300), (5, 200), (5, 1024)])  # level 0 alone, lines, nodes
def test_candidates_of_a_sub_tile(top_log2, n_alloc, each):
    """Exactly so many candidates in every sub-tile, of words and of 4-byte positions: rounds one by one, two to four at
    a time."""
    import paper_2604_06664_amd as fdy

    old = fdy.tune_set(fdy.TUNE_SCAN_TOP_LOG2, top_log2)
    try:
        candidates_of_a_sub_tile(n_alloc, each)
    finally:
        fdy.tune_set(fdy.TUNE_SCAN_TOP_LOG2, old)


def candidates_of_a_sub_tile(n_alloc, each):
    from tests.support import session
    from tests.test_gpu_parity import oracle_rebase

    rng = np.random.default_rng(each)
    t = np.zeros(n_alloc, L.ALLOC)
    t["base"] = np.uint64(0x7F000000 << 32) + np.arange(n_alloc, dtype=np.uint64) * np.uint64(1 << 34)
    t["size"] = np.uint64(1 << 34) - rng.integers(0, 1 << 33, n_alloc, dtype=np.uint64)
    t["size"][-1] = np.uint64(1 << 34)
    n = 20 * SUB
    chosen = np.concatenate([s * SUB + rng.choice(SUB, each, replace=False) for s in range(20)])
    for stride4 in (True, False):
        units = rng.integers(1, 1 << 20, n + 1 if stride4 else 2 * n).astype(np.uint32)
        high = chosen + 1 if stride4 else 2 * chosen + 1  # the half of a candidate that makes it one
        units[high] = (0x7F000000 + rng.integers(0, 4 * n_alloc, len(high))).astype(np.uint32)
        if stride4:
            ref, cnt = orc.scan_stride4(units, t)
            got, have, status = session.scan_stride4(units, t, prepared=True)
        else:
            ref, cnt = orc.scan(units.view(np.uint64), t)
            got, have, status = session.scan(units.view(np.uint64), t, prepared=True)
        assert 0 < cnt <= 20 * each
        assert status == 0 and have == cnt and np.array_equal(got, ref), stride4
    words, nb = units.view(np.uint64), rng.integers(0, 1 << 63, n_alloc, dtype=np.uint64)  # (of the words' turn)
    want, _ = oracle_rebase(orc, words, t, nb)
    run = session.ScanPointersRebaseRun(words, t, nb, prepared=True, staging=False)
    run.launch()
    got, have, status, out = run.result()
    assert status == 0 and have == cnt and np.array_equal(got, ref) and np.array_equal(out, want)


def test_prepared_states_take_turns():
    import torch

    import paper_2604_06664_amd as fdy
    from tests.support import session

    rng = np.random.default_rng(5)
    t = table_of(rng, 3000, "spread")
    words = words_of(rng, 2000 * SUB, t, 0.25)
    run = session.ScanRun(words, t, prepared=True)
    for n in (2000 * SUB, 300, 1600 * SUB + 9, 0, 7 * SUB, 2000 * SUB, 2000 * SUB, 1):
        ref, want = orc.scan(words[:n], t)
        run.d_relocs.fill_(0xEE)
        fdy.fdy_scan_pointers(run.d_words, n, run.d_table, run.n_alloc, run.d_relocs, run.capacity, run.d_count,
                              run.d_prepared, None, 0, run.d_status)
        got, cnt, status = run.result()
        assert status == 0 and cnt == want and np.array_equal(got, ref), n
        assert bool((run.d_relocs[want * 16:] == 0xEE).all())
    torch.cuda.synchronize()


def test_forms_share_a_prepared_table():
    """Launches of every form, of 16 Mi words and of a few thousand, on one prepared table in turn."""
    import paper_2604_06664_amd as fdy
    from tests.support import session
    from tests.test_gpu_parity import oracle_rebase

    rng = np.random.default_rng(6)
    t = table_of(rng, 300, "spread")
    big = 32768 * SUB + 3
    words = np.tile(words_of(rng, 1 << 20, t, 0.1), 17)[:big]
    new_base = rng.integers(0, 1 << 64, len(t), dtype=np.uint64)
    run = session.ScanPointersRebaseRun(words, t, new_base, prepared=True, staging=False)
    ref, _ = orc.scan(words, t)
    want, _ = oracle_rebase(orc, words, t, new_base)
    for n, form in ((big, "out"), (5000, "scan"), (big, "out"), (9000, "out"), (big, "rebase"), (7000, "rebase"),
                    (big, "scan"), (big, "out")):
        cnt = int(np.searchsorted(ref["word"], n))
        run.d_out.fill_(0xEE)
        if form == "scan":
            fdy.fdy_scan_pointers(run.d_words, n, run.d_table, run.n_alloc, run.d_relocs, run.capacity, run.d_count,
                                  run.d_prepared, None, 0, run.d_status)
        elif form == "out":
            fdy.fdy_scan_pointers_rebase(run.d_words, n, run.d_table, run.n_alloc, run.d_relocs, run.capacity,
                                         run.d_count, run.d_new_base, run.d_out, run.d_prepared, None, 0, run.d_status)
        else:
            fdy.fdy_scan_rebase(run.d_words, n, run.d_table, run.n_alloc, run.d_new_base, run.d_out, run.d_count,
                                run.d_prepared, None, 0, run.d_status)
        got, have, status, out = run.result()
        assert status == 0 and have == cnt, (n, form)
        if form != "rebase":
            assert np.array_equal(got, ref[:cnt]), (n, form)
        if form != "scan":
            assert np.array_equal(out[:n], want[:n]), (n, form)
