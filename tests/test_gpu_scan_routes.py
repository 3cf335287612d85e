"""Word-dense inputs through lines and nodes (a small table beyond a level 0 made smaller), through level 0
alone at a size where workgroups take many chunks, and the bounded wait of the ordered scan."""
import numpy as np
import pytest

import oracle as orc
from synth import layout as L

pytestmark = pytest.mark.gpu

SUB = 512


def dense_input(n):
    """301 touching 64-byte regions and one at the top of the address space; nearly every word a hit."""
    rng = np.random.default_rng(5)
    t = np.array([(0x1000 + 64 * i, 64) for i in range(300)] + [(2**64 - 0x100, 0xFF)], L.ALLOC)
    w = (0x1000 + rng.integers(0, 64 * 300, n)).astype(np.uint64)
    w[::97] = np.uint64(2**64 - 1)
    w[1::97] = np.uint64(2**64 - 2)
    w[2::97] = np.uint64(0xFFF)
    return w, t, rng.integers(0, 1 << 64, len(t), dtype=np.uint64)


def dense_with_gaps(n):
    """The same with a stretch of the input without candidates, and one with some."""
    w, t, nb = dense_input(n)
    w[n // 3:n // 2] = np.arange(n // 2 - n // 3, dtype=np.uint64) % np.uint64(0x1000)
    w[n // 2:n // 2 + n // 8:3] = np.uint64(7)
    return w, t, nb


@pytest.mark.parametrize("n", [9000, 70 * SUB + 1, 1 << 20, 4096 * SUB + 777])  # the last two: fifteen workers
@pytest.mark.parametrize("make", [dense_input, dense_with_gaps])
def test_dense_words_of_a_table_with_nodes(n, make):
    import paper_2604_06664_amd as fdy
    from tests.support import session
    from tests.test_gpu_parity import check_rebase, check_scan, check_scan_out, oracle_rebase

    words, t, nb = make(n)
    old = fdy.tune_get(fdy.TUNE_SCAN_TOP_LOG2)
    try:
        fdy.tune_set(fdy.TUNE_SCAN_TOP_LOG2, 4)  # 301 regions do not fit 16 keys: lines and nodes
        check_scan(session, orc, words, t, tag="dense, nodes")
        check_scan_out(session, orc, words, t, nb, tag="dense, nodes")
        check_rebase(session, orc, words, t, nb, tag="dense, nodes")
        units = words.view(np.uint32)[:n + 1 if n > 1 << 20 else 2 * n]
        ref, cnt = orc.scan_stride4(units, t)
        for prepared in (False, True):
            got, have, status = session.scan_stride4(units, t, prepared=prepared, staging=False)
            assert status == 0 and have == cnt and np.array_equal(got, ref)
    finally:
        fdy.tune_set(fdy.TUNE_SCAN_TOP_LOG2, old)


def test_dense_words_of_a_small_table_above_16_mi_words():
    """2,185 chunks, with output."""
    from tests.support import session
    from tests.test_gpu_parity import check_scan_out

    words, t, nb = dense_with_gaps(32768 * SUB + 3)
    check_scan_out(session, orc, words, t, nb, tag="dense, small table, large")


@pytest.mark.parametrize("n_alloc", [300, 20000, 140000])  # level 0 alone, lines, nodes
@pytest.mark.parametrize("n", [200 * SUB, 1500 * SUB, 8000 * SUB])
def test_bounded_wait_and_the_calls_after(n_alloc, n):
    """With a spin limit of 0 a workgroup whose predecessor is not through gives up, says so and ends.
    The chunk states are in order even then: calls on the same prepared table are exact."""
    import paper_2604_06664_amd as fdy
    from tests.support import session
    from tests.test_gpu_flat_scan import table_of, words_of

    rng = np.random.default_rng(n_alloc)
    t = table_of(rng, n_alloc, "spread")
    words = words_of(rng, n, t, 0.25)
    ref, cnt = orc.scan(words, t)
    run = session.ScanRun(words, t, prepared=True)
    for _ in range(2):
        old = fdy.tune_set(fdy.TUNE_SCAN_SPIN_LIMIT, 0)
        try:
            run.launch()
            _, _, status = run.result()
        finally:
            fdy.tune_set(fdy.TUNE_SCAN_SPIN_LIMIT, old)
        assert status & ~(L.ST_SPIN | L.ST_CAPACITY) == 0
        run.d_status.zero_()
        for _ in range(2):
            run.launch()
            got, have, status = run.result()
            assert status == 0 and have == cnt and np.array_equal(got, ref)


@pytest.mark.parametrize("top_log2,n_alloc", [(14, 300), (14, 16384), (14, 20000), (14, 140000), (4, 301)])
@pytest.mark.parametrize("n", [40 * SUB + 3, 1500 * SUB, 8000 * SUB + 511])
def test_one_prepared_table_by_every_form_in_turn(top_log2, n_alloc, n):
    """The same table, scanned by words again and again, by 4-byte positions and with output."""
    import paper_2604_06664_amd as fdy
    from tests.support import session
    from tests.test_gpu_flat_scan import table_of, words_of
    from tests.test_gpu_parity import check_scan_out

    rng = np.random.default_rng(n_alloc + n)
    old = fdy.tune_set(fdy.TUNE_SCAN_TOP_LOG2, top_log2)
    try:
        for shape in ("spread", "run"):
            t = table_of(rng, n_alloc, shape)
            words = words_of(rng, n, t, 0.25)
            ref, cnt = orc.scan(words, t)
            units = words.view(np.uint32)[1:n]
            ref4, cnt4 = orc.scan_stride4(units, t)
            run = session.ScanRun(words, t, prepared=True)
            for again in range(3):
                run.launch()
                got, have, status = run.result()
                assert status == 0 and have == cnt and np.array_equal(got, ref), (shape, again)
            got, have, status = session.scan_stride4(units, t, prepared=False)
            assert status == 0 and have == cnt4 and np.array_equal(got, ref4), shape
            check_scan_out(session, orc, words, t, rng.integers(0, 1 << 63, n_alloc, dtype=np.uint64), tag="in turn")
    finally:
        fdy.tune_set(fdy.TUNE_SCAN_TOP_LOG2, old)


@pytest.mark.parametrize("n_alloc", [300, 20000, 140000])  # level 0 alone, lines, nodes
def test_launches_of_few_and_many_chunks_in_turn(n_alloc):
    """Up to 64 chunks have a state each, more of them share states: calls of both kinds on one prepared table."""
    from tests.support import session
    from tests.test_gpu_flat_scan import table_of, words_of

    rng = np.random.default_rng(n_alloc)
    t = table_of(rng, n_alloc, "spread")
    words = words_of(rng, 1600 * SUB, t, 0.25)
    runs = []
    for n in (1, 7 * SUB, 63 * 7 * SUB, 64 * 7 * SUB - 1, 64 * 7 * SUB, 64 * 7 * SUB + 1, 65 * 7 * SUB, 975 * SUB, 975 * SUB + 1, 1535 * SUB,
              1600 * SUB):
        runs.append((session.ScanRun(words[:n], t), *orc.scan(words[:n], t)))
    big = runs[-1][0]
    big.prepare(len(words))
    for k in rng.permutation(4 * len(runs)):
        run, ref, cnt = runs[k % len(runs)]
        run.d_prepared, run.d_table = big.d_prepared, big.d_table
        run.launch()
        got, have, status = run.result()
        assert status == 0 and have == cnt and np.array_equal(got, ref), run.n_words
