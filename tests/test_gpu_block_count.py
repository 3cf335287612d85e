"""The count of finished blocks in a prepared table's first lines: archives of graph counts around the one
(160) from which four counters share it, one after the other on one prepared table, with scans in
between; graphs of no nodes, one, and more than a block's threads."""
import numpy as np
import pytest

import oracle as orc
from synth import layout as L

pytestmark = pytest.mark.gpu


def test_counts_of_any_size_in_turn():
    import torch

    import paper_2604_06664_amd as fdy
    from tests.support import session
    from tests.test_gpu_flat_scan import table_of, words_of

    rng = np.random.default_rng(160)
    t = table_of(rng, 500, "spread")
    words = words_of(rng, 9000, t, 0.3)
    ref, cnt = orc.scan(words, t)
    run = session.ScanRun(words, t, prepared=True)
    for G in (161, 1, 160, 512, 2, 162, 163, 164, 160, 1000, 8192, 161, 8191, 512):
        # graphs drawn from a few sequences, so that they group
        kinds = [rng.integers(0, 1 << 32, (n, 10), dtype=np.uint32).view(L.NODE).reshape(-1) for n in (0, 1, 7, 513, 40)]
        pick = rng.integers(0, len(kinds), G)
        nodes = np.concatenate([kinds[k] for k in pick])
        node_off = np.concatenate([[0], np.cumsum([len(kinds[k]) for k in pick])]).astype(np.uint64)
        word_off = np.sort(np.concatenate([[0, len(words)], rng.integers(0, len(words) + 1, G - 1)])).astype(np.uint64)
        keys, tid, tg = orc.fingerprint(nodes, node_off, L.FP_ALL)
        run.launch()
        got, n, st = run.result()
        assert st == 0 and n == cnt and np.array_equal(got, ref), G
        d_word_off, d_nodes, d_node_off = fdy.to_device(word_off), fdy.to_device(nodes), fdy.to_device(node_off)
        for _ in range(2):
            d_roff, d_keys = fdy.device_bytes((G + 1) * 8, fill=0xEE), fdy.device_bytes(G * 8, fill=0xEE)
            d_tid, d_tg = fdy.device_bytes(G * 4, fill=0xEE), fdy.device_bytes(G * 4, fill=0xEE)
            d_nt = torch.full((1,), -1, dtype=torch.int32, device="cuda:0")
            fdy.fdy_segment_fingerprint(run.d_relocs, run.d_count, run.capacity, d_word_off, d_roff, d_nodes, d_node_off, G,
                                        L.FP_ALL, d_keys, d_tid, d_tg, d_nt, d_prepared=run.d_prepared)
            torch.cuda.synchronize()
            nt = int(d_nt.item())
            assert nt == len(tg), G
            assert np.array_equal(fdy.to_host(d_roff, np.uint64, G + 1), orc.reloc_segment(ref, word_off)), G
            assert np.array_equal(fdy.to_host(d_keys, np.uint64, G), keys), G
            assert np.array_equal(fdy.to_host(d_tid, np.uint32, G), tid), G
            assert np.array_equal(fdy.to_host(d_tg, np.uint32, nt), tg), G
