"""Boundaries of graphs in the relocation table, eight to a block behind the graphs' own: graph counts around whole
blocks, graphs without words at either end, a table cut off by its capacity; and nodes per thread of each
remainder that the fold takes apart (four, two, one)."""
import numpy as np
import pytest

import oracle as orc
from synth import layout as L

pytestmark = pytest.mark.gpu
NODES = [1, 511, 512, 513, 1024, 1025, 1536, 1537, 2048, 2049, 2560, 2632, 3072, 3585, 4097]


@pytest.mark.parametrize("G", [1, 2, 6, 7, 8, 9, 15, 16, 17])
@pytest.mark.parametrize("cut", [False, True])
def test_boundaries_and_fold(G, cut):
    import torch

    import paper_2604_06664_amd as fdy
    from tests.support import session
    from tests.test_gpu_flat_scan import table_of, words_of

    rng = np.random.default_rng(G)
    t = table_of(rng, 500, "spread")
    words = words_of(rng, 70_001, t, 0.3)
    words[-900:] = 5  # the last graphs have words and no relocation
    ref, cnt = orc.scan(words, t)
    run = session.ScanRun(words, t, prepared=True)
    run.launch()
    got, n, st = run.result()
    assert st == 0 and n == cnt and np.array_equal(got, ref)
    counts = [NODES[(G + i) % len(NODES)] for i in range(G)]
    nodes = rng.integers(0, 1 << 32, (sum(counts), 10), dtype=np.uint32).view(L.NODE).reshape(-1)
    node_off = np.cumsum([0] + counts).astype(np.uint64)
    inner = np.sort(np.r_[rng.integers(0, len(words) + 1, G), [0, 0, len(words) - 1, len(words)]])[:G - 1] if G > 1 else []
    word_off = np.r_[0, inner, len(words)].astype(np.uint64)
    keys, tid, tg = orc.fingerprint(nodes, node_off, L.FP_ALL)
    capacity = cnt // 2 if cut else run.capacity
    want = orc.reloc_segment(ref[:capacity], word_off)
    d_word_off, d_nodes, d_node_off = fdy.to_device(word_off), fdy.to_device(nodes), fdy.to_device(node_off)
    d_roff, d_keys = fdy.device_bytes((G + 1) * 8, fill=0xEE), fdy.device_bytes(G * 8, fill=0xEE)
    d_tid, d_tg = fdy.device_bytes(G * 4, fill=0xEE), fdy.device_bytes(G * 4, fill=0xEE)
    d_nt = torch.full((1,), -1, dtype=torch.int32, device="cuda:0")
    for prepared in (run.d_prepared, run.d_prepared):
        fdy.fdy_segment_fingerprint(run.d_relocs, run.d_count, capacity, d_word_off, d_roff, d_nodes, d_node_off, G,
                                    L.FP_ALL, d_keys, d_tid, d_tg, d_nt, d_prepared=prepared)
        torch.cuda.synchronize()
        assert np.array_equal(fdy.to_host(d_roff, np.uint64, G + 1), want)
        assert np.array_equal(fdy.to_host(d_keys, np.uint64, G), keys)
        assert np.array_equal(fdy.to_host(d_tid, np.uint32, G), tid)
        assert np.array_equal(fdy.to_host(d_tg, np.uint32, len(tg)), tg)
