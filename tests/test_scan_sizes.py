"""What a scan asks of its caller's buffers: a buffer that serves a table serves every smaller one,
and chunk states take 8 bytes per 4,096 words whatever the table (small tables are asked for up to
32 KiB more, and work without)."""
import numpy as np
import pytest

import oracle as orc
from synth import layout as L

ALLOCS = [0, 1, 2, 3, 16, 255, 1000, 4096, 16383, 16384, 16385, 20000, 65536, 131072, 131073, 1 << 20, (1 << 20) + 1,
          1 << 21, (1 << 21) + 1, 1 << 22, (1 << 22) + 1, 1 << 23, (1 << 23) + 1, 1 << 25, (1 << 25) + 1, 1 << 28,
          (1 << 28) + 1, (1 << 31) - 1, 1 << 31, (1 << 32) - 1]
WORDS = [0, 1, 511, 4096, 100_000, 786_431, 1 << 20, (1 << 24) - 1, 1 << 24, 1 << 27, (1 << 32) - 256]


@pytest.mark.parametrize("n_words", WORDS)
def test_sizes_grow_with_the_table(n_words):
    import paper_2604_06664_amd as fdy

    for size in (lambda a: fdy.fdy_scan_workspace_bytes(n_words, a), lambda a: fdy.fdy_scan_table_bytes(a, n_words)):
        got = [size(a) for a in ALLOCS]
        assert got == sorted(got)


def least(size, n_words):
    """Bytes that a call with n_words cannot do without; size(n): the library's answer for n words."""
    return size(0) + (-(-n_words // 4096) * 8 + 255) // 256 * 256


@pytest.mark.parametrize("n_alloc", ALLOCS)
def test_chunk_states_take_8_bytes_per_4096_words(n_alloc):
    import paper_2604_06664_amd as fdy

    for size in (lambda n: fdy.fdy_scan_workspace_bytes(n, n_alloc), lambda n: fdy.fdy_scan_table_bytes(n_alloc, n)):
        for n in WORDS:
            more = size(n) - least(size, n)
            assert 0 <= more <= (32768 if n_alloc <= 16384 else 0), n


@pytest.mark.gpu
@pytest.mark.parametrize("max_words", [9 * 512, 786_431, 1535 * 512, 3_700_001, (1 << 24) - 1, (1 << 24) + 5])
@pytest.mark.parametrize("n_alloc", [2, 300, 16384])
@pytest.mark.parametrize("tight", [False, True])
def test_buffers_of_exactly_these_sizes_serve_every_form(n_alloc, max_words, tight):
    """Sequences of calls of every form and many lengths over one prepared table and one workspace,
    with bytes around both that must not change."""
    import torch

    import paper_2604_06664_amd as fdy
    from tests.test_gpu_flat_scan import table_of, words_of
    from tests.test_gpu_parity import oracle_rebase

    rng = np.random.default_rng(n_alloc + max_words)
    t = table_of(rng, n_alloc, "spread")
    words = np.tile(words_of(rng, 1 << 20, t, 0.2), 17)[:max_words]
    new_base = rng.integers(0, 1 << 63, n_alloc, dtype=np.uint64)
    ref, _ = orc.scan(words, t)
    want, _ = oracle_rebase(orc, words, t, new_base)
    d_words, d_table, d_nb = fdy.to_device(words), fdy.to_device(t), fdy.to_device(new_base)
    d_rel, d_out = fdy.device_bytes(max_words * 16, fill=0xEE), fdy.device_bytes(max_words * 8, fill=0xEE)
    d_count = torch.zeros(1, dtype=torch.int64, device="cuda:0")
    d_status = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    pb = fdy.fdy_scan_table_bytes(n_alloc, max_words)
    wb = fdy.fdy_scan_workspace_bytes(max_words, n_alloc)
    if tight:
        pb = least(lambda n: fdy.fdy_scan_table_bytes(n_alloc, n), max_words)
        wb = least(lambda n: fdy.fdy_scan_workspace_bytes(n, n_alloc), max_words)
    prep, ws = fdy.device_bytes(pb + 512, fill=0x5A), fdy.device_bytes(wb + 512, fill=0x5A)
    d_prep, d_ws = prep[256:256 + pb], ws[256:256 + wb]
    fdy.fdy_scan_table_prepare(d_table, n_alloc, max_words, d_prep, pb)
    lengths = [max_words, 1, max_words, 4097, min(max_words, 1536 * 512 + 7), 1000, max_words, max_words]
    for i, n in enumerate(lengths):
        for form in ("scan", "out", "rebase"):
            rest = (None, d_ws, wb, d_status) if i % 4 == 3 else (d_prep, None, 0, d_status)
            d_out.fill_(0xEE)
            if form == "scan":
                fdy.fdy_scan_pointers(d_words, n, d_table, n_alloc, d_rel, max_words, d_count, *rest)
            elif form == "out":
                fdy.fdy_scan_pointers_rebase(d_words, n, d_table, n_alloc, d_rel, max_words, d_count, d_nb, d_out, *rest)
            else:
                fdy.fdy_scan_rebase(d_words, n, d_table, n_alloc, d_nb, d_out, d_count, *rest)
            torch.cuda.synchronize()
            cnt = int(np.searchsorted(ref["word"], n))
            assert int(d_status.item()) == 0 and int(d_count.item()) == cnt, (n, form)
            if form != "rebase":
                assert np.array_equal(fdy.to_host(d_rel, L.RELOC, cnt), ref[:cnt]), (n, form)
            if form != "scan":
                assert np.array_equal(fdy.to_host(d_out, np.uint64, n), want[:n]), (n, form)
    for whole, size in ((prep, pb), (ws, wb)):
        assert bool((whole[:256] == 0x5A).all()) and bool((whole[256 + size:] == 0x5A).all())


@pytest.mark.gpu
def test_a_buffer_for_the_largest_table_serves_the_smaller_ones():
    import torch

    import paper_2604_06664_amd as fdy
    from tests.test_gpu_flat_scan import table_of, words_of

    rng = np.random.default_rng(8)
    n = 3_000_001
    pb, wb = fdy.fdy_scan_table_bytes(20000, n), fdy.fdy_scan_workspace_bytes(n, 20000)
    d_prep, d_ws = fdy.device_bytes(pb, fill=0x33), fdy.device_bytes(wb, fill=0x33)
    d_rel = fdy.device_bytes(n * 16)
    d_count = torch.zeros(1, dtype=torch.int64, device="cuda:0")
    d_status = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    for n_alloc in (20000, 16385, 16384, 5000, 17, 1):
        t = table_of(rng, n_alloc, "spread")
        words = words_of(rng, n, t, 0.2)
        d_words, d_table = fdy.to_device(words), fdy.to_device(t)
        ref, cnt = orc.scan(words, t)
        fdy.fdy_scan_table_prepare(d_table, n_alloc, n, d_prep, pb)
        for rest in ((d_prep, None, 0, d_status), (None, d_ws, wb, d_status)):
            fdy.fdy_scan_pointers(d_words, n, d_table, n_alloc, d_rel, n, d_count, *rest)
            torch.cuda.synchronize()
            assert int(d_status.item()) == 0 and int(d_count.item()) == cnt
            assert np.array_equal(fdy.to_host(d_rel, L.RELOC, cnt), ref)
