"""Tables of one to five regions through every form of the scan, over buffers whose contents on entry
would be taken for keys, with entries behind the table and the base map that would be found."""
import numpy as np
import pytest

import oracle as orc
from synth import layout as L

pytestmark = pytest.mark.gpu

GIB = 1 << 30
TABLES = {
    # a small region below a large one: both bases in the lower half of the key space
    "small, large": [(0x7F0000000000, 2 << 20), (0x7F0000200000, GIB)],
    "page, MiB": [(0x1000, 0x1000), (0x3000, 0x100000)],
    "touching": [(4096, 16), (4112, 1 << 40)],
    "large, small": [(0x7F0000000000, GIB), (0x7F0040000000, 512)],
    "one": [(0x7F0000000000, 4096)],
    "three": [(4096, 16), (4112, 16), (8192, GIB)],
    "five": [(4096, 16), (4112, 16), (4128, 16), (8192, GIB), (1 << 46, 1 << 20)],
}


@pytest.mark.parametrize("fill", [0x00, 0x10, 0xFF])
@pytest.mark.parametrize("name", list(TABLES))
def test_few_regions(name, fill):
    import torch

    import paper_2604_06664_amd as fdy
    from tests.test_gpu_parity import oracle_rebase

    t = np.array(TABLES[name], L.ALLOC)
    n_alloc, n = len(t), 9 * 512 + 3
    rng = np.random.default_rng(n_alloc)
    base, size = t["base"], t["size"]
    one = np.uint64(1)
    edge = np.concatenate([base - one, base, base + one, base + size // np.uint64(2), base + size - one, base + size,
                           base + size + one, base + np.uint64(16)])
    words = np.where(rng.random(n) < 0.7, rng.choice(edge, n), rng.integers(0, 1 << 63, n, dtype=np.uint64))
    new_base = rng.integers(0, 1 << 63, n_alloc, dtype=np.uint64)
    # entries behind the table hold every word, and their new bases would show in the output
    guard = np.zeros(4, L.ALLOC)
    guard["size"] = ~np.uint64(0)
    d_table = fdy.to_device(np.concatenate([t, guard]))
    d_nb = fdy.to_device(np.concatenate([new_base, np.full(4, 0xBAD << 40, np.uint64)]))
    ref, cnt = orc.scan(words, t)
    want, _ = oracle_rebase(orc, words, t, new_base)
    units = words.view(np.uint32)
    ref4, cnt4 = orc.scan_stride4(units, t)

    d_words, cap = fdy.to_device(words), 2 * n
    d_rel, d_out = fdy.device_bytes(cap * 16, fill=0xEE), fdy.device_bytes(n * 8, fill=0xEE)
    d_count = torch.zeros(1, dtype=torch.int64, device="cuda:0")
    d_status = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    ws_bytes = fdy.fdy_scan_workspace_bytes(2 * n, n_alloc)
    pb = fdy.fdy_scan_table_bytes(n_alloc, 2 * n)
    for prepared in (False, True):
        d_ws, d_prep = fdy.device_bytes(ws_bytes, fill=fill), None
        if prepared:
            d_prep = fdy.device_bytes(pb, fill=fill)
            fdy.fdy_scan_table_prepare(d_table, n_alloc, 2 * n, d_prep, pb)
        rest = (d_prep, None if prepared else d_ws, 0 if prepared else ws_bytes, d_status)

        def check(what, relocs, count, out):
            torch.cuda.synchronize()
            where = (what, prepared)
            assert int(d_status.item()) == 0 and int(d_count.item()) == count, where
            if relocs is not None:
                assert np.array_equal(fdy.to_host(d_rel, L.RELOC, count), relocs), where
            if out is not None:
                assert np.array_equal(fdy.to_host(d_out, np.uint64, n), out), where
            d_ws.fill_(fill)

        fdy.fdy_scan_pointers(d_words, n, d_table, n_alloc, d_rel, cap, d_count, *rest)
        check("scan", ref, cnt, None)
        fdy.fdy_scan_pointers_stride4(d_words, 2 * n, d_table, n_alloc, d_rel, cap, d_count, *rest)
        check("stride4", ref4, cnt4, None)
        fdy.fdy_scan_pointers_rebase(d_words, n, d_table, n_alloc, d_rel, cap, d_count, d_nb, d_out, *rest)
        check("out", ref, cnt, want)
        d_out.fill_(0xEE)
        fdy.fdy_scan_rebase(d_words, n, d_table, n_alloc, d_nb, d_out, d_count, *rest)
        check("rebase", None, cnt, want)
