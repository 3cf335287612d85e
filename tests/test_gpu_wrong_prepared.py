"""A prepared table that is not the call's own: every form of the scan says so and changes nothing,
neither the buffer nor what lies behind it, also where the call's table is much the larger."""
import numpy as np
import pytest

from synth import layout as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mine,other", [(300, 20000), (20000, 70000), (20000, 300), (20000, 20000)])
def test_nothing_is_written(mine, other):
    """Prepared for `mine` allocations, called with a table of `other`."""
    import torch

    import paper_2604_06664_amd as fdy
    from tests.test_gpu_flat_scan import table_of, words_of

    rng = np.random.default_rng(mine)
    t, u = table_of(rng, mine, "spread"), table_of(rng, other, "spread")
    n = 50_000
    d_t, d_u = fdy.to_device(t), fdy.to_device(u)
    d_words = fdy.to_device(words_of(rng, n, u, 0.3))
    d_nb = fdy.to_device(rng.integers(0, 1 << 63, other, dtype=np.uint64))
    size = fdy.fdy_scan_table_bytes(mine, n)
    whole = fdy.device_bytes(max(size, fdy.fdy_scan_table_bytes(other, n)) + 4096, fill=0x5A)
    fdy.fdy_scan_table_prepare(d_t, mine, n, whole[:size], size)
    torch.cuda.synchronize()
    before = whole.clone()
    d_rel, d_out = fdy.device_bytes(n * 16, fill=0xEE), fdy.device_bytes(n * 8, fill=0xEE)
    d_count = torch.full((1,), -1, dtype=torch.int64, device="cuda:0")
    d_status = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    rest = (whole[:size], None, 0, d_status)
    calls = [
        lambda: fdy.fdy_scan_pointers(d_words, n, d_u, other, d_rel, n, d_count, *rest),
        lambda: fdy.fdy_scan_pointers_stride4(d_words, n, d_u, other, d_rel, n, d_count, *rest),
        lambda: fdy.fdy_scan_pointers_rebase(d_words, n, d_u, other, d_rel, n, d_count, d_nb, d_out, *rest),
        lambda: fdy.fdy_scan_rebase(d_words, n, d_u, other, d_nb, d_out, d_count, *rest),
    ]
    for call in calls:
        d_status.zero_()
        call()
        torch.cuda.synchronize()
        assert int(d_status.item()) == L.ST_BAD_PREPARED and int(d_count.item()) == -1
        assert torch.equal(whole, before)
        assert bool((d_rel == 0xEE).all()) and bool((d_out == 0xEE).all())
