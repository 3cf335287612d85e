"""Override derivation where its launches change: tiles with as many differing halves as a slot
holds and one more, more graphs than a workgroup sums itself, more tiles than a workgroup counts
back over."""
import numpy as np
import pytest

import oracle as orc

pytestmark = pytest.mark.gpu

TILE, SLOT = 2048, 32


def check(words, word_off, gt, tg, capacity=None):
    from tests.support import session
    from tests.test_gpu_parity import check_derive

    check_derive(session, orc, words, word_off, gt, tg, capacity=capacity)


def flipped(rng, base, n):
    """base with n of its 32-bit halves changed."""
    h = base.view(np.uint32).copy()
    at = rng.choice(len(h), n, replace=False)
    h[at] ^= rng.integers(1, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
    return h.view(np.uint64)


@pytest.mark.parametrize("n", [0, 1, SLOT - 1, SLOT, SLOT + 1, 2 * TILE])
def test_entries_per_tile(n):
    rng = np.random.default_rng(n)
    base = rng.integers(0, 1 << 64, TILE, dtype=np.uint64)
    parts = [base, flipped(rng, base, n), base[:1], flipped(rng, base, 3), flipped(rng, base, n)]
    off = np.cumsum([0] + [len(p) for p in parts]).astype(np.uint64)
    words = np.concatenate(parts)
    check(words, off, [0, 0, 1, 0, 0], [0, 2])
    check(words, off, [0, 0, 1, 0, 0], [0, 2], capacity=n + 2)


@pytest.mark.parametrize("graphs", [1, 1023, 1024, 1025])
def test_graphs(graphs):
    rng = np.random.default_rng(graphs)
    base = rng.integers(0, 1 << 64, 70, dtype=np.uint64)
    parts = [base] + [flipped(rng, base, i % 5) if i % 7 else base[:0] for i in range(1, graphs)]
    off = np.cumsum([0] + [len(p) for p in parts]).astype(np.uint64)
    empty = next((i for i, p in enumerate(parts) if not len(p)), 0)
    check(np.concatenate(parts), off, [0 if len(p) else 1 for p in parts], [0, empty])


@pytest.mark.parametrize("graphs", [400, 409, 420])  # the launches are sized for tiles + graphs
def test_many_tiles(graphs):
    rng = np.random.default_rng(graphs)
    base = rng.integers(0, 1 << 64, 9 * TILE + 5, dtype=np.uint64)
    parts = [base] + [flipped(rng, base, int(rng.integers(0, 90))) for _ in range(graphs - 1)]
    off = np.cumsum([0] + [len(p) for p in parts]).astype(np.uint64)
    check(np.concatenate(parts), off, [0] * graphs, [0])


@pytest.mark.parametrize("n", [1, 256, 511, 512, 513, 1023, 1024, 1025, 1535, 1536, 1537, 2047, 2048, 2049, TILE + 512, TILE + 513])
def test_lengths_around_whole_requests(n):
    """A short tile asks for two, four, six or eight rounds of words: differences at both ends of each round."""
    rng = np.random.default_rng(n)
    base = rng.integers(0, 1 << 64, n, dtype=np.uint64)
    at = sorted({k for e in range(0, n + 1, 256) for k in (e - 1, e) if 0 <= k < n} | {n - 1})
    few, all_differ = base.copy(), base ^ np.uint64(0x100000001)
    few[at[:15] + at[-1:]] ^= np.uint64(1 << 40)
    ends = base.copy()
    ends[at] ^= np.uint64(0x8000000000000001)
    parts = [base, few, ends, all_differ, base]
    off = np.cumsum([0] + [len(p) for p in parts]).astype(np.uint64)
    check(np.concatenate(parts), off, [0] * len(parts), [0])
