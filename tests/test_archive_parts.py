"""Archives large enough to be summed and checked in several parts: every part's damage is found and named as in one pass."""
import numpy as np
import pytest

from paper_2604_06664_amd import archive as far
from synth import layout as L

G, PER = 37, 3001  # words of a graph


@pytest.fixture(scope="module")
def sections():
    rng = np.random.default_rng(3)
    table = np.zeros(512, L.ALLOC)
    table["base"], table["size"] = 0x10000 + np.arange(512, dtype=np.uint64) * 0x2000, 0x1000
    region, offset = rng.integers(0, 512, G * PER), rng.integers(0, 0x1000, G * PER).astype(np.uint64)
    relocs = np.zeros(G * PER, L.RELOC)
    relocs["word"], relocs["region"], relocs["offset"] = np.arange(G * PER), region, offset
    keep = rng.random(G * PER) < 0.9
    keep[PER:3 * PER] = False  # graphs without any
    relocs = relocs[keep]
    nodes = np.zeros(G * 3, L.NODE)
    nodes["blob_len"] = np.tile([8, 16, (PER - 3) * 8], G)
    zeros = np.zeros(G + 1, np.uint64)
    return {
        far.FDY_SEC_TABLE: table, far.FDY_SEC_WORDS: table["base"][region] + offset,
        far.FDY_SEC_WORD_OFF: np.arange(G + 1, dtype=np.uint64) * np.uint64(PER), far.FDY_SEC_NODES: nodes,
        far.FDY_SEC_NODE_OFF: np.arange(G + 1, dtype=np.uint64) * np.uint64(3), far.FDY_SEC_RELOCS: relocs,
        far.FDY_SEC_RELOC_OFF: np.searchsorted(relocs["word"], np.arange(G + 1) * PER).astype(np.uint64),
        far.FDY_SEC_GRAPH_TMPL: np.arange(G, dtype=np.uint32), far.FDY_SEC_TMPL_GRAPH: np.arange(G, dtype=np.uint32),
        far.FDY_SEC_OVR: np.zeros(0, L.OVR32), far.FDY_SEC_OVR_OFF: zeros, far.FDY_SEC_GOVR: np.zeros(0, L.GRID_OVR),
        far.FDY_SEC_GOVR_OFF: zeros}


def test_sums_of_parts(sections, tmp_path):
    path = str(tmp_path / "a")
    far.fdy_archive_write(path, list(sections.items()))
    data = bytearray(open(path, "rb").read())
    assert len(data) > 2 << 20
    far.fdy_archive_close(far.fdy_archive_open(path, far.FDY_ARCHIVE_VERIFY_SUMS))
    words = sections[far.FDY_SEC_WORDS].tobytes()
    first = bytes(data).index(words[:64])
    relocs = bytes(data).index(sections[far.FDY_SEC_RELOCS].tobytes()[:64])
    n_rel = sections[far.FDY_SEC_RELOCS].nbytes
    for at in (first, first + len(words) // 2, first + len(words) - 1, relocs, relocs + n_rel // 4 - 1, relocs + n_rel // 4 + 64,
               relocs + n_rel // 2, relocs + n_rel - 1):
        bad = bytearray(data)
        bad[at] ^= 0x10
        open(path, "wb").write(bad)
        with pytest.raises(Exception):
            far.fdy_archive_open(path, far.FDY_ARCHIVE_VERIFY_SUMS)
        far.fdy_archive_close(far.fdy_archive_open(path, 0))


@pytest.mark.parametrize("graph", [0, 1, 3, 17, 18, 30, G - 1])
def test_contents_of_parts(sections, tmp_path, graph):
    path = str(tmp_path / "a")
    off = sections[far.FDY_SEC_RELOC_OFF]

    def verdict(**changed):
        far.fdy_archive_write(path, [(k, changed.get(str(k), v)) for k, v in sections.items()])
        a = far.fdy_archive_open(path, 0)
        try:
            far.fdy_archive_check(a)
            return ""
        except Exception:
            return far.fdy_archive_last_failure()
        finally:
            far.fdy_archive_close(a)

    assert verdict() == ""
    nodes = sections[far.FDY_SEC_NODES].copy()
    nodes["blob_len"][graph * 3] += 8
    assert verdict(**{str(far.FDY_SEC_NODES): nodes})
    i, end = int(off[graph]), int(off[graph + 1])
    if i == end:  # (no relocations)
        return
    for field, at, value in (("word", i, graph * PER - 1 if graph else PER), ("word", end - 1, (graph + 1) * PER),
                             ("region", i + 5, 512), ("offset", end - 1, 0x1000), ("word", i + 1, graph * PER)):
        relocs = sections[far.FDY_SEC_RELOCS].copy()
        relocs[field][at] = value
        assert verdict(**{str(far.FDY_SEC_RELOCS): relocs}), (field, at)
    words = sections[far.FDY_SEC_WORDS].copy()
    words[sections[far.FDY_SEC_RELOCS]["word"][end - 1]] ^= np.uint64(8)
    assert verdict(**{str(far.FDY_SEC_WORDS): words})
