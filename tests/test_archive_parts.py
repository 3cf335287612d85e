"""Archives that are summed and checked in several parts, by their size and by force: damage on both sides of every cut is
found, and named as in one pass."""
import struct

import numpy as np
import pytest

import paper_2604_06664_amd as fdy
from paper_2604_06664_amd import archive as far
from synth import layout as L

G, PER = 41, 9001  # graphs, words of each
PARTS = [0, 1, 2, 3, 4]  # 0: by size
MIB = 1 << 20


def make_sections(graphs, per):
    rng = np.random.default_rng(3)
    n = graphs * per
    table = np.zeros(512, L.ALLOC)
    table["base"], table["size"] = 0x10000 + np.arange(512, dtype=np.uint64) * 0x2000, 0x1000
    region, offset = rng.integers(0, 512, n), rng.integers(0, 0x1000, n).astype(np.uint64)
    relocs = np.zeros(n, L.RELOC)
    relocs["word"], relocs["region"], relocs["offset"] = np.arange(n), region, offset
    keep = rng.random(n) < 0.9
    keep[per:3 * per] = False  # graphs without any
    relocs = relocs[keep]
    nodes = np.zeros(graphs * 3, L.NODE)
    nodes["blob_len"] = np.tile([8, 16, (per - 3) * 8], graphs)
    zeros = np.zeros(graphs + 1, np.uint64)
    return {
        far.FDY_SEC_TABLE: table, far.FDY_SEC_WORDS: table["base"][region] + offset,
        far.FDY_SEC_WORD_OFF: np.arange(graphs + 1, dtype=np.uint64) * np.uint64(per), far.FDY_SEC_NODES: nodes,
        far.FDY_SEC_NODE_OFF: np.arange(graphs + 1, dtype=np.uint64) * np.uint64(3), far.FDY_SEC_RELOCS: relocs,
        far.FDY_SEC_RELOC_OFF: np.searchsorted(relocs["word"], np.arange(graphs + 1) * per).astype(np.uint64),
        far.FDY_SEC_GRAPH_TMPL: np.arange(graphs, dtype=np.uint32), far.FDY_SEC_TMPL_GRAPH: np.arange(graphs, dtype=np.uint32),
        far.FDY_SEC_OVR: np.zeros(0, L.OVR32), far.FDY_SEC_OVR_OFF: zeros, far.FDY_SEC_GOVR: np.zeros(0, L.GRID_OVR),
        far.FDY_SEC_GOVR_OFF: zeros}


class Archive:
    """An archive file, its sections writable in place."""

    def __init__(self, path, graphs, per):
        self.path, self.sections = str(path), make_sections(graphs, per)
        far.fdy_archive_write(self.path, list(self.sections.items()))
        self.bytes = np.memmap(self.path, np.uint8, "r+")
        self.at, self.live = {}, {}
        for i in range(len(self.sections)):
            kind, _, at, count, _ = struct.unpack_from("<IIQQQ", self.bytes, 64 + 32 * i)
            if count:
                data = self.sections[kind]
                self.at[kind], self.live[kind] = at, self.bytes[at:at + data.nbytes].view(data.dtype)

    def open(self, flags):
        self.bytes.flush()
        return far.fdy_archive_open(self.path, flags, check=False)

    def check(self):
        rc, a = self.open(0)
        assert rc == 0
        try:
            rc, _ = far.fdy_archive_check(a, check=False)
            return rc, far.fdy_archive_last_failure()
        finally:
            far.fdy_archive_close(a)


@pytest.fixture(scope="module")
def archive(tmp_path_factory):
    return Archive(tmp_path_factory.mktemp("parts") / "a", G, PER)


@pytest.fixture(params=PARTS)
def parts(request):
    old = fdy.tune_set(fdy.TUNE_ARCHIVE_PARTS, request.param)
    assert old == 0
    yield request.param
    fdy.tune_set(fdy.TUNE_ARCHIVE_PARTS, old)


def test_the_archive_is_as_large_as_the_most_parts_want(archive):
    s = archive.sections
    assert s[far.FDY_SEC_RELOCS].nbytes + s[far.FDY_SEC_NODES].nbytes >= 4 * MIB


def damage_sums(archive, places):
    name = {v: n[len("FDY_SEC_"):] for n, v in vars(far).items() if n.startswith("FDY_SEC_") and not n.endswith("KIND_MAX")}
    for kind, byte in places:
        archive.bytes[archive.at[kind] + byte] ^= 0x10
        rc, a = archive.open(far.FDY_ARCHIVE_VERIFY_SUMS)
        archive.bytes[archive.at[kind] + byte] ^= 0x10
        assert (rc, far.fdy_archive_last_failure()) == (far.FDY_ERR_CHECKSUM, f"section {name[kind]}: sum does not match")
    rc, a = archive.open(far.FDY_ARCHIVE_VERIFY_SUMS)
    assert rc == 0
    far.fdy_archive_close(a)


def test_sums(archive, parts):
    kinds = list(archive.sections)
    ends = np.cumsum([archive.sections[k].nbytes for k in kinds])
    places = []
    for n in range(1, 5):
        for cut in [int(ends[-1]) // n * k for k in range(n)] + [int(ends[-1])]:
            for byte in (cut - 65, cut - 1, cut, cut + 64):
                if 0 <= byte < ends[-1]:
                    i = int(np.searchsorted(ends, byte, side="right"))
                    places.append((kinds[i], byte - (int(ends[i - 1]) if i else 0)))
    for k in kinds:  # the ends of every section, with a partial last word among them
        if archive.sections[k].nbytes:
            places += [(k, 0), (k, archive.sections[k].nbytes - 1)]
    damage_sums(archive, sorted(set(places)))


@pytest.mark.parametrize("graphs,per", [(1, 4), (2, 5), (5, 64)])
def test_sums_of_archives_smaller_than_their_parts_want(graphs, per, parts, tmp_path):
    a = Archive(tmp_path / "small", graphs, per)
    assert a.check() == (0, "")
    damage_sums(a, [(k, byte) for k in a.at for byte in (0, a.sections[k].nbytes - 1)])


def test_contents(archive, parts):
    assert archive.check() == (0, "")
    off = archive.sections[far.FDY_SEC_RELOC_OFF].astype(np.int64)
    n = int(off[-1])
    cuts = {int(np.searchsorted(off[:-1], n * i // k)) for k in (2, 3, 4) for i in range(1, k)}
    assert len(cuts) >= 5
    graphs = {0, 1, 2, 3, G - 1} | cuts | {c - 1 for c in cuts}
    nodes, relocs, words = (archive.live[k] for k in (far.FDY_SEC_NODES, far.FDY_SEC_RELOCS, far.FDY_SEC_WORDS))

    def damaged(array, field, at, value, text, more=None):
        old = array[at].copy()
        if field:
            array[field][at] = value
        else:
            array[at] = value
        got = more() if more else archive.check()
        array[at] = old
        assert got == (far.FDY_ERR_CONTENT, text), (field, at)

    def all_of(g, more=None):
        def hurt(array, field, at, value, text):
            damaged(array, field, at, value, text, more)

        hurt(nodes, "blob_len", 3 * g + 1, 17, f"NODES: node {3 * g + 1} has a blob length that is not a multiple of 8")
        hurt(nodes, "blob_len", 3 * g + 2, PER * 8, f"source graph {g}: blob lengths of its nodes do not add up to its words")
        first, last = int(off[g]), int(off[g + 1]) - 1
        if last < first:
            return
        order = "RELOCS: entry {} is outside its graph's words or not ascending".format
        table = "RELOCS: entry {} names a region or offset outside the table".format
        hurt(relocs, "word", first, g * PER - 1 if g else PER, order(first))
        hurt(relocs, "word", first + 1, int(relocs["word"][first]), order(first + 1))
        hurt(relocs, "word", last, (g + 1) * PER, order(last))
        hurt(relocs, "region", first, 512, table(first))
        hurt(relocs, "offset", last, 0x1000, table(last))
        same = "RELOCS: entry {} does not match the word it describes".format
        hurt(words, None, int(relocs["word"][first]), words[relocs["word"][first]] ^ np.uint64(8), same(first))
        hurt(words, None, int(relocs["word"][last]), words[relocs["word"][last]] ^ np.uint64(8), same(last))

    for g in sorted(graphs):
        all_of(g)

    # damage further on does not hide what is wrong first
    def with_more_behind():
        old = nodes[3 * (G - 1)].copy()
        nodes["blob_len"][3 * (G - 1)] = 9
        got = archive.check()
        nodes[3 * (G - 1)] = old
        return got

    for g in sorted(graphs - {G - 1}):
        all_of(g, with_more_behind)
    assert archive.check() == (0, "")
