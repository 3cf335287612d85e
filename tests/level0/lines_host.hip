// Lines and nodes of the table hierarchy (csrc/fdy_lines.hpp), compiled for the host under
// AddressSanitizer: what is packed from a table is searched with words around every edge of it,
// and the entry found is compared with the definition; tables that no valid layout has must not
// lead outside the table.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "fdy_level0.hpp"
#include "fdy_lines.hpp"

using namespace fdy;

namespace {

u64 rng = 0x9e3779b97f4a7c15ull;
u64 next() {  // xorshift64
  rng ^= rng << 13;
  rng ^= rng >> 7;
  return rng ^= rng << 17;
}
u64 below(u64 n) { return next() % n; }
u64 log_uniform(int lo, int hi) {  // between 2^lo and 2^hi
  const int b = lo + (int)below(hi - lo + 1);
  return (1ull << b) | (next() & ((1ull << b) - 1));
}

int failures = 0;
unsigned long long runs = 0, compact_lines = 0, wide_lines = 0, nodes = 0;

struct Table {
  fdy_alloc* t;  // a heap block of its exact size
  u32 n;
  explicit Table(const std::vector<fdy_alloc>& v) : n((u32)v.size()) {
    t = (fdy_alloc*)aligned_alloc(16, n * sizeof(fdy_alloc));
    memcpy(t, v.data(), n * sizeof(fdy_alloc));
  }
  ~Table() { free(t); }
};

void report(const char* what, const Table& t, u64 w, u32 line) {
  if (++failures <= 10) printf("%s: word %llx, line %u of %u entries\n", what, (unsigned long long)w, line, t.n);
}

// The last entry at or below w among the first n, by the definition (0 if there is none).
u32 last_below(const Table& t, u32 n, u64 w) {
  u32 want = 0;
  for (u32 k = 0; k < n; ++k)
    if (t.t[k].base <= w) want = k;
  return want;
}

// The entry found in `line`, as the kernels do: the form asked for, the wide one, the table.
void search_line(const Table& t, u32 line, u64 w, u64 told, bool valid) {
  PackedLine l;
  pack_line(t.t, (u64)line * 8, t.n, told, l);
  uint4 c[2], q[4];
  memcpy(c, l.compact, 32);
  memcpy(q, l.wide, 64);
  const u32 end = line_end(line * 8, t.n), want = last_below(t, end, w);
  for (int form = 0; form < 2; ++form) {
    u32 at = 99, n = line * 8;
    u64x2 e{0, 0};
    const bool got = form ? pick_wide_line(q, w, told, at, e) : pick_compact_line(c, w, told, at, e);
    (form ? wide_lines : compact_lines) += got;
    if (got) n += at;
    else if (t.t[line * 8].base <= w) find_exact(t.t, line * 8, end, w, n, e);
    else find_exact(t.t, 0, t.n, w, n, e);
    ++runs;
    if (n >= t.n || (got && at > 7)) report("outside", t, w, line);
    else if (valid && w >= t.t[0].base && (n != want || e.x != t.t[n].base || e.y != t.t[n].size)) report("line", t, w, line);
  }
}

// The node that holds entry i's line (step 8) or entry i itself (step 1), told all but `drop` low
// bits of its key 0: the child chosen lies inside the table and is the last whose key is not
// above w, but for bits that the node's shift loses; and the child's key is its own first base
// but for bits that it can keep.
void search_node(const Table& t, u32 i, u64 step, u64 w, u32 drop, bool valid) {
  const u64 k0 = i / (8 * step) * (8 * step);
  const u64 b0 = t.t[k0].base, told = (b0 - t.t[0].base) >> drop << drop;
  PackedNode p;
  pack_node(t.t, k0, step, t.n, t.t[0].base + told, p);
  uint4 q[2];
  memcpy(q, p.w, 32);
  u32 at = 0;
  u64 first = t.t[0].base + told;
  ++runs;
  if (!pick_node(q, w, at, first)) {
    if (p.w[0] != kMarked) report("node refused", t, w, i);
    return;
  }
  ++nodes;
  if (at > 7 || k0 + step * at >= t.n) return report("node outside", t, w, i);
  if (!valid || b0 > w) return;
  const u32 s = p.w[0] & 31;
  u32 want = 0;
  for (u32 h = 1; h < 8 && k0 + step * h < t.n; ++h)
    if ((t.t[k0 + step * h].base - b0) >> s <= (w - b0) >> s) want = h;
  const u64 key = t.t[k0 + step * at].base;
  if (at != want || key - first >= 1ull << s || first != told_of_child(t.t, k0, step, t.n, at)) report("node", t, w, i);
}

void search(const std::vector<fdy_alloc>& v, bool valid) {
  const Table t(v);
  const u64 lo = t.t[0].base;
  // told in full, but for the bits that level 0 would drop, and for one more than can be kept
  const u32 own = key_shift_for(t.t[t.n - 1].base + t.t[t.n - 1].size - lo, 31);
  for (u32 i = 0; i < t.n; ++i)
    for (u64 w : {t.t[i].base - 1, t.t[i].base, t.t[i].base + t.t[i].size / 2, t.t[i].base + t.t[i].size - 1,
                  t.t[i].base + t.t[i].size}) {
      for (u32 drop : {0u, own, 28u}) {
        for (u32 line : {i / 8, (i + 7) / 8, (t.n - 1) / 8})
          if (line * 8 < t.n) search_line(t, line, w, lo + ((t.t[line * 8].base - lo) >> drop << drop), valid);
        for (u64 step : {1ull, 8ull}) search_node(t, i, step, w, drop, valid);
      }
    }
}

// Layouts of one granularity and a range of sizes, with a share of much larger blocks.
std::vector<fdy_alloc> layout(u32 n, int granule, int size_granule, int hi, u32 big_every) {
  std::vector<fdy_alloc> v;
  u64 at = (next() & 0xffff) << granule;
  for (u32 i = 0; i < n; ++i) {
    u64 z = log_uniform(0, hi) >> size_granule << size_granule;
    if (!z) z = 1ull << size_granule;
    if (big_every && below(big_every) == 0) z = log_uniform(hi, hi + 8) >> 21 << 21;
    if (!z) z = 1ull << 21;
    v.push_back(fdy_alloc{at, z});
    const u64 step = (z + (1ull << granule) - 1) >> granule << granule;
    at += step + (below(4) << granule);
  }
  return v;
}

// Level-0 keys of units of 2^sh entries each: from the last unit whose key is not above a word's to the last that
// begins at or below the word.
void settle_units(const std::vector<fdy_alloc>& v, u32 sh, bool valid) {
  const Table t(v);
  const u32 n = (t.n + (1u << sh) - 1) >> sh;
  FlatLevel f{};
  f.span_lo = t.t[0].base;
  f.span_len = t.t[t.n - 1].base + t.t[t.n - 1].size - f.span_lo;
  f.key_shift = key_shift_for(f.span_len, 31);
  u32* keys = (u32*)malloc(n * 4);  // heap blocks of their exact sizes
  u64* units = (u64*)malloc((n + kUnitWindow) * 8);
  memset(units, (int)below(256), (n + kUnitWindow) * 8);
  for (u32 i = 0; i < n; ++i) {
    keys[i] = level0_key(t.t, t.n, sh, i, f.span_lo, f.key_shift);
    units[i] = t.t[(u64)i << sh].base;
  }
  f.keys = (const unsigned char*)keys;
  for (u32 i = 0; i < t.n; i += 1 + (t.n > 300 ? (u32)below(40) : 0))
    for (u64 w : {t.t[i].base - 1, t.t[i].base, t.t[i].base + t.t[i].size / 2, t.t[i].base + t.t[i].size}) {
      const u64 d = w - f.span_lo;
      if (d >= f.span_len) continue;
      u32 u = 0, want = 0;
      for (u32 k = 0; k < n; ++k) {
        if (keys[k] <= (u32)(d >> f.key_shift)) u = k;
        if (units[k] <= w) want = k;
      }
      ++runs;
      const u32 got = settle_unit(f, units, d, u);
      const bool share = units_share(f, d, u);
      if (got > u || (valid && (got != want || (!share && got + 1 < u)))) report("unit", t, w, u);
      if (u == 0 || (valid && units[u] <= w)) continue;
      const u32 rare = settle_unit_rare(f, units, d, u);
      if (rare > u || (valid && rare != want)) report("unit, rare", t, w, u);
    }
  free(keys);
  free(units);
}

// Blocks of up to 2^hi bytes in a few places far apart, so that many share a key.
std::vector<fdy_alloc> clusters(u32 n, int hi) {
  std::vector<fdy_alloc> v;
  u64 at = next() & 0xffff0;
  for (u32 i = 0; i < n; ++i) {
    v.push_back(fdy_alloc{at, log_uniform(3, hi)});
    at += v.back().size + (below(3) ? 0 : 16);
    if (below(n) < 2) at += 1ull << (40 + below(7));
  }
  return v;
}

// The last line of a table, also where its places are the last that 32 bits number.
void line_ends() {
  for (u64 n : std::vector<u64>{1, 7, 8, 9, 16, (1ull << 32) - 17, (1ull << 32) - 9, (1ull << 32) - 8, (1ull << 32) - 7, (1ull << 32) - 1})
    for (u64 lo : std::vector<u64>{0, (n - 1) / 8 * 8}) {
      ++runs;
      if (line_end((u32)lo, (u32)n) != std::min(lo + 8, n) && ++failures <= 10) printf("end of the line at %llu of %llu\n", (unsigned long long)lo, (unsigned long long)n);
    }
}

// Tables of every size that an entry point takes, up to 2^32 - 1 allocations: there are bits for every region, and
// what is packed comes back.
void packed_entries() {
  for (u64 n : std::vector<u64>{1, 2, 3, 16384, 1 << 20, (1ull << 31) - 1, 1ull << 31, (1ull << 31) + 1, (1ull << 32) - 1}) {
    const Entries pk{entry_off_bits(n)};
    bool ok = pk.off_bits <= 55 && n < 1ull << (55 - pk.off_bits) && (pk.off_bits == 55 || n >= 1ull << (54 - pk.off_bits));
    for (u64 region : std::vector<u64>{0, n / 2, n - 1})
      for (u32 word : {0u, 1u, 511u})
        for (u64 off : std::vector<u64>{0, 1, pk.none() - 1, pk.none(), ~0ull}) {
          const u64 e = pk.pack(word, (u32)region, off);
          ok = ok && e != ~0ull && pk.word(e) == word && pk.region(e) == region && pk.off(e) == std::min(off, pk.none());
          ++runs;
        }
    if (!ok && ++failures <= 10) printf("entries of %llu allocations: %u bits\n", (unsigned long long)n, pk.off_bits);
  }
}

}  // namespace

int main() {
  packed_entries();
  line_ends();
  for (int round = 0; round < 400; ++round) {
    const u32 n = 1 + (u32)below(200);
    const int g = (int)below(22), sg = (int)below(g + 1);
    search(layout(n, g, sg, std::max(sg, 1) + (int)below(26), round % 3 ? 0 : 5), true);
    settle_units(clusters(1 + (u32)below(round % 20 ? 300 : 9000), 4 + (int)below(14)), (u32)below(4), true);
    search(layout(n, 21, 9, 26, round % 2 ? 12 : 0), true);  // 2 MiB granules, some gigabytes
    search(layout(n, 4, 0, 26, 0), true);                    // a caching allocator's blocks
    std::vector<fdy_alloc> v(n);                             // nothing that fdy_table_validate passes
    const int bits = 1 + (int)below(64);
    for (auto& e : v) e = fdy_alloc{next() >> (64 - bits), next() >> below(64)};
    search(v, false);
    settle_units(v, (u32)below(4), false);
  }
  {  // distances and sizes at the limits of the forms
    for (int bits : {11, 12, 13, 17, 18, 19, 20, 25, 26, 27, 31, 32, 33})
      for (int delta : {-1, 0, 1})
        for (int s : {0, 9, 21, 31, 33}) {
          if (bits + s > 58) continue;
          const u64 x = ((1ull << bits) + delta) << s;
          std::vector<fdy_alloc> a, b;
          for (u32 i = 0; i < 8; ++i) a.push_back(fdy_alloc{(u64)i << s, 1ull << s});
          a[7].base = x;
          if (a[7].base > a[6].base) search(a, true);
          for (u32 i = 0; i < 8; ++i) b.push_back(fdy_alloc{(u64)i << (bits + s + 1), i == 4 ? x : 1ull << s});
          search(b, true);
          std::vector<fdy_alloc> c;
          for (u32 i = 0; i < 64; ++i) c.push_back(fdy_alloc{(u64)i << s, 1ull << s});
          for (u32 i = 56; i < 64; ++i) c[i].base = x + ((u64)i << s);
          search(c, true);
        }
  }
  printf("%llu run (%llu compact lines, %llu wide, %llu nodes), %d wrong\n", runs, compact_lines, wide_lines, nodes, failures);
  return failures ? 1 : 0;
}
