// Level 0's keys, bucket index, staging and search (csrc/fdy_level0.hpp) over small tables, and
// the chunk states of launches in turn (csrc/fdy_flat_state.hpp), compiled for the host.  Built
// with AddressSanitizer: table, keys, buckets and the staged copy lie in heap blocks of their
// exact sizes, so a read behind any of them is reported.  What the library does not write (the
// rest of a 256-byte piece of the caller's buffer) holds `fill`.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "fdy_flat_state.hpp"
#include "fdy_level0.hpp"

using namespace fdy;

namespace {

struct Params {
  const u32* top;
  const unsigned short* bstart;
  u32 top_n, bucket_log2, n_alloc;
  const fdy_alloc* table;
};

u32 bucket_log2_for(u32 top_n) {  // as plan_table
  u32 b = 0;
  while ((2u << b) <= top_n && b < kMostBucketLog2) ++b;
  return b;
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

struct Built {
  std::vector<unsigned char> top, bst;
  unsigned char* smem;  // 16-byte aligned, exactly flat_level_bytes long
  fdy_alloc* table;
  Params p;
  FlatLevel f;

  Built(const std::vector<fdy_alloc>& t, int fill) {
    const u32 n = (u32)t.size();
    table = (fdy_alloc*)aligned_alloc(16, n * sizeof(fdy_alloc));
    memcpy(table, t.data(), n * sizeof(fdy_alloc));
    p.n_alloc = n;
    p.table = table;
    p.top_n = level0_entries(n);
    p.bucket_log2 = bucket_log2_for(p.top_n);
    top.assign(align256((size_t)p.top_n * 4), (unsigned char)fill);
    bst.assign(align256(((1u << p.bucket_log2) + 1) * 2), (unsigned char)fill);
    p.top = (const u32*)top.data();
    p.bstart = (const unsigned short*)bst.data();
    // what scan_init_kernel writes
    const u64 lo = t[0].base, len = t[n - 1].base + t[n - 1].size - lo;
    const u32 ks = key_shift_for(len, 31);
    for (u32 i = 0; i < p.top_n; ++i) ((u32*)top.data())[i] = level0_key(table, n, 0, i, lo, ks);
    for (u32 i = 0; i <= (1u << p.bucket_log2); ++i)
      ((unsigned short*)bst.data())[i] =
          (unsigned short)sampled_lower_bound(table, 0, n, lo, ks, (u64)i << bucket_shift_for(len, ks, p.bucket_log2));
    const size_t bytes = flat_level_bytes(p.top_n, p.bucket_log2);
    smem = (unsigned char*)aligned_alloc(16, bytes);
    memset(smem, fill, bytes);
    for (u32 tid = 0; tid < 64; ++tid) f = flat_stage<64>(p, smem, tid, false);
  }
  ~Built() {
    free(table);
    free(smem);
  }
};

int failures = 0;
unsigned long long runs = 0;

// Searches `words` four lanes' worth at a time (the step count is shared, as in a wave); `exact`:
// compares with the definition, else only asks that a region is one of the table's.
void check(const std::vector<fdy_alloc>& t, const std::vector<u64>& words, int fill, bool exact) {
  Built b(t, fill);
  std::vector<u64> cand;
  for (u64 w : words)
    if (w - b.f.span_lo < b.f.span_len) cand.push_back(w);
  for (size_t i = 0; i < cand.size(); i += 4) {
    u64 d[4], off[4];
    u32 n[4];
    bool hit[4];
    for (int c = 0; c < 4; ++c) d[c] = (i + c < cand.size() ? cand[i + c] : b.f.span_lo) - b.f.span_lo;
    flat_search<4>(b.p, b.f, d, n, off, hit, [](bool x) { return x; });
    runs += 4;
    for (int c = 0; c < 4; ++c) {
      const u64 w = d[c] + b.f.span_lo;
      bool ok = n[c] < t.size();
      if (exact) {
        u32 r = 0xffffffffu;
        for (u32 k = 0; k < t.size(); ++k)
          if (t[k].base <= w && w - t[k].base < t[k].size) r = k;
        ok = ok && hit[c] == (r != 0xffffffffu) && (!hit[c] || (n[c] == r && off[c] == w - t[r].base));
      }
      if (!ok && ++failures <= 10) {
        printf("word %llx in {", (unsigned long long)w);
        for (auto& e : t) printf(" %llx+%llx", (unsigned long long)e.base, (unsigned long long)e.size);
        printf(" }, fill %02x: hit %d region %u offset %llx\n", fill, hit[c], n[c], (unsigned long long)off[c]);
      }
    }
  }
}

const int kFills[] = {0x00, 0x10, 0xA7, 0xFF};

std::vector<u64> edges(const std::vector<fdy_alloc>& t) {
  std::vector<u64> w;
  for (auto& e : t)
    for (u64 x : {e.base - 1, e.base, e.base + 1, e.base + e.size / 2, e.base + e.size - 1, e.base + e.size,
                  e.base + e.size + 1})
      w.push_back(x);
  return w;
}

// Every table of 1 to 5 blocks with sizes and gaps of these, from three places.
void valid_tables(u32 n, std::vector<fdy_alloc>& t, u64 at) {
  static const u64 sizes[] = {1, 16, 4096, 1ull << 30}, gaps[] = {0, 1, 1ull << 21, 1ull << 33};
  if (t.size() == n) {
    const auto w = edges(t);
    for (int fill : kFills) check(t, w, fill, true);
    return;
  }
  for (u64 s : sizes)
    for (u64 g : gaps) {
      if (n > 3 && (s == 16 || g == 1)) continue;  // fewer of the larger tables
      t.push_back(fdy_alloc{at + g, s});
      valid_tables(n, t, at + g + s);
      t.pop_back();
    }
}

u64 next(u64& s) {  // xorshift64
  s ^= s << 13;
  s ^= s >> 7;
  return s ^= s << 17;
}

// The two ways to stage a table, and by how many threads, leave the same bytes: sizes around whole batches of pieces,
// up to the largest level 0.
template <u32 kThreads>
void stage_again(const Built& b, int fill, bool at_once) {
  const size_t bytes = flat_level_bytes(b.p.top_n, b.p.bucket_log2);
  unsigned char* again = (unsigned char*)aligned_alloc(16, bytes);
  memset(again, fill, bytes);
  for (u32 tid = 0; tid < kThreads; ++tid) flat_stage<kThreads>(b.p, again, tid, at_once);
  ++runs;
  if (memcmp(again, b.smem, bytes) && ++failures <= 10)
    printf("%u allocations, %u threads%s: staged differently\n", b.p.n_alloc, kThreads, at_once ? " at once" : "");
  free(again);
}
void staging() {
  for (u32 n : {1u, 4u, 5u, 64u, 255u, 256u, 257u, 1000u, 1024u, 2048u, 4096u, 8192u, 1u << kMostTopLog2}) {
    std::vector<fdy_alloc> t(n);
    for (u32 i = 0; i < n; ++i) t[i] = fdy_alloc{0x7f0000000000ull + ((u64)i << 21), 4096};
    for (int fill : kFills) {
      Built b(t, fill);
      for (bool at_once : {false, true}) {
        stage_again<64>(b, fill, at_once);
        stage_again<512>(b, fill, at_once);
        stage_again<1024>(b, fill, at_once);
      }
    }
  }
}

// Tables that fdy_table_validate refuses: any order, overlaps, spans that wrap.  What is found is
// unspecified, but nothing outside the table may be read and every search ends.
void invalid_tables() {
  u64 s = 0x9e3779b97f4a7c15ull;
  {  // ends below its first base: small integers lie in the span
    std::vector<fdy_alloc> t{{0x7f0000000000ull, 16}, {4096, 16}};
    check(t, {0, 1, 4095, 4096, 0x7f0000000000ull, ~0ull}, 0, false);
  }
  for (int round = 0; round < 60000; ++round) {
    std::vector<fdy_alloc> t(1 + next(s) % (round % 50 ? 6 : 300));
    const int bits = 1 + (int)(next(s) % 64);
    for (auto& e : t) e = fdy_alloc{next(s) >> (64 - bits), next(s) >> (next(s) % 64)};
    if (next(s) % 2) std::swap(t.front(), *std::max_element(t.begin(), t.end(), [](auto& a, auto& b) { return a.base < b.base; }));
    auto w = edges(t);
    if (w.size() > 64) w.resize(64);
    for (int i = 0; i < 16; ++i) w.push_back(next(s) >> (next(s) % 64));
    check(t, w, kFills[round % 4], false);
  }
}

// Sequences of launches over the chunk states of one prepared table: every state lies inside its
// region and is nobody else's, none looks written before its chunk writes it, and what the
// launch clears it does not write.
void chunk_states() {
  u64 r = 0x2545f4914f6cdd1dull;
  auto expect = [](bool ok, const char* what, u32 max_sub, u32 n_sub, u32 i) {
    if (!ok && ++failures <= 10) printf("%s: max_sub %u n_sub %u chunk %u\n", what, max_sub, n_sub, i);
  };
  std::vector<u32> maxima{1, 2, 7, 8, 9, 255, 257, 1343, 1344, 1535, 1536, 1537, 1759, 1761, 2111, 2113, 20000,
                          32767, 32768, 32769, 44685, 300001};
  for (int i = 0; i < 60; ++i) maxima.push_back(1 + (u32)(next(r) % (1u << (1 + next(r) % 17))));
  for (u32 max_sub : maxima)
    for (u32 spare : {512u, 6144u, 49408u})
      for (const bool tight : {false, true}) {
        const size_t least = chunk_state_bytes(max_sub), best = flat_state_bytes(max_sub, spare);
        expect(best >= least && best <= least + 32768, "size", max_sub, 0, 0);
        const size_t bytes = tight ? least : best;
        const FlatRegion g = flat_region(max_sub, spare, bytes);
        expect(g.first >= -(long long)spare && g.first + 8ll * g.states <= (long long)bytes, "region", max_sub, 0, 0);
        std::vector<u64> mem(g.states, 0);
        std::vector<u32> mark(g.states, ~0u);
        u32 turn = 0;
        for (u32 launch = 0; launch < 12; ++launch) {
          u32 n_sub = 1 + (u32)(next(r) % max_sub);
          if (launch % 4 == 1) n_sub = max_sub;
          if (launch % 4 == 3) n_sub = n_sub < 40 ? n_sub : 1 + (u32)(next(r) % 40);
          const u32 n = flat_chunks(n_sub);
          const FlatTurn t = flat_turn(turn, n, g.states);
          const u64 par = t.parity ? kFlatParity : 0;
          expect(flat_extent(t.s, n) <= g.states, "extent", max_sub, n_sub, 0);
          if (bytes == best) expect(t.s == flat_spread(n, ~0u), "spread", max_sub, n_sub, 0);
          for (u32 i = 0; i < n; ++i) {
            const u32 at = state_at(t.s, i);
            if (at >= g.states || mark[at] == launch || chunk_at(t.s, at) != i) {
              expect(false, "place", max_sub, n_sub, i);
              continue;
            }
            mark[at] = launch;
            const u64 flag = (mem[at] ^ par) >> 61;
            expect(flag == 0 || (flag & 1), "looks written", max_sub, n_sub, i);
          }
          for (u32 i = 0; i < t.dirty; ++i) {
            const u32 at = flat_to_clear(t, i, n);
            if (at == ~0u) continue;
            expect(at < g.states && mark[at] != launch, "clears its own", max_sub, n_sub, i);
            if (at < g.states) mem[at] = 0;
          }
          for (u32 i = 0; i < n; ++i) mem[state_at(t.s, i)] = ((2ull << 62) | i) ^ par;
          for (u32 i = 0; i < g.states; ++i)  // the next but one starts from this launch's parity
            expect(mem[i] == 0 || ((mem[i] ^ par) >> 61) == 4, "left behind", max_sub, n_sub, i);
          turn = flat_next_turn(turn, n);
          ++runs;
        }
      }
}

}  // namespace

int main(int argc, char** argv) {
  if (argc < 2) return 2;
  if (!strcmp(argv[1], "valid")) {
    for (u32 n = 1; n <= 5; ++n)
      for (u64 at : {0ull, 0x7f0000000000ull, ~0ull - (1ull << 37)}) {
        if (n > 3 && at != 0x7f0000000000ull) continue;
        std::vector<fdy_alloc> t;
        valid_tables(n, t, at);
      }
  } else if (!strcmp(argv[1], "invalid")) {
    invalid_tables();
  } else if (!strcmp(argv[1], "staging")) {
    staging();
  } else if (!strcmp(argv[1], "states")) {
    chunk_states();
  } else {
    return 2;
  }
  printf("%llu run, %d wrong\n", runs, failures);
  return failures ? 1 : 0;
}
