// scan_states_host.hip - what the ordered scan's states hold (csrc/fdy_flat_state.hpp), compiled for the host: sequences
// of launches of many sizes over one region, in which no field or sum may look written before its chunk has written
// it, whichever kind of state an earlier launch left in its place.
#include <cstdio>
#include <utility>
#include <vector>

#include "fdy_flat_state.hpp"

using namespace fdy;

namespace {

u64 next(u64& s) {
  s ^= s << 13;
  s ^= s >> 7;
  return s ^= s << 17;
}

}  // namespace

int main() {
  u64 r = 0x9e3779b97f4a7c15ull, runs = 0;
  int wrong = 0;
  auto expect = [&](bool ok, const char* what, u32 n, u32 i) {
    ++runs;
    if (!ok && ++wrong <= 10) printf("%s: %u chunks, %u\n", what, n, i);
  };
  for (u32 p = 0; p < 2; ++p)
    for (u64 hits : {0ull, 1ull, 0x7fffull, 0x8000ull, 0x3fffffffull, 0x40000000ull, (1ull << 32) - 1, (1ull << 45) - 1}) {
      const u64 v = make_sum(hits, p);
      expect(is_sum(v, p) && !is_sum(v, p ^ 1) && sum_hits(v) == hits, "sum", p, (u32)hits);
      for (u32 k = 0; k < 4; ++k) expect(!((v >> (16 * k)) & 0x8000), "sum taken for a field", p, k);
    }
  for (u32 most : {1u, 2u, 15u, 16u, 17u, 63u, 64u, 65u, 66u, 80u, 100u, 256u, 1000u, 2300u})
    for (const auto& [spare, workers] : {std::pair{0u, kFlatWorkers}, {512u, kFlatWorkers}, {32768u, kFlatWorkers},
                                         {0u, kFlatWorkersBig}, {512u, kFlatWorkersBig}, {32768u, kFlatWorkersBig}}) {
      const u32 max_sub = most * workers;
      const FlatRegion g = flat_region(max_sub, spare, chunk_state_bytes(max_sub));
      std::vector<u64> mem(g.states, 0);
      u32 turn = 0;
      for (u32 launch = 0; launch < 40; ++launch) {
        u32 n = 1 + (u32)(next(r) % most);
        if (launch % 3 == 0) n = most;
        if (launch % 5 == 4 && most > kFewChunks) n = kFewChunks + 1 - launch % 2;  // both kinds of launches in turn
        const bool few = few_chunks(n);
        const u32 m = scan_states(n);
        const FlatTurn t = flat_turn(turn, m, g.states);
        expect(flat_extent(t.s, m) <= g.states, "extent", n, g.states);
        auto field = [&](u32 c) {
          if (few) return (u32)mem[state_at(t.s, c)] & 0xffffu;
          return (u32)(mem[state_at(t.s, fields_state(c))] >> (16 * (c & 3))) & 0xffffu;
        };
        auto put = [&](u32 c, u32 v) {
          u64& w = mem[state_at(t.s, few ? c : fields_state(c))];
          w = few ? (u64)v : (w & ~(0xffffull << (16 * (c & 3)))) | (u64)v << (16 * (c & 3));
        };
        auto sum = [&](u32 i) -> u64& { return mem[state_at(t.s, sum_state(i))]; };
        std::vector<u32> order(n);
        for (u32 i = 0; i < n; ++i) order[i] = i;
        for (u32 i = n; i > 1; --i) std::swap(order[i - 1], order[next(r) % i]);
        std::vector<char> told(n, 0), summed(n / 16 + 1, 0);
        for (u32 at = 0; at < n; ++at) {
          const u32 c = order[at], probe = (u32)(next(r) % n);
          expect(is_field(field(probe), t.parity) == (told[probe] != 0), "field", n, probe);
          if (!few) expect(is_sum(sum(probe % (n / 16)), t.parity) == (summed[probe % (n / 16)] != 0), "sum", n, probe % (n / 16));
          const u32 hits = (u32)(next(r) % 7681);
          put(c, make_field(hits, t.parity));
          told[c] = 1;
          expect(is_field(field(c), t.parity) && (field(c) & kFieldHits) == hits, "told", n, c);
          if (!few && c % 16 == 15) {
            sum(c / 16) = make_sum((u64)c * 4000000, t.parity);
            summed[c / 16] = 1;
          }
          if (!few && c + 1 == n)
            for (u32 i = c + 1; i % 16; ++i) put(i, 0);
          if (!few && c + 1 == n && c % 16 != 15) sum(c / 16) = 0;
        }
        for (u32 i = 0; i < t.dirty; ++i) {
          const u32 at = flat_to_clear(t, i, m);
          if (at != ~0u) mem[at] = 0;
        }
        turn = flat_next_turn(turn, m);
      }
    }
  printf("%llu run, %d wrong\n", (unsigned long long)runs, wrong);
  return wrong ? 1 : 0;
}
