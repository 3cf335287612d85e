// fdy_flat_state.hpp - chunk states of the ordered scans: how many there are, where they lie and
// what a launch leaves for the next one.  Plain arithmetic, also compiled for the host, where
// tests/level0/level0_host.hip runs sequences of launches over it.
#pragma once
#include "fdy_device.hpp"

namespace fdy {

constexpr u32 kFlatWorkers = 7, kFlatWorkersBig = 15;

// Workers per workgroup.  Many small workgroups start sooner and share the staging's latency, but each chunk costs a
// look-back and a ticket, of which the first are drawn by all workgroups at once, 11.3 ns each.  us, 7 / 15 workers, a
// quarter pointers, scans alone:
//   sub-tiles                       700           830           980           1,250         1,530         1,758
//   4,096 allocations               7.7 / 7.4     7.8 / 7.6     8.4 / 8.0     8.8 / 8.3     9.4 / 8.6     9.7 / 8.9
//   2 % pointers                    7.2 / 7.0     7.4 / 7.2     7.8 / 7.2     8.1 / 7.4     8.6 / 7.8
//   95 %                            10.1 / 10.8   10.3 / 11.1   11.0 / 11.4   11.6 / 12.0   12.4 / 12.5
//   with output                     8.8 / 8.9     8.8 / 9.1     9.3 / 9.4     9.8 / 9.8     10.4 / 10.1
//   4-byte positions                7.6 / 6.9     7.3 / 7.0     8.1 / 7.0     8.1 / 7.4     8.7 / 7.8
//   nothing prepared                11.3 / 11.0   11.6 / 11.3   12.1 / 11.6   12.5 / 11.9   13.0 / 12.2
//   16 allocations, 2 %             6.8 / 7.1     7.0 / 7.3     7.4 / 7.3     7.8 / 7.5     8.1 / 7.7
//   16,384                          8.8 / 8.0     8.8 / 8.0     9.6 / 8.4     10.0 / 8.9    10.4 / 9.5    10.8 / 9.3
// Tables with lines or nodes, whose searches are longer, at 1,368 / 1,758 / 2,344: 20,000 allocations, with output, 11.4 / 12.6,
// 12.4 / 13.0, 19.1 / 13.7; 140,000 12.2 / 12.7, 12.9 / 13.0.
constexpr u32 kFlatFewSubs = 1536, kFlatFewSubsWhole = 976;  // (whole: level 0 holds every base)
__host__ __device__ __forceinline__ u32 flat_workers(u32 n_sub, bool whole = false) {
  return n_sub < (whole ? kFlatFewSubsWhole : kFlatFewSubs) ? kFlatWorkers : kFlatWorkersBig;
}
__host__ __device__ __forceinline__ u32 flat_chunks(u32 n_sub, bool whole = false) {
  const u32 w = flat_workers(n_sub, whole);
  return (n_sub + w - 1) / w;
}

// Most chunks of a launch of up to max_sub sub-tiles, whatever the table.
inline u32 flat_most_chunks(u32 max_sub) {
  u32 most = flat_chunks(max_sub);
  if (max_sub >= kFlatFewSubs && flat_chunks(kFlatFewSubs - 1) > most) most = flat_chunks(kFlatFewSubs - 1);
  return most;
}

// Neighbouring states are spread over 2^s lines of 64 bytes, eight to a line: every
// workgroup in flight reads its predecessors', and states that lie closer are served by too few
// memory channels.  State i lies at state_at(s, i) of blocks of 2^s * 8 states; s is the largest
// for which `states` hold the blocks, at most kFlatSpread, and no larger than the launch's states can use.
// us with 16 allocations and 2 % pointers, in chunk_state_bytes (32, 128 and 128 lines) / 256
// lines / 512 / a line for each: 0.76 M words 10.1 / 8.6 / 8.7 / 8.8, 5.8 M 22.2 / 20.1 / 19.5 /
// 19.5, 16.8 M 46.6 / 41.0 / 40.5 / 41.0 (a state to a chunk, then; with five to sixteen, loads of 0.8 and 5.9 M words with 1 /
// 8 / 32 / 64 / 512 lines: 25.3 / 25.3 / 24.2 / 23.9 / 23.9 and 63.8 / 63.0 / 62.8 / 62.2 / 61.7).
constexpr u32 kFlatSpread = 9;
__host__ __device__ __forceinline__ u32 flat_extent(u32 s, u32 n_states) {
  return (n_states + (8u << s) - 1) >> (s + 3) << (s + 3);
}
__host__ __device__ __forceinline__ u32 flat_spread(u32 n_states, u32 states) {
  u32 s = kFlatSpread;
  while (s > 0 && (flat_extent(s, n_states) > states || (1u << (s - 1)) >= n_states)) --s;
  return s;
}

// Bytes of chunk states that a launch of n_sub sub-tiles is asked for at least: one state for eight
// of them, closer together than the scan likes.
inline size_t chunk_state_bytes(u32 n_sub) { return ((size_t)((n_sub + 7) / 8) * 8 + 255) & ~(size_t)255; }

// Where the states lie, relative to the first chunk state of a buffer made for max_sub sub-tiles with
// `bytes` of chunk states (at least chunk_state_bytes).  The hierarchy's last `spare` bytes, in front
// of the chunk states, are states as well.
struct FlatRegion {
  long long first;  // bytes from the first chunk state
  u32 states;       // at most what the widest spread of a state per chunk uses: no launch has more (see scan_states)
};
inline FlatRegion flat_region(u32 max_sub, u32 spare, size_t bytes) {
  FlatRegion r{-(long long)spare, 0};
  const u32 most = flat_most_chunks(max_sub), want = flat_extent(flat_spread(most, ~0u), most);
  const size_t have = (size_t)((long long)bytes - r.first) / 8;
  r.states = have < want ? (u32)have : want;
  return r;
}

// Bytes of chunk states that let a launch of any size up to max_sub spread its states widest
// (up to 32 KiB more than chunk_state_bytes).
inline size_t flat_state_bytes(u32 max_sub, u32 spare) {
  const size_t least = chunk_state_bytes(max_sub);
  const FlatRegion r = flat_region(max_sub, spare, ~(size_t)0 >> 1);
  const long long best = r.first + 8ll * r.states;
  return best > (long long)least ? ((size_t)best + 255) & ~(size_t)255 : least;
}

__host__ __device__ __forceinline__ u32 state_at(u32 s, u32 i) {
  return (i >> (s + 3) << (s + 3)) | ((i & ((1u << s) - 1)) << 3) | ((i >> s) & 7);
}
__host__ __device__ __forceinline__ u32 chunk_at(u32 s, u32 place) {  // the inverse
  return (place >> (s + 3) << (s + 3)) | ((place >> 3) & ((1u << s) - 1)) | ((place & 7) << s);
}

// The states are left ready for the next launch without a count of the workgroups that are through
// (256 additions to one address at 12 ns each, at the end of the launch where nothing hides
// them): a state carries the parity of its launch, launches alternate, and a state of the other
// parity counts as empty.  A launch writes all of its states; those of the launch
// before that it does not write itself it clears, so that the next but one finds its own parity
// nowhere.  `turn`, kept from launch to launch: states of the launch before << 1 | parity of
// the next.
constexpr u64 kFlatParity = 1ull << 61;
struct FlatTurn {
  u32 s, parity;           // of this launch
  u32 dirty, s_dirty;      // states of the launch before, and how they are spread
};
__host__ __device__ __forceinline__ FlatTurn flat_turn(u32 turn, u32 n_states, u32 states) {
  return FlatTurn{flat_spread(n_states, states), turn & 1, turn >> 1, flat_spread(turn >> 1, states)};
}
__host__ __device__ __forceinline__ u32 flat_next_turn(u32 turn, u32 n_states) { return n_states << 1 | (~turn & 1); }
// Where state i of the launch before lies, if this launch (n_states of its own) has to clear it; else ~0.
__host__ __device__ __forceinline__ u32 flat_to_clear(const FlatTurn& t, u32 i, u32 n_states) {
  const u32 at = state_at(t.s_dirty, i);
  return chunk_at(t.s, at) < n_states ? ~0u : at;
}

// What the states of an ordered scan hold.  With more than 64 chunks, sixteen of them take five: four with a 16-bit field
// for each of four chunks (its hits, once they are known), and one for the hits of all chunks up to the sixteenth, once
// those are.  Either kind says which it is and carries the parity of its launch: fields have their top bit set, a sum has
// none of the four top bits of its 16-bit parts, so that whatever an earlier launch left in a place never looks like the
// other kind.
// Launches of few chunks have a state for each, with the chunk's field in its lowest 16 bits and nothing above.
constexpr u32 kFewChunks = 64;
static_assert(kFewChunks < kFlatFewSubsWhole / kFlatWorkersBig && kFlatFewSubsWhole < kFlatFewSubs,
              "workgroups of many workers never have few chunks");
__host__ __device__ __forceinline__ bool few_chunks(u32 n_chunks) { return n_chunks <= kFewChunks; }
__host__ __device__ __forceinline__ u32 scan_states(u32 n_chunks) {
  return few_chunks(n_chunks) ? n_chunks : 5 * ((n_chunks + 15) / 16);
}
__host__ __device__ __forceinline__ u32 fields_state(u32 chunk) { return 5 * (chunk >> 4) + ((chunk >> 2) & 3); }
__host__ __device__ __forceinline__ u32 sum_state(u32 sixteen) { return 5 * sixteen + 4; }
constexpr u32 kFieldHits = (1u << 14) - 1;
__host__ __device__ __forceinline__ u32 make_field(u32 hits, u32 parity) { return 0x8000u | parity << 14 | hits; }
__host__ __device__ __forceinline__ bool is_field(u32 field, u32 parity) { return field >> 14 == (2u | parity); }
__host__ __device__ __forceinline__ u64 make_sum(u64 hits, u32 parity) {
  return 1ull << 62 | (parity ? kFlatParity : 0) | (hits >> 30 & 0x7fff) << 32 | (hits >> 15 & 0x7fff) << 16 | (hits & 0x7fff);
}
__host__ __device__ __forceinline__ bool is_sum(u64 v, u32 parity) { return v >> 61 == (2u | parity); }
__host__ __device__ __forceinline__ u64 sum_hits(u64 v) {
  return (v >> 32 & 0x7fff) << 30 | (v >> 16 & 0x7fff) << 15 | (v & 0x7fff);
}

}  // namespace fdy
