// fdy_scan.hip - (a1) pointer scan and (a2) relocation segmentation for gfx950.
//
// The scan classifies every 8-byte word of the captured argument blobs against the sorted
// allocation table (the relaxation of Section 4.1.1's identical-layout requirement: find
// every embedded pointer kernel-agnostically, because argument buffers are opaque -
// Section 2.2, Appendix B).  It is one streaming pass over the words.
//
// Work decomposition.  Persistent workgroups, one per compute unit, stage the top level of the
// table's hierarchy in LDS once.  Words come in sub-tiles of 512; a chunk is a sub-tile for each
// of the workgroup's 15 (small inputs: 7) workers, handed out by an atomic ticket.  A worker
//   1. takes its 8 words per lane (16-byte coalesced non-temporal loads) and rejects every word
//      outside the table's span;
//   2. queues the surviving candidates and their places in LDS, in word order (ballot ranks), so
//      that the interval search runs on dense rounds of 64 lanes; with a rebased output, where the
//      sub-tile goes out again, LDS holds a copy of it (the stash) in place of the candidates;
//   3. searches the hierarchy: level 0 in LDS (truncated keys of sampled bases behind a bucket
//      index, fdy_level0.hpp), nodes in global memory for the largest tables only, then one line of
//      eight entries (fdy_lines.hpp), or the table entry itself where level 0 has every base;
//      where truncated keys lead a word too far, exact bases of what the keys stand for settle it;
//      what became of a candidate stays in registers, 64 bits each;
//   4. posts its hits, the last of fifteen workers those of the chunk to everybody (of seven: the clerk does, behind the
//      barrier); one barrier per chunk makes them and the next ticket visible.
// The sixteenth wave, the clerk, owns no words: it draws the tickets and finds the chunk's output
// position by a decoupled look-back over what the chunks say of themselves (16 bits each, four to a word, and the hits so
// far behind every sixteenth: one step looks at 256 chunks, which is what is in flight) while the others search the next
// chunk.  The workers then write the entries of the chunk before from registers, in ascending word order.  The input is
// read once and the relocation table written once.
//
// What bounds it.  A compute unit's vector L1 takes one divergent lane per clock and its
// searches' chains of dependent requests cost 0.6-0.8 us a step; beside them stand the words
// from memory, 300 to 700 vector instructions per sub-tile, and, once a table outgrows the 4 MiB
// L2 of an XCD, the lines that candidates pull through the fabric.  None of these alone is at
// its limit: what counts is how much of them overlaps, so the kernel is built for sixteen waves
// per compute unit.  Hence 128 registers: candidates (or the stash) in LDS in place of the words,
// 64 bits per result, wide lines one chain at a time, and no window, staging area or second search for
// dense stretches (eight rounds hold a whole sub-tile).  They are just enough: with nodes and an output
// four values are spilled (20 bytes of scratch a lane), and fifteen-worker instances keep 2 to 6 scalars in lanes of vector
// registers, for tables with lines 20 to 28, with nodes 44 to 62.  Measured on the way (us; 2^27 words, 2^20 allocations, with
// output / 12.3 M words, 65,537 byte-granular allocations, with output / 33.5 M words, 300,007
// allocations with 8 GiB regions, without):
//   eight waves of 256 registers, two sub-tiles in hand, tables read through up to two nodes   758 / 95 / 227
//   eleven workers, level 0 samples the lines themselves up to 8 * 2^14 allocations, and
//   the line before instead of a search where truncated keys lead a line too far                787 / 75 / 172
//   fifteen workers                                                                            715 / 66 / 161
//   the largest tables' rounds one by one but for sub-tiles with few candidates                685 / 67 / 158
//   positions by one step over 256 chunks, not by 64 at a time; hits told by the last worker    670 / 65 / 152
// A small launch is a chain of waits.  us of scans alone, one after the other, a quarter pointers, 4,096 allocations, 0.3 /
// 0.8 / 1.7 / 5.9 M words: 7.2 / 8.9 / 11.0 / 23.0 with positions by 64 chunks at a time; 7.1 / 8.6 / 10.5 / 21.8 so;
// 8.4 M positions at 4-byte stride 24.7 / 23.1.
// Tried and left: words requested before the search (they hold up its first fetch, which returns
// behind them: 75 -> 90; behind the last fetch of the search, with the ticket there, a load of 5.9 M words 62.4 -> 66.1: a
// compute unit's vector L1 answers in order, so that what comes from memory holds up every other wave's fetches as well),
// the last chunk's position looked for while it is searched (62 -> 65, for the same reason), chunks in a fixed order
// instead of tickets (62.3 -> 64.4), seven workers and two workgroups per compute unit at every size (62 -> 68), tickets, counts and positions through a ring in LDS instead of the
// barrier (workers a chunk apart: 172 -> 215), two sub-tiles per worker and round with up to six
// chains (seven workers: 787 -> 784, 75 -> 80), choosing among a node's keys as a tree of three
// compares (everything a quarter slower).
//
// Variant at 4-byte stride (fdy_scan_pointers_stride4; kHalf): reads the array as 32-bit units and
// treats every unit index as a position whose value is that unit and the next one; only the
// loader and the numbering of positions differ.
//
// Variant with a rebased output (fdy_scan_pointers_rebase; kOut): the same ordered scan also
// writes every word, hits rebased, to a second array, so that an archive whose graphs are
// their own templates needs no second pass over the words (Section 4.2.2: every rank takes the
// same captured blobs and differs only in its layout).  A hit's word in the stash becomes
// new_base[region] + offset, and the stash goes out with the 16-byte stores a copy would use
// (scattered 8-byte fix-ups into lines that have left L2 cost a third more time).  For large inputs
// and tables a launch ahead of the scan lays the base map beside the lines (scan_records_kernel).
//
// The table's part of all this depends on the table alone and can be built once per archive
// (fdy_scan_table_prepare); the per-call state (ticket, chunk states, counters) then lives in the
// same buffer and is left ready for the next call, marked with the launch's parity (FlatTurn), so
// that a scan is one launch.
//
// Tickets are handed out in increasing order and a wave only ever waits for chunks with
// smaller numbers, which are already owned by resident workgroups: a launch never waits for a compute unit that another
// kernel holds.  The wait is bounded by a spin limit after which FDY_ST_SPIN is raised and the kernel still terminates.
//
// Steps whose bodies hold a whole search are not written as loops: past a size the optimizer
// declines to unroll even a `#pragma unroll` loop, and a rolled loop indexes the
// register-resident results dynamically, which sends them to scratch memory.
#include <type_traits>

#include "fdy_device.hpp"
#include "fdy_flat_state.hpp"
#include "fdy_internal.h"
#include "fdy_level0.hpp"
#include "fdy_lines.hpp"

namespace fdy {
namespace {

constexpr u64 kMaxWords = (1ull << 32) - 256;  // word and reloc indices are 32-bit
constexpr int kLoads = 4;                      // 16-byte loads per lane per sub-tile
constexpr int kWpl = 2 * kLoads;               // words per lane per sub-tile
constexpr int kSub = 64 * kWpl;                // words per sub-tile (512)
constexpr int kRounds = 8;                     // rounds of 64 candidates: a sub-tile's words
constexpr int kMaxNodeLevels = 6;
constexpr u32 kRebaseWaves = 8;
constexpr u32 kWorkerLds = kSub * 10;          // a worker's stash and the places of its candidates
struct ScanParams {
  const u64* words;
  u64 n_words;
  const fdy_alloc* table;
  u32 n_alloc;
  fdy_reloc* relocs;
  u64 capacity;
  u64* d_count;
  u32* ticket;
  const u32* top;  // [top_n] level-0 keys, padded with 0xffffffff
  const unsigned short* bstart;  // [n_buckets + 1] level-0 keys below each bucket's first key value
  u32 bucket_log2;  // log2(n_buckets)
  u32 top_n;        // level-0 keys, rounded up to whole 16-byte pieces
  u32 levels;       // 8-ary levels below level 0, the table line included
  u32 f0_log2;      // level 0 samples every (2^f0_log2 * 8^levels)-th base
  const u64* units;         // levels >= 1: the first base of what each level-0 key stands for
  const u64* runs;          // f0_log2 > 0: every 8^levels-th base, padded with ~0
  const uint4* nodes[kMaxNodeLevels];  // nodes[j-1]: level j's, of every 8^j-th base (levels >= 2)
  const uint4* leaf;        // the table's lines in their wide form (levels >= 1)
  const uint4* cleaf;       // ... and in their compact one
  const uint4* records;     // with a base map, large tables: see scan_records_kernel (null: not built)
  u32 n_lines;
  u64* acc;     // fused scan + rebase: hits so far
  u64* cstate;  // chunk states
  u32 n_chunks;
  const u64* prepared;  // the caller's prepared table (its header is checked on the device), or null
  u32 top_log2;         // the tuning that the hierarchy's layout depends on
  u32 off_bits;         // see Entries (fdy_lines.hpp)
  u32 n_sub;            // sub-tiles
  u32* d_status;
  u32 spin_limit;
  const u64* new_base;  // with a rebased output only: [n_alloc]
  u64* out;             // with a rebased output only: [n_words]
  u32* turn;            // what the launch before left (see FlatTurn)
  FlatRegion region;    // where its states lie (a prepared table's header says so itself)
};

__device__ __forceinline__ u64 ld_state(const u64* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_state(u64* p, u64 v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// LDS traffic between lanes of one wave needs no hardware barrier (a wave's LDS operations
// execute in order); this only stops the compiler from moving accesses across the point.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// What chunks say of themselves (fdy_flat_state.hpp): a 16-bit field each, its hits, four to a state, and behind every
// sixteenth the hits of all chunks so far, all written and read by agent-scope relaxed atomics (no fences: flag and
// payload travel in one word).  A chunk's exclusive prefix is then one step back over 256 chunks: as many as a launch
// has in flight, so that it rarely takes a second.  Waits are for chunks that are already being processed, and they are
// bounded by the spin limit.
__device__ __forceinline__ bool spin_once(u32& spins, u32 spin_limit, u32* d_status) {
  if (++spins > spin_limit) {  // give up, flag it, let everybody proceed
    if (lane_id() == 0) raise_status(d_status, FDY_ST_SPIN);
    return false;
  }
  __builtin_amdgcn_s_sleep(1);
  return true;
}

__device__ __forceinline__ void st_field(unsigned short* p, u32 field) {
  __hip_atomic_store(p, (unsigned short)field, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The states of a launch of the flat scan.
struct FlatStates {
  u64* at;  // the region's first state
  u32 s;    // spread (see state_at)
  u32 parity;
  __device__ __forceinline__ u64* place(u32 i) const { return &at[state_at(s, i)]; }
  __device__ __forceinline__ unsigned short* field_of(u32 chunk) const {
    return reinterpret_cast<unsigned short*>(place(fields_state(chunk))) + (chunk & 3);
  }
  __device__ __forceinline__ void store_field(u32 chunk, u32 field) const { st_field(field_of(chunk), field); }
};

// The number of hits in all chunks before `chunk`.  Lane l looks at the four fields of one state, the first sixteen also at
// the sums behind the sixteenths before; polls go to what is missing alone.  (64 chunks at a time, four or five round trips
// in a row: 23.0 us for 5.9 M words, 21.8 so.  The ticket drawn behind the first requests 22.5, behind the whole step 22.6.
// Neighbouring states in the same memory lines: a load of 5.9 M words 62 -> 64.)  meanwhile(): called behind the first requests.
template <typename Meanwhile>
__device__ __forceinline__ u64 exclusive_prefix(const FlatStates& states, u32 chunk, u32 spin_limit, u32* d_status,
                                                Meanwhile meanwhile) {
  const u32 l = lane_id();
  u64 excl = 0;
  u32 spins = 0;
  // `end` chunks are left: their hits are wanted
  if (chunk == 0) meanwhile();
  for (u32 end = chunk; end > 0;) {
    const u32 q = (end - 1) >> 2, g = end >> 4;  // the last state with fields that count; whole sixteenths
    u64 v = 0, sum = 0;
    if (l < g && l < 16) sum = ld_state(states.place(sum_state(g - 1 - l)));
    if (l <= q) v = ld_state(states.place(fields_state(4 * (q - l))));
    __builtin_amdgcn_sched_barrier(0);
    if (end == chunk) meanwhile();
    const u64 known = ballot(is_sum(sum, states.parity));
    // chunks [from, end) are added up here, what lies before is known, or left for the next step
    const u32 back = known ? (u32)__ffsll((long long)known) - 1 : 0u;
    const u32 from = known ? (g - back) << 4 : q >= 64 ? 4 * (q - 63) : 0u;
    u32 hits = 0;  // the lane's
    for (;;) {
      bool missing = false;
      hits = 0;
#pragma unroll
      for (u32 k = 0; k < 4; ++k) {
        const u32 c = 4 * (q - l) + k, field = (u32)(v >> (16 * k)) & 0xffffu;
        const bool counts = l <= q && c >= from && c < end;
        if (counts && !is_field(field, states.parity)) missing = true;
        hits += counts ? field & kFieldHits : 0u;
      }
      if (ballot(missing) == 0) break;
      if (!spin_once(spins, spin_limit, d_status)) return excl;
      if (missing) v = ld_state(states.place(fields_state(4 * (q - l))));  // (the others' are there)
    }
    excl += (u32)__builtin_amdgcn_readlane((int)wave_incl_scan(hits), 63);
    if (known) {
      const u64 s = sum_hits(sum);
      excl += (u64)(u32)__shfl((u32)s, (int)back) | (u64)(u32)__shfl((u32)(s >> 32), (int)back) << 32;
      break;
    }
    end = from;
  }
  return excl;
}

// The same in launches of few chunks, each with a state of its own: 64 states at most, and nobody else's hits in the word
// or the memory line that a chunk writes.  (us of scans alone, sixteen chunks to five states / so: 46,000 words and 5,658
// allocations 7.0 / 6.3, 60,000 and 200,000 9.6 / 9.3, 20,000 and 2^20 10.5 / 10.2, 100,000 with nothing prepared 10.8 /
// 10.6.  Fields of 32 bits, two to a state, 6.8 for the first and 0.2 more for launches of many chunks.)
template <typename Meanwhile>
__device__ __forceinline__ u64 prefix_of_few(const FlatStates& states, u32 chunk, u32 spin_limit, u32* d_status,
                                             Meanwhile meanwhile) {
  const u32 l = lane_id();
  u64 v = 0;
  if (l < chunk) v = ld_state(states.place(l));
  __builtin_amdgcn_sched_barrier(0);
  meanwhile();
  for (u32 spins = 0;;) {
    const bool missing = l < chunk && !is_field((u32)v & 0xffffu, states.parity);
    if (ballot(missing) == 0) break;
    if (!spin_once(spins, spin_limit, d_status)) return 0;
    if (missing) v = ld_state(states.place(l));
  }
  return (u32)__builtin_amdgcn_readlane((int)wave_incl_scan(l < chunk ? (u32)v & kFieldHits : 0u), 63);
}

// A prepared table: magic, what it was made for and where the chunk states lie (six 64-bit
// words), then the counters, the hierarchy and the chunk states.
struct PreparedHeader {
  u64 magic;
  u32 n_alloc, top_log2;
  u64 max_words;
  u64 table_ptr;
  FlatRegion region;
};
constexpr u64 kPreparedMagic = 0x3159445f4c424154ull;  // "TABL_DY1"
constexpr size_t kPreparedHeader = 256;
constexpr size_t kPreparedTurn = 128;  // byte offset of the turn.  The first 512 bytes also hold the scan's ticket (384) and
                                       // the counters of fdy_segment_fingerprint (64, 192, 196, 320, 448)

// Is the caller's prepared table one that was made for this table, this tuning and at least
// this many words?  (The host cannot look into device memory without a round trip.)
__device__ __forceinline__ bool prepared_ok(const u64* prepared, u32 n_alloc, u32 top_log2, u64 n_words,
                                            const fdy_alloc* for_table) {
  if (!prepared) return true;
  const u64 magic = prepared[0], sizes = prepared[1], max_words = prepared[2], table = prepared[3];
  return magic == kPreparedMagic && (u32)sizes == n_alloc && (u32)(sizes >> 32) == top_log2 &&
         n_words <= max_words && table == (u64)(uintptr_t)for_table;
}
__device__ __forceinline__ bool prepared_ok(const ScanParams& p) {
  return prepared_ok(p.prepared, p.n_alloc, p.top_log2, p.n_words, p.table);
}

// kHalf: the array is read as 32-bit units and position q stands for the 64-bit value whose low
// half is unit q and whose high half is unit q + 1 (pointers at 4-byte alignment inside packed
// structures); p.n_words is then the number of positions, one less than the number of units.
// A lane still takes 16-byte pieces, four positions each, and gets the unit that follows its
// piece from the next lane (the last lane from the next piece, or from behind the sub-tile).
//
// The words are requested in one place and taken in another; the ragged tail, and sub-tiles past the end, are read
// where they are taken (no word there is a candidate).
template <bool kHalf>
struct Words {
  v4u32 v[kHalf ? 2 : kLoads];
  u32 behind;
};
template <bool kHalf>
__device__ __forceinline__ bool whole_sub(const ScanParams& p, u32 sub) {  // (kHalf: units wbase .. wbase + 512 exist)
  return (u64)sub * kSub + kSub <= p.n_words;
}
template <bool kHalf>
__device__ __forceinline__ Words<kHalf> request_words(const ScanParams& p, u32 sub) {
  Words<kHalf> r = {};  // (nothing of the words before stays)
  if (!whole_sub<kHalf>(p, sub)) return r;
  const u32 lane = lane_id();
  const u64 wbase = (u64)sub * kSub;
  // streamed once: non-temporal, so that the table levels keep their place in L2
  if constexpr (kHalf) {
    static_assert(kWpl == 8, "two 16-byte pieces of four positions per lane");
    const u32* h = reinterpret_cast<const u32*>(p.words);
#pragma unroll
    for (int k = 0; k < 2; ++k)
      r.v[k] = __builtin_nontemporal_load(reinterpret_cast<const v4u32*>(h + wbase + (k * 64 + lane) * 4));
    r.behind = h[wbase + kSub];
  } else {
#pragma unroll
    for (int k = 0; k < kLoads; ++k)
      r.v[k] = __builtin_nontemporal_load(reinterpret_cast<const v4u32*>(p.words + wbase + (k * 64 + lane) * 2));
  }
  return r;
}
template <bool kHalf>
__device__ __forceinline__ void take_words(const ScanParams& p, u32 sub, u64 span_lo, const Words<kHalf>& r,
                                           u64 (&w)[kWpl]) {
  const u32 lane = lane_id();
  const u64 wbase = (u64)sub * kSub;
  if constexpr (kHalf) {
    const u32* h = reinterpret_cast<const u32*>(p.words);
    if (whole_sub<kHalf>(p, sub)) {
      u32 nx[2];
      nx[0] = __shfl_down(r.v[0].x, 1);
      nx[1] = __shfl_down(r.v[1].x, 1);
      const u32 first1 = __shfl(r.v[1].x, 0);
      if (lane == 63) {
        nx[0] = first1;
        nx[1] = r.behind;
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        w[4 * k + 0] = pair64(r.v[k].x, r.v[k].y);
        w[4 * k + 1] = pair64(r.v[k].y, r.v[k].z);
        w[4 * k + 2] = pair64(r.v[k].z, r.v[k].w);
        w[4 * k + 3] = pair64(r.v[k].w, nx[k]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < kWpl; ++i) {
        const u64 q = wbase + ((i >> 2) * 64 + lane) * 4 + (i & 3);
        w[i] = q < p.n_words ? pair64(h[q], h[q + 1]) : span_lo - 1;  // outside the span
      }
    }
  } else if (whole_sub<kHalf>(p, sub)) {
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      w[2 * k] = pair64(r.v[k].x, r.v[k].y);
      w[2 * k + 1] = pair64(r.v[k].z, r.v[k].w);
    }
  } else {
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      const u64 idx = wbase + (k * 64 + lane) * 2;
      w[2 * k] = idx < p.n_words ? p.words[idx] : span_lo - 1;  // outside the span
      w[2 * k + 1] = idx + 1 < p.n_words ? p.words[idx + 1] : span_lo - 1;
    }
  }
}
template <bool kHalf>
__device__ __forceinline__ void load_words(const ScanParams& p, u32 sub, u64 span_lo, u64 (&w)[kWpl]) {
  take_words<kHalf>(p, sub, span_lo, request_words<kHalf>(p, sub), w);
}

// Register r of a lane holds position (r / kPer * 64 + lane) * kPer + r % kPer of the sub-tile,
// kPer = 2 words per 16-byte piece, or 4 positions per piece when reading 32-bit units.
template <bool kHalf>
__device__ __forceinline__ u32 pos_in_sub(int r, u32 lane) {
  constexpr int kPer = kHalf ? 4 : 2;
  return ((u32)(r / kPer) * 64 + lane) * kPer + (u32)(r % kPer);
}

// A wave's copy of a sub-tile in LDS, to the output: the 16-byte stores a copy would use, non-temporal.
__device__ __forceinline__ void unstash_words(const ScanParams& p, u32 sub, const u64* stash) {
  typedef u64 v2u64 __attribute__((ext_vector_type(2)));
  const u32 lane = lane_id();
  const u64 wbase = (u64)sub * kSub;
  if (wbase + kSub <= p.n_words) {
    u64x2 v[kLoads];
#pragma unroll
    for (int k = 0; k < kLoads; ++k) v[k] = *reinterpret_cast<const u64x2*>(stash + (k * 64 + lane) * 2);
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      v2u64 o;
      o.x = v[k].x;
      o.y = v[k].y;
      __builtin_nontemporal_store(o, reinterpret_cast<v2u64*>(p.out + wbase + (k * 64 + lane) * 2));
    }
  } else {
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      const u32 i = (k * 64 + lane) * 2;
      if (wbase + i < p.n_words) p.out[wbase + i] = stash[i];
      if (wbase + i + 1 < p.n_words) p.out[wbase + i + 1] = stash[i + 1];
    }
  }
}

__device__ __forceinline__ void store_reloc(const ScanParams& p, u64 at, u32 word, u32 region, u64 offset) {
  if (at < p.capacity) {
    fdy_reloc o;
    o.word = word;
    o.region = region;
    o.offset = offset;
    *reinterpret_cast<uint4*>(&p.relocs[at]) = *reinterpret_cast<const uint4*>(&o);
  }
}

// kDepth: 0 - every base has its key in level 0; 1 - level 0 samples the lines; 2 - nodes lie between.
// What a launch's hierarchy is read through (one per wave; kDepth 0 has no use for it).
struct Forms {
  bool lines;            // compact lines
  bool settle;           // kDepth 1: lines share keys, so that a line is settled before it is fetched
  u32 marked, searched;  // marked lines met by this wave's candidates; its candidates
  u64 nb_from;           // records: a code stands for nb_from + (code << nb_shift)
  u32 nb_shift;
};
// Whether the compact lines are worth reading for this table: where most are marked a candidate
// would pay the compact fetch and then the wide one, so the choice is made per table, from 64
// evenly spaced lines (all lanes of the wave take part).
__device__ __forceinline__ bool mostly_packed(const uint4* lines, u32 n) {
  const u64 i = ((u64)lane_id() * n) >> 6;
  return __popcll(ballot(lines[i * 2].x == kMarked)) <= 16;
}
// Whether lines share level-0 keys, in any of 64 evenly spaced pairs of neighbours.  (100,000 blocks of 512 B to 8 KiB,
// 5 % of the pairs share a key, settled before / after a line was fetched in vain: 70 / 78 us.)
__device__ __forceinline__ bool units_share_keys(const FlatLevel& f, u32 n) {
  const u32 i = (u32)(((u64)lane_id() * n) >> 6);
  const u32* keys = reinterpret_cast<const u32*>(f.keys);
  return ballot(keys[i] == keys[i + 1]) != 0;
}
template <int kDepth>
__device__ __forceinline__ Forms pick_forms(const ScanParams& p) {
  Forms m{false, false, 0, 0, 0, 0};
  if constexpr (kDepth >= 1) m.lines = mostly_packed(p.cleaf, p.n_lines);
  if constexpr (kDepth >= 2) {
    if (p.records) {
      const u64* t = reinterpret_cast<const u64*>(p.records + (u64)p.n_lines * 4);
      m.nb_from = t[0];
      m.nb_shift = (u32)t[1];
    }
  }
  return m;
}
// Candidates need not spread over the table as its lines do (most pointers of a serving
// process point into a few huge regions): a wave that meets marked lines more than a
// quarter of the time goes back to the wide form for good.  Either form gives the same answer.
__device__ __forceinline__ void count_marked(Forms& m, u32 candidates) {
  m.searched += candidates;
  if (m.marked * 4 > m.searched + 256) m.lines = false;
}

// Interval search of N distances per lane in a hierarchy below level 0.  A whole node or line is
// fetched at once, with independent loads (requests to one line merge; dependent probes into
// it cost a round trip each, the vector L1 being far too small to keep it between two probes),
// and every chain's before the first is looked at: left to itself the scheduler sinks each
// chain's loads next to their use and the round trips line up.  Wide lines (16 registers) come
// one chain at a time.
template <int kDepth, int N>
__device__ __forceinline__ void deep_search(const ScanParams& p, const FlatLevel& f, Forms& m, const u64 (&d)[N],
                                            u32 (&n)[N], u64 (&off)[N], bool (&hit)[N]) {
  u32 at[N], line[N];
  u64 w[N], first[N];
  flat_place<N>(f, d, at, [](bool b) { return ballot(b) != 0; });
#pragma unroll
  for (int c = 0; c < N; ++c) {
    w[c] = d[c] + f.span_lo;
    line[c] = at[c] >> 2;
  }
  auto told = [&](u32 unit) {  // what its key says of a unit's first base
    return f.span_lo + ((u64)reinterpret_cast<const u32*>(f.keys)[unit] << f.key_shift);
  };
  if constexpr (kDepth == 1) {
    if (m.settle) {
#pragma unroll
      for (int c = 0; c < N; ++c)
        if (reinterpret_cast<const u32*>(f.keys)[line[c]] == (u32)(d[c] >> f.key_shift))
          line[c] = settle_unit(f, p.units, d[c], line[c]);
    }
  }
#pragma unroll
  for (int c = 0; c < N; ++c) first[c] = told(line[c]);
  // The unit for a word that its own unit begins above.  (After the fact: looked for ahead of every search, as
  // Forms.settle has it, tables whose units lie far apart lose 1 to 5 %.)
  auto settled = [&](int c, u32 unit) __attribute__((always_inline)) {
    if (!units_share(f, d[c], unit)) return unit - 1;
    return kDepth == 1 ? settle_unit_rare(f, p.units, d[c], unit) : settle_unit(f, p.units, d[c], unit);
  };
  bool lost[N];  // the way down ended at a node
#pragma unroll
  for (int c = 0; c < N; ++c) lost[c] = false;
  if constexpr (kDepth == 2) {
    if (p.f0_log2) {  // a level-0 key spans 2^f0_log2 nodes of the highest level
#pragma unroll
      for (int c = 0; c < N; ++c) {
        line[c] <<= p.f0_log2;
        first[c] = p.runs[line[c]];
      }
      for (u32 step = 1u << (p.f0_log2 - 1); step; step >>= 1) {
#pragma unroll
        for (int c = 0; c < N; ++c) {
          const u64 b = p.runs[line[c] + step];
          if (b <= w[c] && b != ~0ull) {
            line[c] += step;
            first[c] = b;
          }
        }
      }
#pragma unroll
      for (int c = 0; c < N; ++c)
        if (first[c] > w[c] && line[c]) {
          line[c] = settled(c, line[c] >> p.f0_log2) << p.f0_log2;
          first[c] = p.runs[line[c]];
          for (u32 step = 1u << (p.f0_log2 - 1); step; step >>= 1) {
            const u64 b = p.runs[line[c] + step];
            if (b <= w[c] && b != ~0ull) {
              line[c] += step;
              first[c] = b;
            }
          }
        }
    }
    for (u32 j = p.levels - 1; j >= 1; --j) {
      const uint4* a = p.nodes[j - 1];
      uint4 q[N][2];
#pragma unroll
      for (int c = 0; c < N; ++c) {
        q[c][0] = a[(u64)line[c] * 2];
        q[c][1] = a[(u64)line[c] * 2 + 1];
      }
      __builtin_amdgcn_sched_barrier(0);
      if (j + 1 == p.levels && !p.f0_log2) {
#pragma unroll
        for (int c = 0; c < N; ++c)
          if (first[c] + (q[c][0].x >> 5) > w[c] && line[c]) {
            line[c] = settled(c, line[c]);
            first[c] = told(line[c]);
            q[c][0] = a[(u64)line[c] * 2];
            q[c][1] = a[(u64)line[c] * 2 + 1];
          }
      }
#pragma unroll
      for (int c = 0; c < N; ++c) {
        u32 h = 0;
        const bool ok = pick_node(q[c], w[c], h, first[c]);
        lost[c] = lost[c] | !ok;
        line[c] = line[c] * 8 + (lost[c] ? 0u : h);  // (child 0 exists)
      }
    }
  }
  u64x2 e[N];
  auto wide = [&](int c, const uint4 (&q)[4]) __attribute__((always_inline)) {
    u32 h;
    n[c] = line[c] * 8;
    const bool ok = pick_wide_line(q, w[c], first[c], h, e[c]);
    n[c] += h;
    if (ok & !lost[c]) return;
    // the word lies below the line's first base, with the same truncated key (the end of the region before, for
    // one): most often in the line before, at the cost of one request more and not of a search
    if (!lost[c] && q[0].x != kMarked && line[c]) {
      const u32 l = kDepth == 1 ? settled(c, line[c]) : line[c] - 1;
      uint4 r[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) r[i] = p.leaf[(u64)l * 4 + i];
      const u64 b = kDepth == 1 ? told(l) : p.table[(u64)l * 8].base - (r[0].x >> 5);
      n[c] = l * 8;
      if (pick_wide_line(r, w[c], b, h, e[c])) {
        n[c] += h;
        return;
      }
    }
    // (a marked line, also the last one: among its own entries if it begins at or below w)
    const u32 lo = line[c] * 8;
    const bool own = !lost[c] && p.table[lo].base <= w[c];
    find_exact(p.table, own ? lo : 0u, own ? line_end(lo, p.n_alloc) : p.n_alloc, w[c], n[c], e[c]);
  };
  if (m.lines) {
    const uint4* a = kDepth == 2 && p.records ? p.records : p.cleaf;
    const u32 pieces = kDepth == 2 && p.records ? 4 : 2;
    uint4 q[N][2];
#pragma unroll
    for (int c = 0; c < N; ++c) {
      q[c][0] = a[(u64)line[c] * pieces];
      q[c][1] = a[(u64)line[c] * pieces + 1];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < N; ++c) {
      u32 h;
      n[c] = line[c] * 8;
      const bool ok = pick_compact_line(q[c], w[c], first[c], h, e[c]), packed = ok & !lost[c];
      n[c] += h;
      if (!packed) {
        uint4 r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = p.leaf[(u64)line[c] * 4 + i];
        wide(c, r);
      }
      m.marked += (u32)__popcll(ballot(!packed));
    }
  } else {
#pragma unroll
    for (int c = 0; c < N; ++c) {
      uint4 q[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) q[i] = p.leaf[(u64)line[c] * 4 + i];
      __builtin_amdgcn_sched_barrier(0);
      wide(c, q);
    }
  }
#pragma unroll
  for (int c = 0; c < N; ++c) {
    off[c] = w[c] - e[c].x;
    hit[c] = off[c] < e[c].y;
  }
}

template <int kDepth, int N>
__device__ __forceinline__ void any_search(const ScanParams& p, const FlatLevel& f, Forms& m, const u64 (&d)[N],
                                           u32 (&n)[N], u64 (&off)[N], bool (&hit)[N]) {
  if constexpr (kDepth == 0) flat_search<N>(p, f, d, n, off, hit, [](bool b) { return ballot(b) != 0; });
  else deep_search<kDepth, N>(p, f, m, d, n, off, hit);
}

// The new bases of the hits.
template <int kDepth, int N>
__device__ __forceinline__ void new_bases(const ScanParams& p, const Forms& m, const u32 (&n)[N], const bool (&hit)[N],
                                          u64 (&nb)[N]) {
  if (kDepth == 2 && p.records && m.lines) {
    u32 code[N];
    const u32* codes = reinterpret_cast<const u32*>(p.records);
#pragma unroll
    for (int c = 0; c < N; ++c) code[c] = hit[c] ? codes[(u64)(n[c] >> 3) * 16 + 8 + (n[c] & 7)] : 0;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < N; ++c) {
      nb[c] = m.nb_from + ((u64)code[c] << m.nb_shift);
      if (code[c] == kMarked) nb[c] = p.new_base[n[c]];
    }
  } else {
#pragma unroll
    for (int c = 0; c < N; ++c) nb[c] = hit[c] ? p.new_base[n[c]] : 0;
  }
}

// Which of the lane's eight words are candidates, one bit each.
__device__ __forceinline__ u32 flat_candidates(const FlatLevel& f, const u64 (&w)[kWpl]) {
  u32 mask = 0;
#pragma unroll
  for (int k = 0; k < kWpl; ++k) mask |= w[k] - f.span_lo < f.span_len ? 1u << k : 0u;
  return mask;
}

// Calls visit(k, rank) for the lane's candidates (word k), ranks in word order.  Returns how many there are.
template <bool kHalf, typename Visit>
__device__ __forceinline__ u32 rank_candidates(u32 mask, Visit visit) {
  constexpr int kPer = kHalf ? 4 : 2;
  u32 Q = 0;
  wave_lds_fence();
#pragma unroll
  for (int k = 0; k < kWpl / kPer; ++k) {
    u32 rank = Q;  // of this lane's first candidate in the piece
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const u64 m = ballot((mask >> (kPer * k + j) & 1) != 0);
      rank = __builtin_amdgcn_mbcnt_hi((u32)(m >> 32), __builtin_amdgcn_mbcnt_lo((u32)m, rank));
      Q += __popcll(m);
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (mask >> (kPer * k + j) & 1) visit(kPer * k + j, rank++);
  }
  wave_lds_fence();
  return Q;
}

// Chunks are handed out by one ticket counter, the first ones too: a workgroup only ever waits for chunks with smaller
// numbers, and those are in the hands of workgroups that run.  (First chunks by workgroup number, further ones from four
// counters: 0.8 / 1.7 / 5.9 M words 8.6 / 10.5 / 21.7 -> 7.7 / 8.6 / 19.8 us, but where other kernels hold compute units,
// the workgroups that run wait for those that cannot: 5.9 M words with 32 of 256 units held 46 -> 3,500 us.)  Counter and
// turn are reset by whoever makes the launch's last draw: every workgroup has read the turn before its first draw, so
// nobody looks at either again.
__device__ __forceinline__ u32 draw(const ScanParams& p) { return atomicAdd(p.ticket, 1u); }
__device__ __forceinline__ u32 drawn(const ScanParams& p, u32 turn, u32 last_draw, u32 got) {
  if (got == last_draw) {
    __hip_atomic_store(p.ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(p.turn, flat_next_turn(turn, scan_states(p.n_chunks)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  return got;
}

// A worker's sub-tile: round k's lane l has candidate 64 k + l.
struct Results {
  u64 e[kRounds];
  u32 Q, H, sub;
};

// Candidates [64 R0, 64 (R0 + N)).  stash: with output the sub-tile's words, else the candidates alone: read through
// their places, 26.8 M positions at 4-byte stride with 2 to 20 % candidates took 2 to 3 % longer.
template <int kDepth, bool kOut, int N, int R0>
__device__ __forceinline__ void search_rounds(const ScanParams& p, const FlatLevel& f, Forms& m, Entries pk, u64* stash,
                                            const unsigned short* places, Results& r) {
  const u32 lane = lane_id();
  u64 d[N], off[N];
  u32 n[N], idx[N];
  bool hit[N];
#pragma unroll
  for (int c = 0; c < N; ++c) idx[c] = places[(R0 + c) * 64 + lane] & (kSub - 1);
#pragma unroll
  for (int c = 0; c < N; ++c) {
    const bool valid = c < N - 1 || (u32)(R0 + c) * 64 + lane < r.Q;  // rounds before the last are full
    d[c] = valid ? stash[kOut ? idx[c] : (u32)(R0 + c) * 64 + lane] - f.span_lo : 0;
  }
  any_search<kDepth, N>(p, f, m, d, n, off, hit);
#pragma unroll
  for (int c = 0; c < N; ++c) {
    if (c == N - 1) hit[c] = hit[c] && (u32)(R0 + c) * 64 + lane < r.Q;
    r.e[R0 + c] = hit[c] ? pk.pack(idx[c], n[c], off[c]) : ~0ull;
    r.H += __popcll(ballot(hit[c]));
  }
  if constexpr (kOut) {
    u64 nb[N];
    new_bases<kDepth, N>(p, m, n, hit, nb);
#pragma unroll
    for (int c = 0; c < N; ++c)
      if (hit[c]) stash[idx[c]] = nb[c] + off[c];
  }
}
// Rounds [R0, R0 + N) as far as there are any, exactly as many as there are.
template <int kDepth, bool kOut, int N, int R0>
__device__ __forceinline__ void search_step(const ScanParams& p, const FlatLevel& f, Forms& m, Entries pk, u64* stash,
                                            const unsigned short* places, Results& r) {
  if constexpr (R0 + N > kRounds) {
    search_step<kDepth, kOut, N - 1, R0>(p, f, m, pk, stash, places, r);
  } else {
    if constexpr (N > 1) {
      if (r.Q <= (R0 + N - 1) * 64) return search_step<kDepth, kOut, N - 1, R0>(p, f, m, pk, stash, places, r);
    }
    search_rounds<kDepth, kOut, N, R0>(p, f, m, pk, stash, places, r);
  }
}
// Sub-tiles with up to so many candidates have their two rounds searched at once although the table has
// nodes, the others' rounds go one by one: sixteen waves cover each other's latency, and more chains
// per lane only thrash the vector L1 between a line's two halves.  2^27 words with 15 % candidates,
// 2^20 allocations: 685 us with the two rounds at once, 728 one by one; 16.8 M words with 25 %
// and 8 GiB regions: 160 and 145.  Where the line lies depends on table and form: us one by one / at once, 8.4 M words
// with exactly so many candidates in each sub-tile,
//                                  80            90            96            102           112
//   200,000 allocations            37.2 / 34.8   37.8 / 35.7   37.9 / 36.3   38.3 / 36.9   38.8 / 38.0
//   200,000, with output           49.4 / 47.1   50.1 / 49.2   50.7 / 50.5   51.6 / 51.9   53.6 / 54.1
//   2^20                           45.9 / 42.3   46.3 / 44.1   46.7 / 45.2   47.4 / 46.7   48.9 / 49.3
//   2^20, with output              70.6 / 70.6   74.2 / 75.4   76.9 / 78.3   79.6 / 81.2   84.4 / 85.9
constexpr u32 kFewCandidates = 96;
template <int kDepth, bool kOut, int R0 = 0>
__device__ __forceinline__ void search_all(const ScanParams& p, const FlatLevel& f, Forms& m, Entries pk, u64* stash,
                                           const unsigned short* places, Results& r) {
  if constexpr (R0 < kRounds) {
    if (r.Q <= R0 * 64) return;
    if constexpr (kDepth == 2 && R0 == 0) {
      if (r.Q > 64 && r.Q <= kFewCandidates) return search_rounds<kDepth, kOut, 2, 0>(p, f, m, pk, stash, places, r);
    }
    // Four rounds, seven and eight: four at once, where three would leave one or two alone.  (Not with output, whose
    // chains hold new bases as well.)  us, three / four at once: 13.4 M words, 4,096 allocations, 43 % candidates 51.0 /
    // 48.4; twice as many 4-byte positions 80 % dense 84.8 / 78.1, 100 % 88.8 / 84.2; 16,384 allocations, 100 % of 13.4 M
    // words 93.3 / 94.9.  Five rounds as four and one instead of three and two: 66.3 -> 68.7.
    if constexpr (kDepth == 0 && !kOut && R0 % 4 == 0) {
      if (const u32 left = r.Q - R0 * 64; left > 192 && (left <= 256 || left > 384)) {
        search_rounds<kDepth, kOut, 4, R0>(p, f, m, pk, stash, places, r);
        return search_all<kDepth, kOut, R0 + 4>(p, f, m, pk, stash, places, r);
      }
    }
    constexpr int N = kDepth == 0 ? 3 : kDepth == 1 ? 2 : 1;
    search_step<kDepth, kOut, N, R0>(p, f, m, pk, stash, places, r);
    search_all<kDepth, kOut, R0 + N>(p, f, m, pk, stash, places, r);
  }
}

// Position `at` of the input: the word, or the 64-bit value that starts at the 32-bit unit.
template <bool kHalf>
__device__ __forceinline__ u64 word_at(const ScanParams& p, u64 at) {
  if constexpr (!kHalf) return p.words[at];
  const u32* h = reinterpret_cast<const u32*>(p.words);
  return (u64)h[at] | (u64)h[at + 1] << 32;
}

// The wave's copy of a sub-tile in LDS: register k of a lane at its word's place.
template <bool kHalf>
__device__ __forceinline__ void stash_words(u64* stash, const u64 (&w)[kWpl]) {
  constexpr int kPer = kHalf ? 4 : 2;
#pragma unroll
  for (int k = 0; k < kWpl; k += 2) {
    u64x2 v;
    v.x = w[k];
    v.y = w[k + 1];
    *reinterpret_cast<u64x2*>(stash + (k / kPer * 64 + lane_id()) * kPer + k % kPer) = v;
  }
}

// The clerk works out where the states lie while the keys are staged, or behind the barrier where so few keys are there
// sooner.  us, before / behind the barrier: 9,000 words, 300 allocations 5.7 / 5.4, with output 6.0 / 5.8, 0.26 M words and 16
// 6.6 / 6.4; 0.26 M words and 4,096 with output 7.7 / 8.0, at 4-byte stride 6.5 / 6.7.
constexpr u32 kFewKeys = 1024;

// The ordered scan.
template <int kW, int kDepth, bool kHalf, bool kOut>
__global__ __launch_bounds__((kW + 1) * 64) void scan_kernel(ScanParams p) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ u32 s_next[2], s_cnt[2][kW], s_sum[2];
  __shared__ u64 s_excl[2];
  __shared__ u64 s_field[2];  // where the chunk tells its hits, and in the lowest bit the parity
  static_assert((u32)kW * kSub <= kFieldHits && (u32)kW * kSub < 1u << 16 && kW < 1 << 16,
                "a chunk's hits fit its field, and s_sum below the number of workers that are through");
  const u32 tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool clerk = wave == kW;
  u32 turn = 0;  // (lies in the prepared table's first block, which the check reads too)
  if (clerk) turn = __hip_atomic_load(p.turn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // Who tells a chunk's hits: the last of many workers, ahead of the barrier, or the clerk of few behind it.  us by the
  // clerk / by the last worker, a quarter pointers: seven workers, 0.3 M words 7.08 / 7.15, 0.6 M and 16,384 allocations 9.55 /
  // 9.70, 0.7 M with lines and output 11.83 / 12.00; fifteen, 1.7 M words 10.64 / 10.50, 5.9 M 22.1 / 21.8, 8.4 M 4-byte
  // positions 23.2 / 23.1, 12.3 M with lines and output 68.1 / 68.4, 2^27 with nodes and output 1,363 / 1,347.
  constexpr bool kWorkersTell = kW != (int)kFlatWorkers;
  FlatRegion region = p.region;  // (the header's first block as well)
  if (p.prepared) region = FlatRegion{(long long)p.prepared[4], (u32)p.prepared[5]};
  if (!prepared_ok(p)) {  // every workgroup sees the same: nothing is written
    if (blockIdx.x == 0 && tid == 0) raise_status(p.d_status, FDY_ST_BAD_PREPARED);
    return;
  }
  const bool few = kW == (int)kFlatWorkers && few_chunks(p.n_chunks);
  const bool single = gridDim.x >= p.n_chunks;  // every workgroup's first draw is its only chunk
  // the draw after which nobody draws again
  const u32 last_draw = single ? gridDim.x - 1 : p.n_chunks + gridDim.x - 1;
  FlatTurn t;
  FlatStates states;
  const u32 n_states = scan_states(p.n_chunks);
  const bool late = !kWorkersTell && p.top_n <= kFewKeys;
  auto lay_out = [&] {
    t = flat_turn(uniform(turn), n_states, region.states);
    states = FlatStates{reinterpret_cast<u64*>(reinterpret_cast<unsigned char*>(p.cstate) + region.first), t.s, t.parity};
  };
  if (clerk) {  // meanwhile the others stage the keys
    asm volatile("" : "+v"(turn) : : "memory");  // the turn has arrived before the draw goes out
    u32 got = 0;
    if (lane == 0) got = draw(p);
    if (!late) lay_out();
    if (lane == 0) {
      s_sum[0] = s_sum[1] = 0;
      s_next[0] = drawn(p, turn, last_draw, got);
      if (kWorkersTell && got < p.n_chunks) s_field[1] = (u64)states.field_of(got) | states.parity;
    }
  } else {
    (void)flat_stage<kW * 64>(p, smem_raw, tid, false);
  }
  const FlatLevel f = flat_level(p, smem_raw);
  __syncthreads();
  u32 chunk = s_next[0];
  if (clerk) {
    if (late) lay_out();
    for (u32 i = blockIdx.x * 64 + lane; i < t.dirty; i += gridDim.x * 64) {
      const u32 at = flat_to_clear(t, i, n_states);
      if (at != ~0u) st_state(&states.at[at], 0);
    }
    u32 prev = 0, prev_total = 0, b = 1;
    // the exclusive prefix of the chunk before, for the workers that wait to write it
    auto close = [&](u32 slot, auto meanwhile) __attribute__((always_inline)) {
      const u64 excl = few ? prefix_of_few(states, prev, p.spin_limit, p.d_status, meanwhile)
                           : exclusive_prefix(states, prev, p.spin_limit, p.d_status, meanwhile);
      if (lane == 0) {
        if (!few && (prev & 15) == 15) st_state(states.place(sum_state(prev >> 4)), make_sum(excl + prev_total, states.parity));
        if (prev + 1 == p.n_chunks) {  // the last chunk: the grand total
          *p.d_count = excl + prev_total;
          if (excl + prev_total > p.capacity) raise_status(p.d_status, FDY_ST_CAPACITY);
        }
        s_excl[slot] = excl;
      }
    };
    bool have_prev = false;
    for (; chunk < p.n_chunks; b ^= 1) {
      u32 got = p.n_chunks;
      if (lane == 0 && !single) got = draw(p);
      auto tell = [&] {
        if (lane != 0) return;
        if (!single) (void)drawn(p, turn, last_draw, got);
        s_next[b] = got;
        if (kWorkersTell && got < p.n_chunks) s_field[b ^ 1] = (u64)states.field_of(got) | states.parity;
      };
      if (have_prev) close(b, tell);
      else tell();
      __syncthreads();
      u32 total = 0;
#pragma unroll
      for (int i = 0; i < kW; ++i) total += s_cnt[b][i];
      if (!kWorkersTell && lane == 0) {
        const u32 field = make_field(total, states.parity);
        if (few) st_state(states.place(chunk), field);
        else states.store_field(chunk, field);
      }
      if (!few && chunk + 1 == p.n_chunks) {  // what the last sixteenth has no chunks for is nobody else's to write
        if (lane > (chunk & 15) && lane < 16) states.store_field((chunk & ~15u) + lane, 0);
        if (lane == 16 && (chunk & 15) != 15) st_state(states.place(sum_state(chunk >> 4)), 0);
      }
      prev = chunk;
      prev_total = total;
      have_prev = true;
      chunk = s_next[b];
    }
    if (have_prev) {
      close(b, [] {});
      __syncthreads();
    }
    return;
  }
  unsigned char* qb = smem_raw + flat_level_bytes(p.top_n, p.bucket_log2);
  u64* stash = reinterpret_cast<u64*>(qb) + wave * kSub;
  unsigned short* places = reinterpret_cast<unsigned short*>(qb + (size_t)kW * kSub * 8) + wave * kSub;
  const Entries pk{p.off_bits};
  auto write = [&](const Results& r, u64 pos) {
    const u32 wbase = r.sub * (u32)kSub;
#pragma unroll
    for (int k = 0; k < kRounds; ++k) {
      if ((u32)k * 64 < r.Q) {
        const u64 e = r.e[k];
        const bool hit = e != ~0ull;
        const u64 bl = ballot(hit);
        if (hit) {
          const u32 word = wbase + pk.word(e), region = pk.region(e);
          u64 off = pk.off(e);
          if (off == pk.none()) off = word_at<kHalf>(p, word) - p.table[region].base;
          store_reloc(p, pos + __builtin_amdgcn_mbcnt_hi((u32)(bl >> 32), __builtin_amdgcn_mbcnt_lo((u32)bl, 0)), word, region,
                      off);
        }
        pos += __popcll(bl);
      }
    }
  };
  Forms m = pick_forms<kDepth>(p);
  if constexpr (kDepth == 1) m.settle = units_share_keys(f, p.n_lines);
  Words<kHalf> raw = request_words<kHalf>(p, chunk * kW + wave);
  Results cur, prev;
  u32 prev_before = 0, b = 1;
  bool have_prev = false;
  for (; chunk < p.n_chunks; b ^= 1) {
    cur.sub = chunk * kW + wave;
    cur.H = 0;
    u64 w[kWpl];
    take_words<kHalf>(p, cur.sub, f.span_lo, raw, w);
    if constexpr (kOut) stash_words<kHalf>(stash, w);
    cur.Q = rank_candidates<kHalf>(flat_candidates(f, w), [&](int k, u32 rank) {
      places[rank] = (unsigned short)pos_in_sub<kHalf>(k, lane);
      if constexpr (!kOut) stash[rank] = w[k];
    });
    search_all<kDepth, kOut>(p, f, m, pk, stash, places, cur);
    if constexpr (kDepth != 0) count_marked(m, cur.Q);
    wave_lds_fence();
    if constexpr (kOut) unstash_words(p, cur.sub, stash);
    if (lane == 0) {
      s_cnt[b][wave] = cur.H;
      // the last of the workers tells the chunk's hits, ahead of the barrier and of what the others request behind it
      if constexpr (kWorkersTell) {
        const u64 to = s_field[b];
        const u32 sum = atomicAdd(&s_sum[b], 1u << 16 | cur.H) + (1u << 16 | cur.H);
        if (sum >> 16 == (u32)kW) {
          s_sum[b ^ 1] = 0;
          st_field(reinterpret_cast<unsigned short*>(to & ~1ull), make_field(sum & 0xffffu, (u32)to & 1));
        }
      }
    }
    __syncthreads();  // counts, the next ticket and the previous chunk's prefix are visible
    chunk = s_next[b];
    raw = request_words<kHalf>(p, chunk * kW + wave);  // in flight during the write
    u32 before = 0;
#pragma unroll
    for (int i = 0; i < kW; ++i) before += (u32)i < wave ? s_cnt[b][i] : 0;
    if (have_prev) write(prev, s_excl[b] + prev_before);
    prev = cur;
    prev_before = before;
    have_prev = true;
  }
  if (have_prev) {
    __syncthreads();
    write(prev, s_excl[b] + prev_before);
  }
}

// The unordered form (fdy_scan_rebase: rebased words, no relocation table): no tickets and no look-back,
// waves stride over the sub-tiles on their own, with the next words in flight during a search (no
// barrier lines the waves up here).  Eight waves a workgroup, two workgroups a compute unit: how many are best moves
// with the rounds that a size takes (us with 8 / 10 / 12 / 15 waves, sub-tiles per compute unit, a quarter candidates):
//   16,384 allocations   20  15.2 / 14.6 / 14.3 / 14.2   32  20.8 / 22.4 / 21.1 / 24.9   64  39.0 / 40.0 / 41.7 / 44.7
//                        256  139 / 136 / 144 / 155
//   300,000              20  23.8 / 20.9 / 21.6 / 25.2   32  29.8 / 37.2 / 31.8 / 39.3   64  57.3 / 61.2 / 61.4 / 64.9
//                        256  219 / 213 / 211 / 217
// and eight are seldom far from the best.  A workgroup's hits and "one more is through" go to one
// 64-bit counter in one addition (same-address additions are served one after the other, 12 ns
// each: one per wave is 25 us of them); the workgroup that finds itself last publishes the sum and
// leaves the counter zero.  out may be the input array itself: a wave has read a sub-tile
// completely before it writes any of it, and nobody else touches that sub-tile.
template <int kDepth>
__global__ __launch_bounds__(kRebaseWaves * 64) void scan_rebase_kernel(ScanParams p) {
  constexpr int kW = kRebaseWaves;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ u32 s_hits[kW];
  const u32 tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (!prepared_ok(p)) {  // every workgroup sees the same: nothing is read or written
    if (blockIdx.x == 0 && tid == 0) raise_status(p.d_status, FDY_ST_BAD_PREPARED);
    return;
  }
  const FlatLevel f = flat_stage<kW * 64>(p, smem_raw, tid, kDepth == 2 || !p.prepared);
  unsigned char* qb = smem_raw + flat_level_bytes(p.top_n, p.bucket_log2);
  u64* stash = reinterpret_cast<u64*>(qb) + wave * kSub;
  unsigned short* places = reinterpret_cast<unsigned short*>(qb + (size_t)kW * kSub * 8) + wave * kSub;
  const Entries pk{p.off_bits};
  const u32 stride = gridDim.x * kW;
  u32 sub = blockIdx.x * kW + wave;
  u64 w[kWpl];
  load_words<false>(p, sub, f.span_lo, w);
  Forms m = pick_forms<kDepth>(p);
  __syncthreads();
  if constexpr (kDepth == 1) m.settle = units_share_keys(f, p.n_lines);
  u32 H = 0;
  for (; sub < p.n_sub; sub += stride) {
    Results r;  // (nobody asks for the entries)
    r.H = 0;
    stash_words<false>(stash, w);
    r.Q = rank_candidates<false>(flat_candidates(f, w), [&](int k, u32 rank) {
      places[rank] = (unsigned short)pos_in_sub<false>(k, lane);
    });
    load_words<false>(p, sub + stride, f.span_lo, w);  // in flight during the search
    search_all<kDepth, true>(p, f, m, pk, stash, places, r);
    if constexpr (kDepth != 0) count_marked(m, r.Q);
    wave_lds_fence();
    unstash_words(p, sub, stash);
    wave_lds_fence();
    H += r.H;
  }
  if (lane == 0) s_hits[wave] = H;
  __syncthreads();
  if (tid == 0) {
    constexpr int kDoneShift = 40;  // hits stay below 2^32, workgroups below 2^20
    u64 mine = 1ull << kDoneShift;
    for (int i = 0; i < kW; ++i) mine += s_hits[i];
    const u64 sum = __hip_atomic_fetch_add(p.acc, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + mine;
    if ((sum >> kDoneShift) == gridDim.x) {
      *p.d_count = sum & ((1ull << kDoneShift) - 1);
      __hip_atomic_store(p.acc, (u64)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

struct ScanInit {
  const fdy_alloc* table;
  u32 n_alloc;
  u32 build;  // 0: only the state is cleared (the table's hierarchy exists already)
  u32 top_n;
  u32 sampled;  // level-0 keys that are real (the rest is padding)
  u32* top;
  unsigned short* bstart;
  u32 bucket_log2;
  u32 levels;
  u32 f0_log2;
  u64* units;  // see ScanParams
  u32 n_units;
  u64* runs;
  u32 n_runs;
  uint4* nodes[kMaxNodeLevels];
  u32 n_nodes[kMaxNodeLevels];
  uint4* leaf;   // the table's lines, wide and compact
  uint4* cleaf;
  u32 leaf_lines;  // ceil(n_alloc / 8), 0 if level 0 holds every base
  u64* cstate;   // states to clear (null: none)
  u32 n_states;
  u32* header;   // the 64 counters in front of the hierarchy
  u64* d_count;  // written 0 if not null (calls that find nothing to launch)
  u64* prepared;  // a prepared table's first block: 32 words, the first six from hdr, the rest 0
  PreparedHeader hdr;
};

// A call's base map beside the table's lines, for tables that outgrow the L2s: a record of 64
// bytes per line, its compact form and eight codes of 32 bits, one for each region's new base, which is
// from + (code << shift) with `from` and `shift` the same for all (behind the last record); a new
// base that has no such code is marked and read from the base map.  What bounds those scans is
// what their candidates pull through the fabric: a hit's new base then comes from the 128-byte line
// that the search has just fetched, two records to a line.
// `from` and `shift` are chosen from 64 evenly spaced regions, by every wave for itself: bases lie
// at multiples of a mapping granule, so a shift of theirs is good for all others nearly always.
// One thread per 16-byte piece, so that reads and writes are whole lines.  A prepared table that is
// not this call's is left alone, as by the scan that follows (which reports it): its lines may lie
// behind its end.
__global__ void scan_records_kernel(const uint4* cleaf, const u64* new_base, u32 n_alloc, u32 lines, uint4* out,
                                    const u64* prepared, u32 top_log2, u64 n_words, const fdy_alloc* table) {
  if (!prepared_ok(prepared, n_alloc, top_log2, n_words, table)) return;
  const u64 t = (u64)blockIdx.x * blockDim.x + threadIdx.x;
  const u64 i = t >> 2;
  const u32 piece = (u32)t & 3;
  const u64 sample = new_base[((u64)lane_id() * n_alloc) >> 6];
  u64 nb[4];
  uint4 v = make_uint4(0, 0, 0, 0);
  if (i < lines) {
    if (piece < 2) {
      v = cleaf[i * 2 + piece];
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const u64 r = i * 8 + (piece - 2) * 4 + k;
        nb[k] = r < n_alloc ? new_base[r] : sample;
      }
    }
  }
  u64 least = sample, any = sample ^ __shfl(sample, 0);
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const u64 o = __shfl_xor(least, d);
    least = o < least ? o : least;
    any |= __shfl_xor(any, d);
  }
  u32 shift = any ? (u32)__ffsll((long long)any) - 1u : 0u;
  if (shift > 31u) shift = 31u;
  // room below the least of the sample, a quarter of what the codes reach
  const u64 from = (least >> shift) > (1ull << 30) ? least - (1ull << (30 + shift)) : least & ((1ull << shift) - 1);
  if (t == 0) {
    u64* tail = reinterpret_cast<u64*>(out + (u64)lines * 4);
    tail[0] = from;
    tail[1] = shift;
  }
  if (i >= lines) return;
  if (piece >= 2) {
    u32 code[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const u64 x = nb[k] - from, c = x >> shift;
      code[k] = c << shift == x && c < kMarked ? (u32)c : kMarked;
    }
    v = make_uint4(code[0], code[1], code[2], code[3]);
  }
  out[t] = v;
}

// Builds the hierarchy and clears chunk states and counters: one thread per key, bucket, line, node.
// (kLines false: small tables.  Their few threads took 2.5 us longer in the code of both.)
template <bool kLines>
__global__ void scan_init_kernel(ScanInit a) {
  const u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
  if (a.cstate && i < a.n_states) a.cstate[i] = 0;
  if (a.header && i < 64) a.header[i] = 0;
  if (a.d_count && i == 0) *a.d_count = 0;
  if (a.prepared && i < 32) {
    const u64 h[6] = {a.hdr.magic,     (u64)a.hdr.n_alloc | ((u64)a.hdr.top_log2 << 32), a.hdr.max_words,
                      a.hdr.table_ptr, (u64)a.hdr.region.first,                          a.hdr.region.states};
    a.prepared[i] = i < 6 ? h[i] : 0;
  }
  if (!a.build) return;
  const u64 span_lo = a.n_alloc ? a.table[0].base : 0;
  const u64 span_len =
      a.n_alloc ? a.table[a.n_alloc - 1].base + a.table[a.n_alloc - 1].size - span_lo : 1;
  const u32 sh0 = 3 * a.levels + a.f0_log2;
  const u32 key_shift = key_shift_for(span_len, 31);
  if (i < a.top_n) a.top[i] = level0_key(a.table, a.n_alloc, sh0, i, span_lo, key_shift);
  if (i <= (1ull << a.bucket_log2)) {
    // bucket i starts at key value i << shift: how many level-0 keys lie below it
    const u64 target = i << bucket_shift_for(span_len, key_shift, a.bucket_log2);
    a.bstart[i] = (unsigned short)sampled_lower_bound(a.table, sh0, a.sampled, span_lo, key_shift, target);
  }
  if constexpr (!kLines) return;
  if (i < a.n_units) {
    const u64 j = i << sh0;
    a.units[i] = j < a.n_alloc ? a.table[j].base : ~0ull;
  }
  if (i < a.n_runs) {
    const u64 j = i << (3 * a.levels);
    a.runs[i] = j < a.n_alloc ? a.table[j].base : ~0ull;
  }
  // what leads to unit i of level j (lines: level 0) says of its first base
  auto told = [&](u64 i, u32 j) {
    const u64 k = i << (3 * (j + 1)), b = a.table[k].base;
    if (j + 1 < a.levels) {
      const u64 k0 = i >> 3 << (3 * (j + 2));
      return told_of_child(a.table, k0, 8ull << (3 * j), a.n_alloc, (u32)i & 7u);
    }
    return a.f0_log2 ? b : span_lo + ((b - span_lo) >> key_shift << key_shift);
  };
  for (u32 j = 1; j < a.levels; ++j)
    if (i < a.n_nodes[j - 1]) {
      PackedNode n;
      pack_node(a.table, i << (3 * (j + 1)), 1ull << (3 * j), a.n_alloc, told(i, j), n);
      a.nodes[j - 1][i * 2] = make_uint4(n.w[0], n.w[1], n.w[2], n.w[3]);
      a.nodes[j - 1][i * 2 + 1] = make_uint4(n.w[4], n.w[5], n.w[6], n.w[7]);
    }
  if (i < a.leaf_lines) {
    PackedLine l;
    pack_line(a.table, i * 8, a.n_alloc, told(i, 0), l);
#pragma unroll
    for (int h = 0; h < 4; ++h)
      a.leaf[i * 4 + h] = make_uint4(l.wide[4 * h], l.wide[4 * h + 1], l.wide[4 * h + 2], l.wide[4 * h + 3]);
#pragma unroll
    for (int h = 0; h < 2; ++h)
      a.cleaf[i * 2 + h] = make_uint4(l.compact[4 * h], l.compact[4 * h + 1], l.compact[4 * h + 2], l.compact[4 * h + 3]);
  }
}

// (a2) one wave per boundary: lower bound of word_off[s] among the reloc words.
__global__ void reloc_segment_kernel(const fdy_reloc* relocs, const u64* d_count, u64 capacity,
                                     const u64* word_off, u32 n_off, u64* reloc_off) {
  const u32 s = blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
  if (s >= n_off) return;
  u64 n = *d_count;
  if (n > capacity) n = capacity;
  const u64 target = word_off[s];
  const u32 r = wave_lower_bound([&](u32 i) { return (u64)relocs[i].word; }, 0u, (u32)n, target);
  if (lane_id() == 0) reloc_off[s] = r;
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// The search hierarchy of one table, as it lies in memory (a caller's prepared buffer or the
// front of a workspace).  Offsets are relative to the block's start.
struct TablePlan {
  u32 top_n, levels, f0_log2, sampled, bucket_log2;
  u32 n_units, n_runs, n_nodes[kMaxNodeLevels], leaf_lines;
  u32 spare;  // bytes for chunk states, the plan's last
  size_t off_top, off_bst, off_units, off_runs, off_nodes[kMaxNodeLevels], off_leaf, off_cleaf, off_records, bytes;
};

// From so many sub-tiles on a base map is laid beside the lines of a table with nodes, a launch of 5 to
// 8 us.  us without / with, a fifth candidates, 2 MiB granules:
//   allocations     4 Mi words    8 Mi          12 Mi         16 Mi         32 Mi
//   140,000         31.4 / 37.0   49.5 / 56.7   68.3 / 75.5   87.1 / 94.2   163 / 172
//   200,000         33.8 / 38.2   52.2 / 57.4   71.5 / 76.7   90.3 / 95.4   169 / 173
//   300,000         36.3 / 40.9   57.5 / 60.5   78.8 / 80.0   99.5 / 99.4   187 / 180
//   450,000         39.1 / 44.0   62.9 / 64.5   86.1 / 85.1   110 / 106     208 / 192
//   2^20            48.0 / 51.1   80.1 / 75.8   112 / 100     143 / 124     271 / 224
// So the line that would fit depends on the table: this one, for all, is where most tables gain; below 300,000
// allocations it costs up to a tenth.
constexpr u32 kRecordSubs = 24576;

bool plan_table(u32 n_alloc, TablePlan* pl) {
  const u32 top_log2 = (u32)fdy__tune_get(FDY_TUNE_SCAN_TOP_LOG2), top_cap = 1u << (top_log2 < kMostTopLog2 ? top_log2 : kMostTopLog2);
  // smallest sampling stride 2^f0_log2 * 8^levels for which the sampled bases fit the LDS level.
  // Strides between 8 and 64 are left out: the line's first base would have to be found among two
  // or four with a request of its own, and one more whole node costs no more.
  u32 levels = 0, f0_log2 = 0;
  auto sampled_at = [&](u32 lv, u32 f) { return (u32)(((u64)n_alloc + (1ull << (3 * lv + f)) - 1) >> (3 * lv + f)); };
  if (n_alloc > top_cap) {
    levels = sampled_at(1, 0) <= top_cap ? 1 : 2;
    while (sampled_at(levels, f0_log2) > top_cap) {
      if (++f0_log2 == 3) {
        f0_log2 = 0;
        ++levels;
      }
    }
  }
  if (levels > (u32)kMaxNodeLevels) return false;
  const u32 sampled = sampled_at(levels, f0_log2);
  pl->top_n = level0_entries(sampled);
  pl->levels = levels;
  pl->f0_log2 = f0_log2;
  pl->sampled = sampled;
  size_t off = 0;
  // level 0: one bucket per key, at most 2^13 (16 KiB of LDS; with 2^14 fifteen workers would not fit)
  pl->off_top = off;
  off += align256((size_t)pl->top_n * 4);
  pl->bucket_log2 = 0;
  while ((2u << pl->bucket_log2) <= pl->top_n && pl->bucket_log2 < kMostBucketLog2) ++pl->bucket_log2;
  pl->off_bst = off;
  off += align256((((size_t)1 << pl->bucket_log2) + 1) * 2);
  // (a buffer for a table serves every smaller one: where a level takes the place of longer arrays, these keep
  // the room of their longest)
  pl->n_units = levels ? sampled + kUnitWindow : 0;
  pl->off_units = off;
  off += align256((size_t)(levels >= 2 ? top_cap + kUnitWindow : pl->n_units) * 8);
  pl->n_runs = f0_log2 ? sampled << f0_log2 : 0;
  pl->off_runs = off;
  off += align256((levels >= 3 ? (size_t)top_cap * 4 : (size_t)pl->n_runs) * 8);
  for (u32 j = 1; j <= (u32)kMaxNodeLevels; ++j) {
    pl->n_nodes[j - 1] = j < levels ? (u32)(((u64)n_alloc + (8ull << 3 * j) - 1) >> (3 * j + 3)) : 0;
    pl->off_nodes[j - 1] = off;
    off += align256((size_t)pl->n_nodes[j - 1] * 32);
  }
  pl->leaf_lines = levels ? (u32)(((u64)n_alloc + 7) / 8) : 0;
  pl->off_leaf = off;
  off += align256((size_t)pl->leaf_lines * 64);
  pl->off_cleaf = off;
  off += align256((size_t)pl->leaf_lines * 32);
  pl->off_records = off;
  if (levels >= 2) off += align256((size_t)pl->leaf_lines * 64 + 16);
  // Room for chunk states beside chunk_state_bytes, so that even few of them lie far apart.  (Small
  // tables: no more than a buffer for one of them has always had, the rest is asked for on top.)
  pl->spare = levels ? 32768u
                     : (u32)(align256((size_t)pl->top_n * 2) +
                             align256((((size_t)1 << pl->bucket_log2) + 1) * 2));
  off += pl->spare;
  pl->bytes = off;
  return true;
}

constexpr size_t kStateHeader = 256;
u32 sub_tiles(u64 n_words) { return (u32)((n_words + kSub - 1) / kSub); }
// Counters, hierarchy and chunk states: the least a scan works with, and what it asks for.
size_t least_bytes(u64 n_words, const TablePlan& tp) {
  return kStateHeader + tp.bytes + chunk_state_bytes(sub_tiles(n_words));
}
size_t best_bytes(u64 n_words, const TablePlan& tp) {
  if (tp.levels) return least_bytes(n_words, tp);
  return kStateHeader + tp.bytes + flat_state_bytes(sub_tiles(n_words), tp.spare);
}

void fill_init(ScanInit* a, const fdy_alloc* d_table, u32 n_alloc, const TablePlan& tp, unsigned char* tb) {
  a->table = d_table;
  a->n_alloc = n_alloc;
  a->build = 1;
  a->top_n = tp.top_n;
  a->sampled = tp.sampled;
  a->top = (u32*)(tb + tp.off_top);
  a->bstart = (unsigned short*)(tb + tp.off_bst);
  a->bucket_log2 = tp.bucket_log2;
  a->levels = tp.levels;
  a->f0_log2 = tp.f0_log2;
  a->units = (u64*)(tb + tp.off_units);
  a->n_units = tp.n_units;
  a->runs = (u64*)(tb + tp.off_runs);
  a->n_runs = tp.n_runs;
  for (int j = 0; j < kMaxNodeLevels; ++j) {
    a->nodes[j] = (uint4*)(tb + tp.off_nodes[j]);
    a->n_nodes[j] = tp.n_nodes[j];
  }
  a->leaf = (uint4*)(tb + tp.off_leaf);
  a->cleaf = (uint4*)(tb + tp.off_cleaf);
  a->leaf_lines = tp.leaf_lines;
  a->cstate = nullptr;
  a->n_states = 0;
  a->header = nullptr;
  a->d_count = nullptr;
  a->prepared = nullptr;
  a->hdr = PreparedHeader{};
}

u32 init_threads(const TablePlan& tp, u32 n_states) {
  u32 n = tp.top_n > n_states ? tp.top_n : n_states;
  if (tp.n_runs > n) n = tp.n_runs;
  if (tp.leaf_lines > n) n = tp.leaf_lines;  // (more than nodes)
  if ((1u << tp.bucket_log2) + 1 > n) n = (1u << tp.bucket_log2) + 1;
  return n < 64 ? 64 : n;
}

}  // namespace
}  // namespace fdy

using namespace fdy;

extern "C" size_t fdy_scan_workspace_bytes(uint64_t n_words, uint32_t n_alloc) {
  if (n_words > kMaxWords) return 0;
  TablePlan tp;
  if (!plan_table(n_alloc, &tp)) return 0;
  return best_bytes(n_words, tp);
}

extern "C" size_t fdy_scan_staging_bytes(uint64_t n_words) {
  if (n_words > kMaxWords) return 0;
  // No scan has a use for it any more (a worker's registers hold the results of a whole sub-tile).  The answer stays
  // what it was, so that a caller's sizes do not move.
  constexpr u32 kStageWgs = 320;
  const u32 n_sub = sub_tiles(n_words), chunk = n_sub < (1u << fdy__tune_get(FDY_TUNE_SCAN_SMALL_LOG2)) ? 8 : 32;
  const u32 n_chunks = (n_sub + chunk - 1) / chunk;
  return align256((size_t)(n_chunks < kStageWgs ? n_chunks : kStageWgs) * 2 * chunk * kSub * sizeof(fdy_reloc));
}

extern "C" size_t fdy_scan_table_bytes(uint32_t n_alloc, uint64_t max_words) {
  if (max_words > kMaxWords) return 0;
  TablePlan tp;
  if (!plan_table(n_alloc, &tp)) return 0;
  return kPreparedHeader + best_bytes(max_words, tp);
}

extern "C" int fdy_scan_table_prepare(const fdy_alloc* d_table, uint32_t n_alloc, uint64_t max_words,
                                      void* d_prepared, size_t prepared_bytes, void* hip_stream) {
  if (max_words > kMaxWords) return FDY_ERR_INVALID_ARG;
  if (n_alloc && (!d_table || ((uintptr_t)d_table & 15))) return FDY_ERR_INVALID_ARG;
  TablePlan tp;
  if (!plan_table(n_alloc, &tp)) return FDY_ERR_INVALID_ARG;
  const size_t need = kPreparedHeader + least_bytes(max_words, tp);
  if (!d_prepared || ((uintptr_t)d_prepared & 255) || prepared_bytes < need) return FDY_ERR_WORKSPACE;
  hipStream_t stream = (hipStream_t)hip_stream;
  (void)hipGetLastError();
  unsigned char* pb = (unsigned char*)d_prepared;
  ScanInit a;
  fill_init(&a, d_table, n_alloc, tp, pb + kPreparedHeader + kStateHeader);
  a.prepared = (u64*)pb;
  a.hdr.magic = kPreparedMagic;
  a.hdr.n_alloc = n_alloc;
  a.hdr.top_log2 = (u32)fdy__tune_get(FDY_TUNE_SCAN_TOP_LOG2);
  a.hdr.max_words = max_words;
  a.hdr.table_ptr = (u64)(uintptr_t)d_table;
  a.header = (u32*)(pb + kPreparedHeader);
  const FlatRegion region = flat_region(sub_tiles(max_words), tp.spare,
                                        prepared_bytes - kPreparedHeader - kStateHeader - tp.bytes);
  a.hdr.region = region;
  a.cstate = (u64*)(pb + kPreparedHeader + kStateHeader + tp.bytes + region.first);
  a.n_states = region.states;
  a.d_count = nullptr;
  const u32 n_init = init_threads(tp, a.n_states);
  launch(FDY_PROF_SCAN_INIT, tp.levels ? scan_init_kernel<true> : scan_init_kernel<false>, dim3((n_init + 255) / 256),
         dim3(256), 0, stream, a);
  FDY_HIP_TRY(hipGetLastError());
  return FDY_OK;
}

namespace {

// One launch of a scan kernel: as many workgroups as can be resident (16 waves of 128 registers per
// compute unit), at most one per unit of work.
template <typename Kernel>
int launch_resident(int slot, Kernel kernel, std::atomic<u64>& allowed, u32 waves, size_t lds, u32 n_units, int dev,
                    int n_cu, hipStream_t stream, const ScanParams& p) {
  const u32 fit = (u32)(160 * 1024 / (lds + 512)), room = 16u / waves;
  u32 grid = (u32)n_cu * (fit < room ? fit : room);
  if (grid > n_units) grid = n_units;
  if (const int rc = allow_full_lds(kernel, dev, allowed)) return rc;
  launch(slot, kernel, dim3(grid), dim3(waves * 64), lds, stream, p);
  FDY_HIP_TRY(hipGetLastError());
  return FDY_OK;
}

template <int kW, int kDepth, bool kHalf, bool kOut>
int launch_workers(size_t lds, int dev, int n_cu, hipStream_t stream, const ScanParams& p) {
  static std::atomic<u64> allowed;
  return launch_resident(kOut ? FDY_PROF_SCAN_OUT : FDY_PROF_SCAN_MAIN, scan_kernel<kW, kDepth, kHalf, kOut>, allowed,
                         kW + 1, lds + kW * kWorkerLds, p.n_chunks, dev, n_cu, stream, p);
}
template <int kDepth>
int launch_ordered(u32 workers, bool half, bool out, size_t lds, int dev, int n_cu, hipStream_t stream,
                   const ScanParams& p) {
  auto with = [&](auto half_c, auto out_c) {
    constexpr bool h = decltype(half_c)::value, o = decltype(out_c)::value;
    return workers == kFlatWorkers ? launch_workers<kFlatWorkers, kDepth, h, o>(lds, dev, n_cu, stream, p)
                                   : launch_workers<kFlatWorkersBig, kDepth, h, o>(lds, dev, n_cu, stream, p);
  };
  return out    ? with(std::false_type{}, std::true_type{})
         : half ? with(std::true_type{}, std::false_type{})
                : with(std::false_type{}, std::false_type{});
}
template <int kDepth>
int launch_rebase(size_t lds, int dev, int n_cu, hipStream_t stream, const ScanParams& p) {
  static std::atomic<u64> allowed;
  return launch_resident(FDY_PROF_SCAN_REBASE, scan_rebase_kernel<kDepth>, allowed, kRebaseWaves,
                         lds + kRebaseWaves * kWorkerLds, (p.n_sub + kRebaseWaves - 1) / kRebaseWaves, dev, n_cu, stream, p);
}

}  // namespace

// Shared by the scans: checks, where hierarchy and state lie (in the caller's prepared table, or
// built into the workspace by a launch of this call), then the main kernel.
static int scan_launch(const uint64_t* d_words, uint64_t n_words, const fdy_alloc* d_table,
                       uint32_t n_alloc, fdy_reloc* d_relocs, uint64_t reloc_capacity, uint64_t* d_count,
                       const uint64_t* d_new_base, uint64_t* d_out, const void* d_prepared, void* d_workspace,
                       size_t workspace_bytes, uint32_t* d_status, void* hip_stream, bool half = false,
                       bool ordered_out = false) {
  const bool fused = d_out != nullptr && !ordered_out;  // no relocation table, no ordering
  if (n_words > kMaxWords) return FDY_ERR_INVALID_ARG;
  if (!d_count) return FDY_ERR_INVALID_ARG;
  if (n_words && (!d_words || ((uintptr_t)d_words & 15))) return FDY_ERR_INVALID_ARG;
  if (n_alloc && (!d_table || ((uintptr_t)d_table & 15))) return FDY_ERR_INVALID_ARG;
  if (reloc_capacity && (!d_relocs || ((uintptr_t)d_relocs & 15))) return FDY_ERR_INVALID_ARG;
  if (d_prepared && ((uintptr_t)d_prepared & 255)) return FDY_ERR_INVALID_ARG;
  TablePlan tp;
  if (!plan_table(n_alloc, &tp)) return FDY_ERR_INVALID_ARG;
  const u32 n_sub = sub_tiles(n_words);
  const bool whole = tp.levels == 0;
  const u32 workers = flat_workers(n_sub, whole), n_chunks = flat_chunks(n_sub, whole);
  // where things lie
  unsigned char* ws = (unsigned char*)d_workspace;
  unsigned char* state;
  if (d_prepared) {
    // the caller vouches for the buffer (made by fdy_scan_table_prepare for this table and at
    // least this many words, under the same tuning)
    unsigned char* pb = (unsigned char*)const_cast<void*>(d_prepared);
    state = pb + kPreparedHeader;
    if (ws && ((uintptr_t)ws & 255)) return FDY_ERR_WORKSPACE;
  } else {
    if (!ws || ((uintptr_t)ws & 255) || workspace_bytes < least_bytes(n_words, tp)) return FDY_ERR_WORKSPACE;
    state = ws;
  }
  unsigned char* const tb = state + kStateHeader;
  u64* const cstate = (u64*)(tb + tp.bytes);
  hipStream_t stream = (hipStream_t)hip_stream;
  (void)hipGetLastError();  // drop any stale error left by earlier, unrelated runtime calls
  int dev = 0, n_cu = 256;
  if (const int rc = current_device(&dev, &n_cu)) return rc;
  const bool nothing = n_sub == 0 || n_alloc == 0;  // no word can be a pointer
  FlatRegion region{0, 0};
  ScanInit a;
  fill_init(&a, d_table, n_alloc, tp, tb);
  if (d_prepared) {
    if (nothing) {  // only the count is owed
      ScanInit z = ScanInit{};
      z.d_count = (u64*)d_count;
      hipLaunchKernelGGL(scan_init_kernel<false>, dim3(1), dim3(64), 0, stream, z);
      FDY_HIP_TRY(hipGetLastError());
    }
  } else {
    a.header = (u32*)state;
    if (!fused) {
      region = flat_region(n_sub, tp.spare, workspace_bytes - kStateHeader - tp.bytes);
      a.cstate = cstate + region.first / 8;
      a.n_states = flat_extent(flat_spread(scan_states(n_chunks), region.states), scan_states(n_chunks));
    }
    a.d_count = nothing ? (u64*)d_count : nullptr;
    const u32 n_init = init_threads(tp, a.n_states);
    launch(FDY_PROF_SCAN_INIT, tp.levels ? scan_init_kernel<true> : scan_init_kernel<false>, dim3((n_init + 255) / 256),
           dim3(256), 0, stream, a);
    FDY_HIP_TRY(hipGetLastError());
  }
  if (n_sub == 0) return FDY_OK;
  if (n_alloc == 0) {  // nothing can be a pointer; forms with an output still owe the copy
    if (d_out && d_out != d_words)
      FDY_HIP_TRY(hipMemcpyAsync(d_out, d_words, n_words * 8, hipMemcpyDeviceToDevice, stream));
    return FDY_OK;
  }

  ScanParams p;
  p.words = (const u64*)d_words;
  p.n_words = n_words;
  p.table = d_table;
  p.n_alloc = n_alloc;
  p.relocs = d_relocs;
  p.capacity = reloc_capacity;
  p.d_count = (u64*)d_count;
  // state: 2..3 = hit accumulator (64 bits), 8 = turn (a prepared table's lies in its header), 32 = ticket, in a memory
  // line of its own
  p.ticket = (u32*)state + 32;
  p.acc = (u64*)state + 1;
  p.turn = d_prepared ? (u32*)const_cast<void*>(d_prepared) + kPreparedTurn / 4 : (u32*)state + 8;
  p.region = region;
  p.cstate = cstate;
  p.n_chunks = n_chunks;
  p.prepared = (const u64*)d_prepared;
  p.top_log2 = (u32)fdy__tune_get(FDY_TUNE_SCAN_TOP_LOG2);
  p.top = a.top;
  p.bstart = a.bstart;
  p.bucket_log2 = a.bucket_log2;
  p.top_n = (tp.sampled + 3) & ~3u;
  p.levels = tp.levels;
  p.f0_log2 = tp.f0_log2;
  p.units = a.units;
  p.runs = a.runs;
  for (int j = 0; j < kMaxNodeLevels; ++j) p.nodes[j] = a.nodes[j];
  p.leaf = a.leaf;
  p.cleaf = a.cleaf;
  p.n_lines = tp.leaf_lines;
  p.records = nullptr;
  if ((ordered_out || fused) && tp.levels >= 2 && n_sub >= kRecordSubs) {
    uint4* rec = (uint4*)(tb + tp.off_records);
    launch(FDY_PROF_SCAN_RECORDS, scan_records_kernel, dim3((u32)(((u64)tp.leaf_lines * 4 + 255) / 256)), dim3(256), 0,
           stream, (const uint4*)a.cleaf, (const u64*)d_new_base, n_alloc, tp.leaf_lines, rec, p.prepared, p.top_log2,
           p.n_words, p.table);
    FDY_HIP_TRY(hipGetLastError());
    p.records = rec;
  }
  p.n_sub = n_sub;
  p.off_bits = entry_off_bits(n_alloc);
  p.d_status = d_status;
  p.spin_limit = (u32)fdy__tune_get(FDY_TUNE_SCAN_SPIN_LIMIT);
  p.new_base = (const u64*)d_new_base;
  p.out = (u64*)d_out;

  const size_t lds = flat_level_bytes(p.top_n, p.bucket_log2);
  if (fused)
    return tp.levels == 0   ? launch_rebase<0>(lds, dev, n_cu, stream, p)
           : tp.levels == 1 ? launch_rebase<1>(lds, dev, n_cu, stream, p)
                            : launch_rebase<2>(lds, dev, n_cu, stream, p);
  return tp.levels == 0   ? launch_ordered<0>(workers, half, ordered_out, lds, dev, n_cu, stream, p)
         : tp.levels == 1 ? launch_ordered<1>(workers, half, ordered_out, lds, dev, n_cu, stream, p)
                          : launch_ordered<2>(workers, half, ordered_out, lds, dev, n_cu, stream, p);
}

extern "C" int fdy_scan_pointers(const uint64_t* d_words, uint64_t n_words, const fdy_alloc* d_table,
                                 uint32_t n_alloc, fdy_reloc* d_relocs, uint64_t reloc_capacity,
                                 uint64_t* d_count, const void* d_prepared, void* d_workspace,
                                 size_t workspace_bytes,
                                 uint32_t* d_status, void* hip_stream) {
  return scan_launch(d_words, n_words, d_table, n_alloc, d_relocs, reloc_capacity, d_count, nullptr, nullptr,
                     d_prepared, d_workspace, workspace_bytes, d_status, hip_stream);
}

extern "C" int fdy_scan_pointers_stride4(const uint32_t* d_units, uint64_t n_units, const fdy_alloc* d_table,
                                         uint32_t n_alloc, fdy_reloc* d_relocs, uint64_t reloc_capacity,
                                         uint64_t* d_count, const void* d_prepared, void* d_workspace,
                                 size_t workspace_bytes,
                                         uint32_t* d_status, void* hip_stream) {
  // position q pairs unit q with unit q + 1: one position less than units
  const uint64_t n_pos = n_units >= 2 ? n_units - 1 : 0;
  if (n_units && !d_units) return FDY_ERR_INVALID_ARG;
  return scan_launch(reinterpret_cast<const uint64_t*>(d_units), n_pos, d_table, n_alloc, d_relocs,
                     reloc_capacity, d_count, nullptr, nullptr, d_prepared, d_workspace, workspace_bytes, d_status,
                     hip_stream, true);
}

extern "C" int fdy_scan_rebase(const uint64_t* d_words, uint64_t n_words, const fdy_alloc* d_table,
                               uint32_t n_alloc, const uint64_t* d_new_base, uint64_t* d_out_words,
                               uint64_t* d_count, const void* d_prepared, void* d_workspace,
                                 size_t workspace_bytes,
                               uint32_t* d_status, void* hip_stream) {
  if (n_words && (!d_out_words || ((uintptr_t)d_out_words & 15))) return FDY_ERR_INVALID_ARG;
  if (n_alloc && (!d_new_base || ((uintptr_t)d_new_base & 7))) return FDY_ERR_INVALID_ARG;
  if (n_words == 0) {  // nothing to write; keep the count defined
    if (!d_count) return FDY_ERR_INVALID_ARG;
    return scan_launch(d_words, 0, d_table, n_alloc, nullptr, 0, d_count, nullptr, nullptr, d_prepared, d_workspace,
                       workspace_bytes, d_status, hip_stream);
  }
  if (d_out_words != d_words) {  // exactly the same array, or disjoint
    const uintptr_t a = (uintptr_t)d_words, b = (uintptr_t)d_out_words, len = (uintptr_t)n_words * 8;
    if (a < b + len && b < a + len) return FDY_ERR_INVALID_ARG;
  }
  return scan_launch(d_words, n_words, d_table, n_alloc, nullptr, 0, d_count, d_new_base, d_out_words,
                     d_prepared, d_workspace, workspace_bytes, d_status, hip_stream);
}

extern "C" int fdy_scan_pointers_rebase(const uint64_t* d_words, uint64_t n_words, const fdy_alloc* d_table,
                                        uint32_t n_alloc, fdy_reloc* d_relocs, uint64_t reloc_capacity,
                                        uint64_t* d_count, const uint64_t* d_new_base, uint64_t* d_out_words,
                                        const void* d_prepared, void* d_workspace, size_t workspace_bytes, uint32_t* d_status,
                                        void* hip_stream) {
  if (n_words && (!d_out_words || ((uintptr_t)d_out_words & 15))) return FDY_ERR_INVALID_ARG;
  if (n_alloc && (!d_new_base || ((uintptr_t)d_new_base & 7))) return FDY_ERR_INVALID_ARG;
  if (n_words) {  // the output is written while other workgroups still read the input
    const uintptr_t a = (uintptr_t)d_words, b = (uintptr_t)d_out_words, len = (uintptr_t)n_words * 8;
    if (a < b + len && b < a + len) return FDY_ERR_INVALID_ARG;
  }
  return scan_launch(d_words, n_words, d_table, n_alloc, d_relocs, reloc_capacity, d_count, d_new_base,
                     n_words ? d_out_words : nullptr, d_prepared, d_workspace, workspace_bytes, d_status, hip_stream, false,
                     true);
}

extern "C" int fdy_reloc_segment(const fdy_reloc* d_relocs, const uint64_t* d_count,
                                 uint64_t reloc_capacity, const uint64_t* d_word_off, uint32_t n_off,
                                 uint64_t* d_reloc_off, void* hip_stream) {
  if (n_off == 0) return FDY_OK;
  if (!d_count || !d_word_off || !d_reloc_off) return FDY_ERR_INVALID_ARG;
  if (reloc_capacity && !d_relocs) return FDY_ERR_INVALID_ARG;
  (void)hipGetLastError();
  launch(FDY_PROF_SEGMENT, reloc_segment_kernel, dim3((n_off + 3) / 4), dim3(256), 0, (hipStream_t)hip_stream,
         d_relocs, (const u64*)d_count, reloc_capacity, (const u64*)d_word_off, n_off, (u64*)d_reloc_off);
  FDY_HIP_TRY(hipGetLastError());
  return FDY_OK;
}
