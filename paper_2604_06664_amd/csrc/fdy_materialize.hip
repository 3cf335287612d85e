// fdy_materialize.hip - (c) template materialization for gfx950.
//
// Section 4.2.1 prepares, at LOAD time, the parameter set of every non-template graph on
// CPU worker threads; Section 4.2.2 patches rank-dependent communication arguments.  Here
// the same preparation is one streaming pass on the GPU over all (base map, graph, tile)
// units, bounded by the HBM write of the output:
//
//   prep A (one workgroup)   prefix sums over the output graphs: where each graph's words,
//                            nodes and tiles start; verifies the caller's totals.  A launch
//                            of its own only above 1024 output graphs: up to there every
//                            block of prep B computes the sums itself, in LDS.
//   prep B (one launch)      three kinds of blocks side by side.  Tile blocks (one thread per
//                            tile) resolve each output tile once, independent of the base map:
//                            its graph, template, source words, and the sub-ranges of the
//                            template's relocation list and the graph's override list that
//                            fall inside the tile (a thread searches where its tile's ranges
//                            begin; they end where the next tile's begin).  Patch blocks (one
//                            thread per tile and rank) do the same for each rank's patch list.
//                            Dims blocks (one thread per node) write the launch dimensions of
//                            the template with the graph's grid overrides.  The kernel's time is
//                            its longest chain of dependent loads: up to 2,048 tiles several lanes
//                            search for each end of a slice together; beyond, per-lane searches,
//                            tens of thousands side by side.  One launch rather than four because
//                            small archives are bound by launch latency.
//   main  (tile x map group) stages the template tile in LDS and the tile's relocation entries
//                            in registers once, then per base map of its group scatters c2
//                            rebased pointers (new_base[m][region] + offset), c3 32-bit
//                            overrides and c4 64-bit rank patches into LDS in that order and
//                            streams the tile out by whole memory lines.  Templates,
//                            relocation lists and base maps are re-read per group from L2 /
//                            Infinity Cache; only the output is compulsory HBM traffic.
//   small launches           (every workgroup of main resident at once): no prep launch at
//                            all; each workgroup of main resolves its own tile first, and
//                            extra blocks of the same launch write the dimensions and check
//                            the short lists.  Same results, one launch less.
// What bounds main is round trips to memory in front of a workgroup's first store, as far as the
// workgroups of a compute unit (five, by 96 registers; more registers at once than that cost more than
// they hide) do not cover each other's, and the rate of the stores beyond: hence loads without branches.
// The order of every list is verified on the way (FDY_ST_BAD_ORDER): the relocation lists
// where main reads them, the short lists by blocks of the prep launch (or of main).
#include <mutex>
#include <type_traits>

#include "fdy_device.hpp"
#include "fdy_internal.h"

namespace fdy {
namespace {

constexpr int kMatBlock = 256;
constexpr int kMatBuf = 2048;             // words of a workgroup's tile buffer (16 KiB)
constexpr int kLine = 16;                 // words of a 128-byte memory line
// Words per tile.  A wave stores whole 128-byte lines, wherever the tile begins: a store that straddles two more lines
// than it fills cost the launch 3 to 5 % (us per pass: 67 graphs to 8 ranks, 240 MB, 93.6 -> 91.2; to 256 maps, 1.56 GB,
// 297 -> 287) and wrote partial lines (256 maps 1,571.96 -> 1,559.29 MB by counter, of 1,559.27 of output).  A line less than the buffer, so that a tile and the words in front of it in its first line are four
// 16-byte stores per thread: with a fifth for a few lanes, or with assignments that wrap, the gain went into registers.
// The lines that two tiles share are left (without them 88.9 and 285).
constexpr int kMatTile = kMatBuf - kLine;
// Tiles of a graph, and the words of one that has `left` words before its graph's end: a graph's last tile fills the
// buffer before another is begun.  (Graphs of 2,033 to 2,048 words as two tiles: 2,000 of 2,040 to 8 maps 62 -> 89 us.)
__device__ __forceinline__ u64 tiles_of(u64 nw) {
  return nw > (u64)kMatBuf ? (nw - kLine + kMatTile - 1) / kMatTile : (u64)(nw != 0);
}
__device__ __forceinline__ u32 tile_words(u64 left) { return left <= (u64)kMatBuf ? (u32)left : (u32)kMatTile; }

struct __attribute__((aligned(16))) MatTile {  // 48 B
  u64 src_word;  // index into src_words of the tile's first word
  u64 out_word;  // word offset of the tile inside one map's output
  u32 n_words;   // 0: unused entry
  u32 k0;
  u32 reloc_lo, reloc_hi, ovr_lo, ovr_hi;
  u32 reloc_seg;  // first entry of the template's relocation list (order checks stop there)
  u32 pad;
};
static_assert(sizeof(MatTile) == 48, "MatTile");

struct MatHeader {
  u32 n_tiles;
  u32 ok;
};

struct MatWs {
  MatHeader* hdr;
  u64* out_word_off;  // [G+1]
  u64* out_node_off;  // [G+1]
  u64* tile_off;      // [G+1]
  uint2* tile_patch;  // [max_tiles * R]
  MatTile* tiles;     // [n_entries], those from max_tiles on for no tile
  u32 max_tiles;
  u32 n_entries;
};

struct MatParams {
  fdy_mat_desc d;
  MatWs ws;
  u64* out_words;
  u32* out_dims;
  u32* d_status;
  u32 map_group;  // consecutive base maps handled by one workgroup of the main kernel
  u32 stream_once;  // templates and relocation lists are read once and too large to stay cached
};

// Word and node counts of output graph g (those of its template).  False, with zero counts, if
// its template or the template's source graph is out of range or has 2^32 words or more.
__device__ __forceinline__ bool graph_sizes(const MatParams& p, u32 g, u64& nw, u64& nn) {
  const fdy_mat_desc& d = p.d;
  nw = 0;
  nn = 0;
  const u32 t = d.graph_tmpl[g];
  const u32 s = t < d.n_templates ? d.tmpl_graph[t] : 0xffffffffu;
  if (s >= d.n_src_graphs) return false;
  nw = d.src_word_off[s + 1] - d.src_word_off[s];
  if (p.out_dims) nn = d.src_node_off[s + 1] - d.src_node_off[s];
  if (nw >> 32) {  // a template must stay below 2^32 words
    nw = 0;
    nn = 0;
    return false;
  }
  // a graph without words has no tile that would meet (and reject) its entries
  if (nw == 0 && (d.src_reloc_off[s + 1] != d.src_reloc_off[s] || d.ovr_off[g + 1] != d.ovr_off[g])) return false;
  return true;
}

// The same for the graphs i * 256 + threadIdx.x, i < kPer, of a workgroup of 256 threads, loads
// of one step requested for all of them before the next step: three round trips (template, source
// graph, offsets) however many graphs there are.  (One graph after the other they were twelve,
// half of what the small launches took: prep of the MoE archive's 67 graphs 13.5 -> 11.2 us.)
// rows: null, or where else a graph's words and lists lie (requested with the offsets).
struct GraphRow {
  u64 src_word;
  u32 rl0, rl1, ov0, ov1;
};
template <u32 kPer>
__device__ __forceinline__ bool graphs_sizes(const MatParams& p, u64 (&nw)[kPer], u64 (&nn)[kPer], u32 (&src)[kPer],
                                             GraphRow* rows = nullptr, u32* tmpl = nullptr) {
  const fdy_mat_desc& d = p.d;
  const u32 G = d.n_graphs, tid = threadIdx.x;
  u32 t[kPer];
  u64 w0[kPer], w1[kPer], n0[kPer], n1[kPer];
  bool bad = false;
#pragma unroll
  for (u32 i = 0; i < kPer; ++i) {
    const u32 g = i * 256 + tid;
    t[i] = g < G ? d.graph_tmpl[g] : 0xffffffffu;
  }
#pragma unroll
  for (u32 i = 0; i < kPer; ++i) src[i] = t[i] < d.n_templates ? d.tmpl_graph[t[i]] : 0xffffffffu;
#pragma unroll
  for (u32 i = 0; i < kPer; ++i) {
    w0[i] = w1[i] = n0[i] = n1[i] = 0;
    if (src[i] < d.n_src_graphs) {
      w0[i] = d.src_word_off[src[i]];
      w1[i] = d.src_word_off[src[i] + 1];
      if (p.out_dims) {
        n0[i] = d.src_node_off[src[i]];
        n1[i] = d.src_node_off[src[i] + 1];
      }
      if (rows) {
        const u32 g = i * 256 + tid;
        rows[i].rl0 = (u32)d.src_reloc_off[src[i]];
        rows[i].rl1 = (u32)d.src_reloc_off[src[i] + 1];
        rows[i].ov0 = (u32)d.ovr_off[g];
        rows[i].ov1 = (u32)d.ovr_off[g + 1];
      }
    }
  }
#pragma unroll
  for (u32 i = 0; i < kPer; ++i) {
    if (rows) rows[i].src_word = w0[i];
    if (tmpl) tmpl[i] = t[i];
  }
#pragma unroll
  for (u32 i = 0; i < kPer; ++i) {
    const u32 g = i * 256 + tid, s = src[i];
    nw[i] = w1[i] - w0[i];
    nn[i] = n1[i] - n0[i];
    if (g >= G) continue;
    if (s >= d.n_src_graphs) {
      bad = true;
    } else if (nw[i] >> 32) {  // a template must stay below 2^32 words
      nw[i] = 0;
      nn[i] = 0;
      bad = true;
    } else if (nw[i] == 0 && (d.src_reloc_off[s + 1] != d.src_reloc_off[s] || d.ovr_off[g + 1] != d.ovr_off[g])) {
      bad = true;  // a graph without words has no tile that would meet (and reject) its entries
    }
  }
  return bad;
}

// Exclusive scans of three values per thread at once over a workgroup of 256; s_buf: 12 u64.
__device__ __forceinline__ void block_excl_scan3(u64 (&v)[3], u64 (&total)[3], u64* s_buf) {
  const u32 l = lane_id(), w = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const u64 inc = wave_incl_scan(v[k]);
    if (l == 63) s_buf[k * 4 + w] = inc;
    v[k] = inc - v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    total[k] = 0;
#pragma unroll
    for (u32 i = 0; i < 4; ++i) {
      const u64 x = s_buf[k * 4 + i];
      if (i < w) v[k] += x;
      total[k] += x;
    }
  }
  __syncthreads();
}

// Do the totals match what the caller sized the launch and the outputs for?
__device__ __forceinline__ bool totals_ok(const MatParams& p, u64 words, u64 nodes, u64 tiles) {
  bool ok = words == p.d.out_words_per_map && tiles <= p.ws.max_tiles;
  if (p.out_dims && nodes != p.d.out_nodes_total) ok = false;
  return ok;
}

__global__ __launch_bounds__(1024) void mat_prep_graphs_kernel(MatParams p) {
  __shared__ u64 s_buf[17];
  const fdy_mat_desc& d = p.d;
  const u32 G = d.n_graphs;
  u64 carry_w = 0, carry_n = 0, carry_t = 0;
  bool bad = false;
  for (u32 g0 = 0; g0 < G; g0 += 1024) {
    const u32 g = g0 + threadIdx.x;
    u64 nw = 0, nn = 0;
    if (g < G && !graph_sizes(p, g, nw, nn)) bad = true;
    const u64 nt = tiles_of(nw);
    u64 tw, tn, tt;
    const u64 ew = block_excl_scan(nw, s_buf, tw);
    const u64 en = block_excl_scan(nn, s_buf, tn);
    const u64 et = block_excl_scan(nt, s_buf, tt);
    if (g < G) {
      p.ws.out_word_off[g] = carry_w + ew;
      p.ws.out_node_off[g] = carry_n + en;
      p.ws.tile_off[g] = carry_t + et;
    }
    carry_w += tw;
    carry_n += tn;
    carry_t += tt;
  }
  if (bad) raise_status(p.d_status, FDY_ST_BAD_INDEX);
  if (threadIdx.x == 0) {
    p.ws.out_word_off[G] = carry_w;
    p.ws.out_node_off[G] = carry_n;
    p.ws.tile_off[G] = carry_t;
    const bool ok = totals_ok(p, carry_w, carry_n, carry_t);
    if (!ok) raise_status(p.d_status, FDY_ST_BAD_SIZE);
    p.ws.hdr->n_tiles = ok ? (u32)carry_t : 0u;
    p.ws.hdr->ok = ok ? 1u : 0u;
  }
}

// Per-lane lower bound: first index in [lo, hi) whose key is not below target (hi if none).
// One dependent load per halving; used where thousands of independent searches run side by
// side (one per lane), so that the memory system sees few requests per search.
template <typename KeyFn>
__device__ __forceinline__ u32 lane_lower_bound(KeyFn key, u32 lo, u32 hi, u64 target) {
  while (lo < hi) {
    const u32 mid = lo + ((hi - lo) >> 1);
    if (key(mid) < target) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// Two per-lane lower bounds at once (A and B: independent lists), four-way: each step loads
// three keys per list, all six before any is used, so a list of n entries takes log4 n
// dependent round trips and the shorter search hides behind the longer one.  This kernel's
// time is its longest chain of dependent loads.
template <typename KeyA, typename KeyB>
__device__ __forceinline__ void lane_lower_bound_pair(KeyA key_a, u32 lo_a, u32 hi_a, u64 target_a, KeyB key_b,
                                                      u32 lo_b, u32 hi_b, u64 target_b, u32& res_a, u32& res_b) {
  while (lo_a < hi_a || lo_b < hi_b) {
    const u32 na = hi_a - lo_a, nb = hi_b - lo_b;
    // probe positions (ascending; equal ones for ranges below four entries are harmless)
    const u32 a1 = lo_a + na / 4, a2 = lo_a + na / 2, a3 = lo_a + na / 2 + na / 4;
    const u32 b1 = lo_b + nb / 4, b2 = lo_b + nb / 2, b3 = lo_b + nb / 2 + nb / 4;
    u64 ka1 = 0, ka2 = 0, ka3 = 0, kb1 = 0, kb2 = 0, kb3 = 0;
    if (na) {
      ka1 = key_a(a1);
      ka2 = key_a(a2);
      ka3 = key_a(a3);
    }
    if (nb) {
      kb1 = key_b(b1);
      kb2 = key_b(b2);
      kb3 = key_b(b3);
    }
    if (na) {
      if (ka3 < target_a) lo_a = a3 + 1;
      else if (ka2 < target_a) { lo_a = a2 + 1; hi_a = a3; }
      else if (ka1 < target_a) { lo_a = a1 + 1; hi_a = a2; }
      else hi_a = a1;
    }
    if (nb) {
      if (kb3 < target_b) lo_b = b3 + 1;
      else if (kb2 < target_b) { lo_b = b2 + 1; hi_b = b3; }
      else if (kb1 < target_b) { lo_b = b1 + 1; hi_b = b2; }
      else hi_b = b1;
    }
  }
  res_a = lo_a;
  res_b = lo_b;
}

// Lower bound by K neighbouring lanes together (a power of two; each K of a wave search for their own
// target, all lanes of the wave call): K probes a step, so that a list of n entries takes log K n
// round trips, where one lane alone takes log2 n.  For launches whose searches leave most of the
// chip's lanes idle.
template <u32 K, typename KeyFn>
__device__ __forceinline__ u32 group_lower_bound(KeyFn key, u32 lo, u32 hi, u64 target) {
  static_assert(K >= 2 && K < 64 && (K & (K - 1)) == 0, "lanes of one search");
  const u32 l = lane_id(), i = l & (K - 1);
  if (hi < lo) hi = lo;  // (offsets that decrease)
  while (ballot(lo < hi)) {
    const u32 n = hi - lo, stride = (n + K - 1) / K, at = lo + (i + 1) * stride - 1;
    const u64 k = n && at < hi ? key(at) : ~0ull;  // past the end: never below
    const u32 below = __popcll(ballot(k < target) >> (l & ~(K - 1)) & ((1ull << K) - 1));  // a prefix
    const u32 nlo = min(lo + below * stride, hi);
    hi = n ? nlo + min(stride - 1, hi - nlo) : hi;
    lo = n ? nlo : lo;
  }
  return lo;
}

// The per-graph prefix sums as the tile, patch and dims blocks read them: from the workspace
// (written by mat_prep_graphs_kernel) or from the block's own LDS copy.
template <bool kOwn>
struct PrepView {
  const u64* out_word_off;  // [G+1]
  const u64* out_node_off;  // [G+1]
  const typename std::conditional<kOwn, u32, u64>::type* tile_off;  // [G+1]
  const u32* src;           // [G] source graphs, own sums only
  u32 n_tiles;              // 0 if the totals do not match
  u32 ok;
};

// Where tile j (j < n_tiles) lies: its graph, template, source graph, first word inside the
// graph, word count, first source word, and whether it is the graph's last tile.
struct TileGeom {
  u32 g, t, s, n;
  u64 k0, src_word;
  bool last;
};
template <bool kOwn>
__device__ __forceinline__ TileGeom tile_geometry(const MatParams& p, const PrepView<kOwn>& v, u32 j) {
  const fdy_mat_desc& d = p.d;
  TileGeom q;
  // largest g with tile_off[g] <= j
  q.g = lane_lower_bound([&](u32 i) { return (u64)v.tile_off[i]; }, 0u, d.n_graphs + 1u, (u64)j + 1) - 1;
  q.t = d.graph_tmpl[q.g];
  if constexpr (kOwn) q.s = v.src[q.g];
  else q.s = d.tmpl_graph[q.t];  // valid: graphs with a bad template have no tiles
  const u64 w0 = d.src_word_off[q.s];
  const u64 nw = d.src_word_off[q.s + 1] - w0;
  q.k0 = ((u64)j - v.tile_off[q.g]) * kMatTile;
  q.n = tile_words(nw - q.k0);
  q.src_word = w0 + q.k0;
  q.last = q.k0 + q.n == nw;
  return q;
}

// A block of 256 threads resolves kPrepTiles = 255 consecutive output tiles (independent of the
// base map).  Every thread finds where its tile's slices of the template's relocation list
// and of the graph's override list BEGIN; where they end is where the next tile's begin (the
// next thread's result, through LDS) or, for a graph's last tile, the end of the list.  That
// halves the chain of dependent loads, which is all this kernel's time.  Thread 255 only
// supplies the begins of the tile after the block's last.  Both ends stay bounded by the tile
// size, so a malformed list can never index outside what mat_main_kernel reserves; entries
// that do not belong to the tile are caught there.
constexpr u32 kPrepTiles = 255;
template <bool kOwn>
__device__ __forceinline__ void prep_tiles_block(const MatParams& p, const PrepView<kOwn>& v, u32 block, uint2* s_lo) {
  const fdy_mat_desc& d = p.d;
  const u32 tid = threadIdx.x;
  const u32 j = block * kPrepTiles + tid;
  const bool valid = j < v.n_tiles;
  TileGeom q;
  u32 rl0 = 0, rl1 = 0, ov1 = 0, reloc_lo = 0, ovr_lo = 0;
  if (valid) {
    q = tile_geometry(p, v, j);
    const fdy_reloc* relocs = d.relocs;
    rl0 = (u32)d.src_reloc_off[q.s];
    rl1 = (u32)d.src_reloc_off[q.s + 1];
    const fdy_ovr32* ovr = d.ovr;
    const u32 ov0 = (u32)d.ovr_off[q.g];
    ov1 = (u32)d.ovr_off[q.g + 1];
    lane_lower_bound_pair([&](u32 i) { return (u64)relocs[i].word; }, rl0, rl1, q.src_word,
                          [&](u32 i) { return (u64)ovr[i].byte_off; }, ov0, ov1, q.k0 * 8, reloc_lo, ovr_lo);
  }
  s_lo[tid] = make_uint2(reloc_lo, ovr_lo);
  __syncthreads();
  if (tid >= kPrepTiles || j >= p.ws.n_entries) return;
  MatTile* ent = &p.ws.tiles[j];
  if (!valid) {
    ent->n_words = 0;
    return;
  }
  // a tile that is not its graph's last is followed by a tile of the same graph (j + 1 < n_tiles)
  u32 reloc_hi = q.last ? rl1 : s_lo[tid + 1].x;
  const u32 ovr_hi = q.last ? ov1 : s_lo[tid + 1].y;
  if (rl1 < rl0) {  // offsets that decrease: no list
    reloc_hi = reloc_lo;
    raise_status(p.d_status, FDY_ST_BAD_ORDER);
  }
  // the list is strictly ascending by word: at most n entries fall inside the tile, and none
  // lies before the template's first word
  if (reloc_hi - reloc_lo > q.n) {
    reloc_hi = reloc_lo + q.n;
    raise_status(p.d_status, FDY_ST_BAD_ORDER);
  }
  if (q.k0 == 0 && reloc_lo != rl0) raise_status(p.d_status, FDY_ST_BAD_INDEX);
  MatTile e;
  e.src_word = q.src_word;
  e.out_word = v.out_word_off[q.g] + q.k0;
  e.n_words = q.n;
  e.k0 = (u32)q.k0;
  e.reloc_lo = reloc_lo;
  e.reloc_hi = reloc_hi;
  e.ovr_lo = ovr_lo;
  e.ovr_hi = ovr_hi;
  e.reloc_seg = rl0;
  e.pad = 0;
  *ent = e;
}

// The same with half a wave per tile, eight lanes for each of its four ends: what the kernel takes is
// its longest chain of dependent loads, and 13,400 relocations and 1,880 patches are five and six
// steps, not seven and 22.  For up to kGroupTiles tiles: each workgroup that this takes repeats the
// per-graph sums, and beside as many that write dimensions they come to cost what the steps save.  us
// of the launch, a thread per tile / half a wave: 1,870 tiles and 8 ranks 12.9 / 10.1, 446 tiles 8.5 / 7.6; 3,391
// tiles of 512 graphs with 295,000 dimensions 13.7 / 15.6; without dimensions 8 to 512 graphs gain 2 to 3 everywhere
// from 1,100 to 3,400 tiles (9.4 to 10.7 / 6.2 to 8.4) and nothing from 4,100 on.
constexpr u32 kGroupTiles = 2048;
template <bool kOwn>
__device__ __forceinline__ void prep_tile_group(const MatParams& p, const PrepView<kOwn>& v, u32 j) {
  const fdy_mat_desc& d = p.d;
  const u32 l = lane_id() & 31;
  if (v.n_tiles == 0) {  // (the same for all; no tile has a place)
    if (l == 0 && j < p.ws.n_entries) p.ws.tiles[j].n_words = 0;
    return;
  }
  const bool valid = j < v.n_tiles;
  const TileGeom q = tile_geometry(p, v, valid ? j : 0);
  const u32 rl0 = (u32)d.src_reloc_off[q.s], rl1 = (u32)d.src_reloc_off[q.s + 1];
  const u32 ov0 = (u32)d.ovr_off[q.g], ov1 = (u32)d.ovr_off[q.g + 1];
  // lanes 0..15: the relocation list, its entries from the tile's first word on, and from behind its
  // last; lanes 16..31: the overrides
  const bool of_ovr = l & 16, end = l & 8;
  const fdy_reloc* relocs = d.relocs;
  const fdy_ovr32* ovr = d.ovr;
  const u64 target = of_ovr ? (q.k0 + (end ? q.n : 0u)) * 8 : q.src_word + (end ? q.n : 0u);
  const u32 lo = of_ovr ? ov0 : rl0, hi = of_ovr ? ov1 : rl1;
  const u32 found = group_lower_bound<8>([&](u32 i) { return of_ovr ? (u64)ovr[i].byte_off : (u64)relocs[i].word; },
                                          !valid || (q.last && end) ? hi : lo, hi, target);
  MatTile e;
  e.src_word = q.src_word;
  e.out_word = v.out_word_off[q.g] + q.k0;
  e.n_words = q.n;
  e.k0 = (u32)q.k0;
  const u32 at = lane_id() & 32;
  e.reloc_lo = __shfl(found, at);
  e.reloc_hi = max((u32)__shfl(found, at + 8), e.reloc_lo);  // (a list out of order can cross them)
  e.ovr_lo = __shfl(found, at + 16);
  e.ovr_hi = max((u32)__shfl(found, at + 24), e.ovr_lo);
  e.reloc_seg = rl0;
  e.pad = 0;
  if (l != 0 || j >= p.ws.n_entries) return;
  MatTile* ent = &p.ws.tiles[j];
  if (!valid) {
    ent->n_words = 0;
    return;
  }
  if (e.reloc_hi - e.reloc_lo > q.n) {  // strictly ascending: at most one entry per word
    e.reloc_hi = e.reloc_lo + q.n;
    raise_status(p.d_status, FDY_ST_BAD_ORDER);
  }
  if (rl1 < rl0) raise_status(p.d_status, FDY_ST_BAD_ORDER);  // offsets that decrease: no list
  if (q.k0 == 0 && e.reloc_lo != rl0) raise_status(p.d_status, FDY_ST_BAD_INDEX);
  *ent = e;
}

// A slice of a rank's patch list by eight lanes, four for either end: up to kGroupPairs pairs of
// tile and rank, beyond which the workgroups that this takes cost what the steps save.  us of the launch, a
// thread per slice / eight lanes, 8 templates with 20, 300 and 1,880 patches to a rank: 9,648 pairs 6.2 / 6.3,
// 7.9 / 6.2, 9.5 / 6.6; 32,096 pairs 6.9 / 7.3, 8.7 / 8.0, 10.3 / 9.2 (30 templates 7.0 / 7.1, 10.1 / 11.0,
// 21.1 / 23.1); 38,592 pairs 6.7 / 7.2, 8.6 / 9.0, 12.5 / 14.9; 64,192 pairs 7.0 / 10.2, 9.0 / 12.8, 13.7 / 21.0.
constexpr u32 kGroupPairs = 32768;
template <bool kOwn>
__device__ __forceinline__ void prep_patch_group(const MatParams& p, const PrepView<kOwn>& v, u32 i) {
  const fdy_mat_desc& d = p.d;
  const u32 R = d.n_ranks;
  const bool valid = i < v.n_tiles * R;  // (at most kGroupPairs)
  const fdy_patch* patch = d.patch;
  u32 p0 = 0, p1 = 0;
  u64 target = 0;
  if (valid) {
    const TileGeom e = tile_geometry(p, v, i / R);
    const u64 row = (u64)e.t * R + i % R;
    p0 = (u32)d.patch_off[row];
    p1 = (u32)d.patch_off[row + 1];
    target = e.k0 + ((lane_id() & 4) ? e.n : 0u);
  }
  const u32 found = group_lower_bound<4>([&](u32 q) { return (u64)patch[q].word; }, p0, p1, target);
  const u32 lo = __shfl(found, lane_id() & ~7u), hi = __shfl(found, lane_id() | 4u);
  if (valid && (lane_id() & 7) == 0) p.ws.tile_patch[i] = make_uint2(lo, max(lo, hi));
}

// Thread i: (output tile, rank) pair i: the slice of the rank's patch list inside the tile.
// Works from the tile's geometry, not from the tile table, which the same launch is writing.
template <bool kOwn>
__device__ __forceinline__ void prep_patch(const MatParams& p, const PrepView<kOwn>& v, u64 i) {
  const fdy_mat_desc& d = p.d;
  const u32 R = d.n_ranks;
  if (i >= (u64)v.n_tiles * R) return;
  const u32 j = (u32)(i / R), r = (u32)(i % R);
  const TileGeom e = tile_geometry(p, v, j);
  const fdy_patch* patch = d.patch;
  const u64 row = (u64)e.t * R + r;
  const u32 p0 = (u32)d.patch_off[row], p1 = (u32)d.patch_off[row + 1];
  const u32 lo = lane_lower_bound([&](u32 q) { return (u64)patch[q].word; }, p0, p1, e.k0);
  const u32 hi = lane_lower_bound([&](u32 q) { return (u64)patch[q].word; }, lo, p1, e.k0 + e.n);
  p.ws.tile_patch[i] = make_uint2(lo, hi);
}

// The template tile on its way to LDS: 16-byte loads from the first even word on.
constexpr int kTileChunks = kMatBuf / (2 * kMatBlock);
struct TileRegs {
  v4u32 v[kTileChunks];
  u64 first, last;
};
template <int kPolicy>
__device__ __forceinline__ void tile_load(TileRegs& r, const u64* src, u64 src_word, u32 n, u32 tid) {
  const u32 head = (u32)(src_word & 1);  // words before 16-byte alignment (n >= 1 here)
  const __amdgpu_buffer_rsrc_t from = buffer(src + head, (n - head) >> 1 << 4);
#pragma unroll
  for (int c = 0; c < kTileChunks; ++c)
    r.v[c] = __builtin_amdgcn_raw_buffer_load_b128(from, (tid + (u32)c * kMatBlock) * 16, 0, kPolicy);
  r.first = src[0];
  r.last = src[n - 1];
}
__device__ __forceinline__ void tile_store(u64* buf, const TileRegs& r, u64 src_word, u32 n, u32 tid) {
  const u32 head = (u32)(src_word & 1);
  const u32 pairs = (n - head) >> 1;
#pragma unroll
  for (int c = 0; c < kTileChunks; ++c) {
    const u32 i = tid + (u32)c * kMatBlock;
    if (i < pairs) {
      buf[head + 2 * i] = pair64(r.v[c].x, r.v[c].y);
      buf[head + 2 * i + 1] = pair64(r.v[c].z, r.v[c].w);
    }
  }
  if (tid == 0) {  // what lies outside the pairs, or the same again
    buf[0] = r.first;
    buf[n - 1] = r.last;
  }
}

// Order of the short lists (overrides, grid overrides, rank patches): every entry against the
// one before it, all lists of a kind in one sweep over their concatenation; where the key does
// not ascend, a new list must begin.  The relocation lists, which are long, are checked where
// they are read anyway (mat_main_kernel).
// The three kinds go side by side: ends of the concatenations, then every kind's offsets (to s_at, as far as they fit) and
// the thread's first pair of keys, then whatever further pairs there are.  (One kind after the other, and the lists that
// begin searched among offsets in memory, these blocks were the last of a prep launch to end: 512 graphs with 72 overrides
// and 72 grids each 11.6 of 11.6 us.  us of whole loads, before / now: these 61.0 / 60.0, 67 graphs for 8 ranks 87.8 / 87.0.)
constexpr u32 kCheckOffsets = 2048;  // u32 of LDS
__device__ __forceinline__ void check_lists(const MatParams& p, u32 cb, u32 n_cb, u32* s_at) {
  const fdy_mat_desc& d = p.d;
  const u32 tid = threadIdx.x;
  const u64 first = (u64)cb * 256 + tid, stride = (u64)n_cb * 256;
  constexpr int kKinds = 3;
  const u64* off[kKinds] = {d.ovr_off, p.out_dims ? d.govr_off : nullptr, d.map_rank ? d.patch_off : nullptr};
  const u64 n_rows = (u64)d.n_templates * d.n_ranks;
  const u64 lists[kKinds] = {d.n_graphs, p.out_dims ? d.n_graphs : 0u, d.map_rank ? n_rows : 0u};
  auto key = [&](int kind, u64 i) {
    return kind == 0 ? d.ovr[i].byte_off : kind == 1 ? d.govr[i].node : d.patch[i].word;
  };
  u64 lo[kKinds], hi[kKinds];
#pragma unroll
  for (int k = 0; k < kKinds; ++k) {
    lo[k] = hi[k] = 0;
    if (lists[k]) {
      lo[k] = off[k][0];
      hi[k] = off[k][lists[k]];
    }
  }
  u32 k0[kKinds], k1[kKinds];
#pragma unroll
  for (int k = 0; k < kKinds; ++k) {
    const u64 i = lo[k] + 1 + first;
    k0[k] = 0;
    k1[k] = 1;
    if (i < hi[k]) {
      k0[k] = key(k, i - 1);
      k1[k] = key(k, i);
    }
  }
  u32 at[kKinds + 1] = {0, 0, 0, 0};  // where a kind's offsets lie in s_at (empty: they do not fit)
#pragma unroll
  for (int k = 0; k < kKinds; ++k) {
    const bool fits = lists[k] <= kCheckOffsets - at[k] && hi[k] >> 32 == 0;
    at[k + 1] = at[k] + (fits ? (u32)lists[k] : 0u);
    for (u32 l = tid; l < at[k + 1] - at[k]; l += 256) s_at[at[k] + l] = (u32)min(off[k][l], (u64)0xffffffffu);
  }
  __syncthreads();
  bool disorder = false;
#pragma unroll
  for (int k = 0; k < kKinds; ++k) {
    const bool staged = at[k + 1] != at[k];
    u32 before = k0[k], here = k1[k];
    for (u64 i = lo[k] + 1 + first; i < hi[k];) {
      if (before >= here) {
        u64 a = 0, b = lists[k], found;  // the last list that begins at or before entry i
        while (b - a > 1) {
          const u64 mid = a + (b - a) / 2;
          if ((staged ? (u64)s_at[at[k] + mid] : off[k][mid]) <= i) a = mid;
          else b = mid;
        }
        found = staged ? (u64)s_at[at[k] + a] : off[k][a];
        if (found != i) disorder = true;
      }
      i += stride;
      if (i < hi[k]) {
        before = key(k, i - 1);
        here = key(k, i);
      }
    }
  }
  if (disorder) raise_status(p.d_status, FDY_ST_BAD_ORDER);
}

// Thread i: launch dimensions of output node i.  What it takes is its chain of dependent loads
// (with own sums: source node offset, node, and the search among the graph's grid overrides).
// The lanes of a wave search for neighbouring nodes, so eight-way steps touch the same lines and
// cost one request each: 72 overrides are three steps, not seven.
template <bool kOwn>
__device__ __forceinline__ void write_dims(const MatParams& p, const PrepView<kOwn>& v, u64 i) {
  const fdy_mat_desc& d = p.d;
  if (!v.ok) return;
  if (i >= d.out_nodes_total) return;
  // largest g with out_node_off[g] <= i
  const u64* off = v.out_node_off;
  u32 lo = 0, hi = d.n_graphs;  // answer in [lo, hi)
  while (hi - lo > 1) {
    const u32 mid = lo + (hi - lo) / 2;
    if (off[mid] <= i) lo = mid;
    else hi = mid;
  }
  const u32 g = lo;
  const u32 n = (u32)(i - off[g]);
  u32 s;
  if constexpr (kOwn) s = v.src[g];
  else s = d.tmpl_graph[d.graph_tmpl[g]];
  const fdy_node nd = d.src_nodes[d.src_node_off[s] + n];
  u32 gx = nd.grid[0], gy = nd.grid[1], gz = nd.grid[2];
  // grid override of this node, if any (list ascending by node): the last entry not above it
  const u64 a0 = d.govr_off[g], a1 = d.govr_off[g + 1];
  u64 a = a0, b = a1;  // entries before a lie below n, those from b on do not
  while (a < b) {
    u64 at[7];
    u32 key[7];
#pragma unroll
    for (u32 k = 0; k < 7; ++k) {
      at[k] = a + (((b - a) * (k + 1)) >> 3);
      key[k] = d.govr[at[k]].node;
    }
    u64 na = a, nb = b;
#pragma unroll
    for (u32 k = 0; k < 7; ++k)
      if (key[k] < n) na = at[k] + 1;
#pragma unroll
    for (int k = 6; k >= 0; --k)
      if (key[k] >= n) nb = at[k];
    a = na;
    b = nb > na ? nb : na;  // (a list out of order can cross them)
  }
  if (a < a1) {
    u32 node = d.govr[a].node, x = d.govr[a].grid[0], y = d.govr[a].grid[1], z = d.govr[a].grid[2];
    asm volatile("" : "+v"(node), "+v"(x), "+v"(y), "+v"(z));  // (one round trip, not the grid's behind the node's)
    if (node == n) {
      gx = x;
      gy = y;
      gz = z;
    }
  }
  uint2* o = reinterpret_cast<uint2*>(p.out_dims + i * 6);
  o[0] = make_uint2(gx, gy);
  o[1] = make_uint2(gz, nd.block[0]);
  o[2] = make_uint2(nd.block[1], nd.block[2]);
}

// One workgroup per (tile, group of consecutive base maps).  What does not depend on the map
// is fetched once per workgroup: the tile entry, the template tile (LDS) and this thread's
// share of the tile's relocation entries (registers; the slice holds at most kMatTile
// entries, kMatPre per thread).  Per map only the base-map gathers, the scatter into LDS
// and the store of the tile repeat.  Relocations and overrides hit the same words for every
// map, so the LDS copy needs no refresh between maps; rank patches differ per map, so the
// words the previous map's rank patched are given their template values back first.
constexpr int kMatPre = kMatBuf / kMatBlock;
constexpr int kMatStore = kMatBuf / (2 * kMatBlock);  // 16-byte chunks per thread
constexpr u32 kMatMostMaps = 64;                       // base maps of a workgroup: a lane each keeps their patch slices
constexpr int kMatOvrPre = 2;                          // overrides of the tile a thread keeps in registers

//
// kSelf (small launches: every workgroup resident at once, at most kSelfGraphs output graphs):
// no tile table exists; the workgroup works out its own tile first (per-graph prefix sums in
// LDS, then its slices of the lists, one cooperative search per wave), and further blocks of
// the same launch write the launch dimensions and check the order of the short lists.  That
// is mat_prep_tiles_kernel's work without its launch: the model-shaped archives are bound by
// launches, and an extra 4 us of prologue in workgroups that all run side by side is less than
// the 10 us the launch costs.
constexpr u32 kSelfGraphs = 1000;   // four graphs to a thread; their node offsets fit the tile buffer
constexpr u32 kSelfMaxGroup = 8;    // most base maps per workgroup in this mode
// Most groups of maps: the blocks for dimensions and list order stand idle in each group but the first, and a prep launch
// comes to cost less.  us of the call resolving its tiles / with a prep launch: 7 tiles to 128 maps (64 groups) 11.1 / 11.3,
// 160 11.8 / 11.7, 256 14.8 / 12.4; 8 to 128 11.7 / 11.9, 224 16.1 / 13.0; 5 to 400 17.1 / 12.5; 21 to 90 (45 groups) 12.9 / 13.7.
constexpr u32 kSelfGroups = 64;

// Per-graph sums of a kSelf block that writes dimensions, in the 16 KiB tile buffer: source graph u32[1024] |
// out_node_off u64[1024].
struct SelfSums {
  u32* src;
  u64* off;
  bool ok;  // the totals match what the caller sized the launch for
};
__device__ __forceinline__ SelfSums self_sums(const MatParams& p, u64* buf, u64* s_buf) {
  SelfSums r;
  r.src = reinterpret_cast<u32*>(buf);
  r.off = buf + 512;
  const u32 G = p.d.n_graphs, tid = threadIdx.x;
  constexpr u32 kPer = 1024 / kMatBlock;
  static_assert(kMatBlock == 256, "graphs_sizes");
  u64 nw[kPer], nn[kPer], tw = 0, tn = 0, tt = 0;
  u32 from[kPer];
  graphs_sizes<kPer>(p, nw, nn, from);
#pragma unroll
  for (u32 i = 0; i < kPer; ++i) {
    if (i * kMatBlock >= G) break;  // uniform
    const u32 g = i * kMatBlock + tid;
    u64 e[3] = {nw[i], nn[i], tiles_of(nw[i])}, sum[3];
    block_excl_scan3(e, sum, s_buf);
    if (g < G) {
      r.src[g] = from[i];
      r.off[g] = tn + e[1];
    }
    tw += sum[0];
    tn += sum[1];
    tt += sum[2];
  }
  if (tid == 0) r.off[G] = tn;
  r.ok = totals_ok(p, tw, tn, tt);
  __syncthreads();
  return r;
}

// Output tile j for a kSelf block that resolves it: the thread that has its graph in hand leaves it in LDS.  (With all
// graphs' sums in LDS, a search among them and the graph's offsets read behind it 1 us longer.)
struct SelfTile {
  u64 src_word, out_word;
  u32 n, k0, tmpl, last;
  GraphRow row;
};
__device__ __forceinline__ bool self_tile(const MatParams& p, u32 j, u64* s_buf, SelfTile* s_tile, bool reports) {
  const u32 G = p.d.n_graphs;
  constexpr u32 kPer = 1024 / kMatBlock;
  u64 nw[kPer], nn[kPer], tw = 0, tn = 0, tt = 0;
  u32 from[kPer], tmpl[kPer];
  GraphRow rows[kPer];
  const bool bad = graphs_sizes<kPer>(p, nw, nn, from, rows, tmpl);
#pragma unroll
  for (u32 i = 0; i < kPer; ++i) {
    if (i * kMatBlock >= G) break;  // uniform
    const u64 tiles = tiles_of(nw[i]);
    u64 e[3] = {nw[i], nn[i], tiles}, sum[3];
    block_excl_scan3(e, sum, s_buf);
    const u64 k = j - (tt + e[2]);  // (wraps where the graph begins behind tile j)
    if (k < tiles) {
      const u64 k0 = k * kMatTile, left = nw[i] - k0;
      SelfTile q;
      q.src_word = rows[i].src_word + k0;
      q.out_word = tw + e[0] + k0;
      q.n = tile_words(left);
      q.k0 = (u32)k0;
      q.tmpl = tmpl[i];
      q.last = left <= (u64)kMatBuf;
      q.row = rows[i];
      *s_tile = q;
    }
    tw += sum[0];
    tn += sum[1];
    tt += sum[2];
  }
  const bool ok = totals_ok(p, tw, tn, tt);
  if (reports) {  // what the prep launch reports
    if (bad) raise_status(p.d_status, FDY_ST_BAD_INDEX);
    if (threadIdx.x == 0 && !ok) raise_status(p.d_status, FDY_ST_BAD_SIZE);
  }
  __syncthreads();
  return ok && j < tt;
}

template <bool kSelf>
__global__ __launch_bounds__(kMatBlock) void mat_main_kernel(MatParams p, u32 first_tile, u32 n_tile_blocks, u32 nb_dims) {
  __shared__ __align__(16) u64 buf[kMatBuf];
  __shared__ u64 s_buf[kSelf ? 17 : 1];
  __shared__ u32 s_found[kSelf ? 4 + 2 * kSelfMaxGroup : 1];
  __shared__ typename std::conditional<kSelf, SelfTile, char>::type s_tile;
  const fdy_mat_desc& d = p.d;
  const u32 j = first_tile + blockIdx.x, tid = threadIdx.x;
  const u32 m0 = blockIdx.y * p.map_group;
  const u32 m1 = min(m0 + p.map_group, d.n_maps);
  // Template words and relocation entries that no other map group reads again, in an archive
  // too large to stay in the L2s anyway (the host decides: one map group, and from 4,096 tiles
  // = 64 MiB on, twice the chip's L2s), are loaded non-temporally, so that the base map keeps
  // its place in L2 for the gathers (config 4: 0.51 -> 0.47 ms); small archives stay cached for
  // whoever reads them next.
  const bool once = p.stream_once != 0;
  MatTile ent;
  TileRegs tile;
  if constexpr (kSelf) {
    if (j >= n_tile_blocks) {  // launch dimensions, then the order of the short lists
      if (blockIdx.y) return;
      if (j < n_tile_blocks + nb_dims) {
        const SelfSums q = self_sums(p, buf, s_buf);
        PrepView<true> v;
        v.src = q.src;
        v.out_word_off = nullptr;
        v.out_node_off = q.off;
        v.tile_off = nullptr;
        v.n_tiles = 0;
        v.ok = q.ok ? 1u : 0u;
        write_dims(p, v, (u64)(j - n_tile_blocks) * kMatBlock + tid);
      } else {
        check_lists(p, j - n_tile_blocks - nb_dims, gridDim.x - n_tile_blocks - nb_dims, reinterpret_cast<u32*>(buf));
      }
      return;
    }
    if (!self_tile(p, j, s_buf, &s_tile, j == 0 && blockIdx.y == 0)) return;
    const u32 k0 = uniform(s_tile.k0), n_here = uniform(s_tile.n), t = uniform(s_tile.tmpl);
    const u64 src_word = uniform(s_tile.src_word), out_word = uniform(s_tile.out_word);
    const bool last = uniform(s_tile.last);
    const u32 rl0 = uniform(s_tile.row.rl0), rl1 = uniform(s_tile.row.rl1);
    const u32 ov0 = uniform(s_tile.row.ov0), ov1 = uniform(s_tile.row.ov1);
    // in flight during the searches
    if (once) tile_load<kNonTemporal>(tile, d.src_words + src_word, src_word, n_here, tid);
    else tile_load<0>(tile, d.src_words + src_word, src_word, n_here, tid);
    {
      // one cooperative search per wave: where the tile's slices of the template's relocation
      // list and of the graph's override list begin and end; then the patch slices of the
      // group's maps, two searches each
      const u32 w = tid >> 6;
      const fdy_reloc* relocs = d.relocs;
      const fdy_ovr32* ovr = d.ovr;
      u32 r = 0;
      if (w == 0) r = wave_lower_bound([&](u32 i) { return (u64)relocs[i].word; }, rl0, rl1, src_word);
      if (w == 1) r = last ? rl1 : wave_lower_bound([&](u32 i) { return (u64)relocs[i].word; }, rl0, rl1, src_word + n_here);
      if (w == 2) r = wave_lower_bound([&](u32 i) { return (u64)ovr[i].byte_off; }, ov0, ov1, (u64)k0 * 8);
      if (w == 3) r = last ? ov1 : wave_lower_bound([&](u32 i) { return (u64)ovr[i].byte_off; }, ov0, ov1, ((u64)k0 + n_here) * 8);
      if (lane_id() == 0) s_found[w] = r;
      if (d.map_rank) {
        const fdy_patch* patch = d.patch;
        for (u32 e = w; e < 2 * (m1 - m0); e += kMatBlock / 64) {
          const u32 rank = d.map_rank[m0 + (e >> 1)];
          u32 f = (e & 1) ? 0u : 0xffffffffu;  // a bad rank: the slice that mat_main takes for "none, and flag it"
          if (rank < d.n_ranks) {
            const u64 row = (u64)t * d.n_ranks + rank;
            const u32 p0 = (u32)d.patch_off[row], p1 = (u32)d.patch_off[row + 1];
            f = wave_lower_bound([&](u32 i) { return (u64)patch[i].word; }, p0, p1, (u64)k0 + ((e & 1) ? n_here : 0u));
          }
          if (lane_id() == 0) s_found[4 + e] = f;
        }
      }
    }
    tile_store(buf, tile, src_word, n_here, tid);  // c1
    __syncthreads();
    ent.src_word = src_word;
    ent.out_word = out_word;
    ent.n_words = n_here;
    ent.k0 = k0;
    ent.reloc_lo = uniform(s_found[0]);
    ent.reloc_hi = uniform(s_found[1]);
    ent.ovr_lo = uniform(s_found[2]);
    ent.ovr_hi = uniform(s_found[3]);
    ent.reloc_seg = rl0;
    if (ent.reloc_hi < ent.reloc_lo) ent.reloc_hi = ent.reloc_lo;  // (a list out of order can cross them)
    if (ent.ovr_hi < ent.ovr_lo) ent.ovr_hi = ent.ovr_lo;
    if (ent.reloc_hi - ent.reloc_lo > n_here) {  // strictly ascending: at most one entry per word
      ent.reloc_hi = ent.reloc_lo + n_here;
      if (blockIdx.y == 0) raise_status(p.d_status, FDY_ST_BAD_ORDER);
    }
    if (rl1 < rl0 && blockIdx.y == 0) raise_status(p.d_status, FDY_ST_BAD_ORDER);  // offsets that decrease: no list
    if (k0 == 0 && ent.reloc_lo != rl0 && blockIdx.y == 0) raise_status(p.d_status, FDY_ST_BAD_INDEX);
  } else {
    ent = p.ws.tiles[j];
  }
  const u32 n = ent.n_words;
  if (n == 0) return;
  const u64* src = d.src_words + ent.src_word;
  const u32 lane = tid & 63;
  const u32 n_rel = ent.reloc_hi - ent.reloc_lo;  // (at most n, see where entries are made)
  const u32 n_ovr = ent.ovr_hi > ent.ovr_lo ? ent.ovr_hi - ent.ovr_lo : 0u;  // (a list out of order can cross them)
  const bool has_ovr = n_ovr != 0;
  const bool has_patch = d.map_rank != nullptr;
  bool bad = false, disorder = false;
  // Everything that depends on the tile's entry alone is requested before any of it is looked at, in buffer loads that
  // need no branches: with a loop that waits for each piece of the template, a wait per register of relocation
  // entries, one more for the word in front of it, and two for an override, a workgroup spent a dozen round trips in a
  // row here.  us of main among the kernels of a load, sixty passes warm, before this and the stores by whole lines / with both:
  // 512 graphs, 5.9 M words to one map 22.1 / 16.0; 67 graphs to 8 ranks 54.3 / 51.4, to 256 maps (of which most is the
  // fill's 245) 271 / 257; 67 graphs to one map, tiles resolved here, 9.9 / 8.8.
  v4u32 raw[kMatPre];
  auto request = [&](auto policy) __attribute__((always_inline)) {
    constexpr int kPolicy = decltype(policy)::value;
    if constexpr (!kSelf) tile_load<kPolicy>(tile, src, ent.src_word, n, tid);
    const __amdgpu_buffer_rsrc_t from = buffer(d.relocs + ent.reloc_lo, n_rel * 16);
#pragma unroll
    for (int i = 0; i < kMatPre; ++i)
      if ((u32)i * kMatBlock < n_rel)
        raw[i] = __builtin_amdgcn_raw_buffer_load_b128(from, (tid + (u32)i * kMatBlock) * 16, 0, kPolicy);
  };
  if (once) request(std::integral_constant<int, kNonTemporal>{});
  else request(std::integral_constant<int, 0>{});
  // lane i: the word in front of what this wave has of the slice in its registers i
  u32 in_front = 0;
  {
    const u32 q = ent.reloc_lo + lane * kMatBlock + (tid & ~63u);
    if (lane < (u32)kMatPre && q < ent.reloc_hi && q > ent.reloc_seg) in_front = d.relocs[q - 1].word;
  }
  // the tile's overrides (the same for every map), kMatOvrPre per thread; longer lists take the rest from memory
  v2u32 ov[kMatOvrPre];
  {
    const __amdgpu_buffer_rsrc_t from = buffer(d.ovr + ent.ovr_lo, min(n_ovr, (u32)(kMatOvrPre * kMatBlock)) * 8);
#pragma unroll
    for (int i = 0; i < kMatOvrPre; ++i)
      ov[i] = __builtin_amdgcn_raw_buffer_load_b64(from, (tid + (u32)i * kMatBlock) * 8, 0, 0);
  }
  // lane i: the slice of map (m0 + i)'s rank inside this tile; empty for a bad rank
  uint2 slices = make_uint2(0, 0);
  if (const u32 m = m0 + lane; has_patch && m < m1) {
    if constexpr (kSelf) {
      const u32 lo = s_found[4 + 2 * lane], hi = s_found[5 + 2 * lane];
      slices = make_uint2(lo, lo == 0xffffffffu ? 0u : max(hi, lo));
    } else {
      const u32 rk_m = d.map_rank[m];
      slices = rk_m < d.n_ranks ? p.ws.tile_patch[(u64)j * d.n_ranks + rk_m] : make_uint2(0xffffffffu, 0);
    }
  }
  auto patch_slice = [&](u32 m) __attribute__((always_inline)) {
    return make_uint2(__builtin_amdgcn_readlane(slices.x, m - m0), __builtin_amdgcn_readlane(slices.y, m - m0));
  };
  // this thread's patch entry of a slice (zero behind its end)
  auto patch_entry = [&](uint2 pr) __attribute__((always_inline)) {
    const u32 c = pr.x != 0xffffffffu ? min(pr.y - pr.x, (u32)kMatBlock) : 0u;
    return __builtin_amdgcn_raw_buffer_load_b128(buffer(d.patch + pr.x, c * 16), tid * 16, 0, 0);
  };
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (!kSelf) tile_store(buf, tile, ent.src_word, n, tid);  // c1
  u32 rk[kMatPre / 2], rr[kMatPre];  // words of the tile in 16 bits each (all ones: none); regions
  u64 ro[kMatPre];
#pragma unroll
  for (int i = 0; i < kMatPre; ++i) {
    if (i % 2 == 0) rk[i / 2] = 0xffffffffu;
    rr[i] = 0;
    ro[i] = 0;
    if ((u32)i * kMatBlock >= n_rel) continue;  // uniform
    const u32 q = ent.reloc_lo + tid + (u32)i * kMatBlock;
    const u32 word = raw[i].x, region = raw[i].y;
    const u64 k = (u64)word - ent.src_word;
    const bool mine = q < ent.reloc_hi;
    if (mine && k < n && region < d.n_alloc) {
      rk[i / 2] = i % 2 ? (rk[i / 2] & 0xffffu) | (u32)k << 16 : 0xffff0000u | (u32)k;
      rr[i] = region;
    } else if (mine) {
      bad = true;
    }
    ro[i] = pair64(raw[i].z, raw[i].w);
    // Strictly ascending by word: every entry of the slice against the one before it in the
    // template's list (the lower lane holds it; a wave's first lane has read it).  The slices of a
    // template's tiles cover its list, so a list that passes everywhere is in order, which is
    // what the slices themselves (found by binary search) rely on.
    u32 before = __shfl_up(word, 1);
    const u32 of_first = __builtin_amdgcn_readlane(in_front, i);
    if (lane == 0) before = of_first;
    if (mine && q > ent.reloc_seg && before >= word) disorder = true;
  }
  u32 ov_at[kMatOvrPre];
#pragma unroll
  for (int i = 0; i < kMatOvrPre; ++i) {
    const u64 b = (u64)ov[i].x - (u64)ent.k0 * 8;
    const bool mine = tid + (u32)i * kMatBlock < n_ovr, fits = (b >> 3) < n && (b & 3) == 0;
    ov_at[i] = mine && fits ? (u32)(b >> 2) : 0xffffffffu;
    if (mine && !fits) bad = true;
  }
  // The base-map gathers of a map (c2).
  auto gather = [&](u32 m, u64 (&base)[kMatPre]) __attribute__((always_inline)) {
    const u64* nb = d.n_alloc ? d.new_base + (u64)m * d.n_alloc : d.src_word_off;  // (no allocations: no entry is valid)
#pragma unroll
    for (int i = 0; i < kMatPre; ++i)
      if ((u32)i * kMatBlock < n_rel) base[i] = nb[rr[i]];
  };
  auto add_offsets = [&](u64 (&base)[kMatPre]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kMatPre; ++i)
      if ((u32)i * kMatBlock < n_rel) base[i] += ro[i];
  };
  u64 base[kMatPre];
#pragma unroll
  for (int i = 0; i < kMatPre; ++i) base[i] = 0;
  uint2 pr = make_uint2(0, 0);
  v4u32 pe = v4u32{0, 0, 0, 0};
  if (has_patch) {
    pr = patch_slice(m0);
    pe = patch_entry(pr);
  }
  gather(m0, base);
  add_offsets(base);
  __syncthreads();
  for (u32 m = m0; m < m1; ++m) {
    const bool more = m + 1 < m1;
    // c2: rebase
#pragma unroll
    for (int i = 0; i < kMatPre; ++i)
      if ((u32)i * kMatBlock < n_rel) {
        asm volatile("" : "+v"(rk[i / 2]));  // (neither address nor comparison is kept across maps)
        const u32 k = i % 2 ? rk[i / 2] >> 16 : rk[i / 2] & 0xffffu;
        if (k != 0xffffu) buf[k] = base[i];
      }
    // What the next map needs is requested here, ahead of this map's stores, and taken behind them: a wave's
    // memory operations are waited for in order, and a gather behind the stores would wait for all of them.
    if (more) gather(m + 1, base);
    // c3: 32-bit overrides
    if (has_ovr) {
      __syncthreads();
      u32* buf32 = reinterpret_cast<u32*>(buf);
#pragma unroll
      for (int i = 0; i < kMatOvrPre; ++i) {
        asm volatile("" : "+v"(ov_at[i]));
        if (ov_at[i] != 0xffffffffu) buf32[ov_at[i]] = ov[i].y;
      }
      for (u32 q = ent.ovr_lo + tid + kMatOvrPre * kMatBlock; q < ent.ovr_hi; q += kMatBlock) {
        const fdy_ovr32 o = d.ovr[q];
        const u64 b = (u64)o.byte_off - (u64)ent.k0 * 8;
        if ((b >> 3) < n && (b & 3) == 0) buf32[b >> 2] = o.value;
        else bad = true;
      }
    }
    // c4: rank patches; what the patched word held goes to a register for the way back (the template's value, or a
    // rebased or overridden one that the next map's c2 / c3 write again anyway)
    u32 undo_at = 0xffffffffu;
    u64 undo_val = 0;
    const u32 n_patch = pr.x != 0xffffffffu ? pr.y - pr.x : 0u;
    const bool long_slice = n_patch > (u32)kMatBlock;
    if (has_patch) {
      if (pr.x == 0xffffffffu) bad = true;
      __syncthreads();
      if (tid < n_patch) {
        const u64 k = (u64)pe.x - ent.k0;
        if (k < n) {
          undo_at = (u32)k;
          undo_val = buf[k];
          buf[k] = pair64(pe.z, pe.w);
        } else {
          bad = true;
        }
      }
      if (long_slice)
        for (u32 q = pr.x + tid + kMatBlock; q < pr.y; q += kMatBlock) {
          const u64x2 e = *reinterpret_cast<const u64x2*>(&d.patch[q]);
          const u64 k = (u64)(u32)e.x - ent.k0;
          if (k < n) buf[k] = e.y;
          else bad = true;
        }
    }
    __syncthreads();
    // stream the tile out: LDS -> registers, then 16-byte non-temporal stores (the output is
    // written once and not read again here; keeping it out of L2 leaves the templates, lists
    // and base maps there: with plain stores 256 maps take 407 us, not 287).  The barrier sits between the LDS reads and
    // the global stores so that the next map's scatter can start while the stores drain.
    u64* out = p.out_words + (u64)m * d.out_words_per_map + ent.out_word;
    const u32 behind = (u32)((uintptr_t)out >> 3) & (kLine - 1);  // words of the first line in front of the tile
    if (behind + n > (u32)kMatBuf) {  // (the same for all; seldom) what lies behind the fourth store
      const u32 k = kMatBuf - behind + tid;
      if (k < n) __builtin_nontemporal_store(buf[k], out + k);
    }
    u32 twice = 2 * tid;
    asm volatile("" : "+v"(twice));  // (what follows from it is not kept across maps)
    const u32 at = twice - behind;  // (wraps below the tile's first word)
    u64 v[2 * kMatStore];
#pragma unroll
    for (int c = 0; c < kMatStore; ++c) {
      const u32 i = at + (u32)c * 2 * kMatBlock, k = i < n - 1 ? i : 0u;
      v[2 * c] = buf[k];
      v[2 * c + 1] = buf[k + 1];
    }
    const uint2 pr_next = more && has_patch ? patch_slice(m + 1) : make_uint2(0, 0);
    if (more && has_patch) pe = patch_entry(pr_next);
    const u64 edge = buf[tid == 0 ? 0u : n - 1];  // thread 0: the tile's first word, thread 1: its last
    if (more) {
      __syncthreads();
      if (has_patch) {
        // the patched words get back what they held (the surplus of a long slice: the template's
        // value from memory); relocations and overrides that touch them are applied again
        if (undo_at != 0xffffffffu) buf[undo_at] = undo_val;
        if (long_slice)
          for (u32 q = pr.x + tid + kMatBlock; q < pr.y; q += kMatBlock) {
            const u64 k = (u64)d.patch[q].word - ent.k0;
            if (k < n) buf[k] = src[k];
          }
        __syncthreads();
      }
    }
    const u32 odd_end = (behind + n) & 1;
    const __amdgpu_buffer_rsrc_t pairs = buffer(out - behind, (behind + n - odd_end) * 8);
    const __amdgpu_buffer_rsrc_t words = buffer(out - behind, (behind + n) * 8);
#pragma unroll
    for (int c = 0; c < kMatStore; ++c) {
      const v4u32 o = v4u32{(u32)v[2 * c], (u32)(v[2 * c] >> 32), (u32)v[2 * c + 1], (u32)(v[2 * c + 1] >> 32)};
      const u32 to = c == 0 && twice < behind ? kNowhere : twice * 8 + (u32)c * (kMatBlock * 16);
      __builtin_amdgcn_raw_buffer_store_b128(o, pairs, to, 0, kNonTemporal);
    }
    if (tid < 64) {
      const u32 to = tid == 0 && (behind & 1) ? behind * 8 : tid == 1 && odd_end ? (behind + n - 1) * 8 : kNowhere;
      __builtin_amdgcn_raw_buffer_store_b64(v2u32{(u32)edge, (u32)(edge >> 32)}, words, to, 0, kNonTemporal);
    }
    if (more) {
      add_offsets(base);
      pr = pr_next;
      asm volatile("" : "+v"(pe));
    }
  }
  if (bad) raise_status(p.d_status, FDY_ST_BAD_INDEX);
  if (disorder) raise_status(p.d_status, FDY_ST_BAD_ORDER);
}

// Everything that only needs the per-graph prefix sums, in one launch (these are small and
// launch-bound: three launches cost three times one): blocks [0, nb_tiles) resolve tiles,
// the next nb_patch blocks the (tile, rank) patch slices, the rest write launch dimensions.
// kOwnSums (at most kOwnSumsMax output graphs): every block computes the prefix sums itself,
// in LDS, instead of reading what mat_prep_graphs_kernel left in the workspace; that launch
// is then not needed at all.  Block 0 reports what that kernel would have reported.
constexpr u32 kOwnSumsMax = 1024;
constexpr u32 kCheckBlocks = 96;
// group_tiles, group_patch: the tiles' and patch slices' ends by several lanes each.
template <bool kOwnSums>
__global__ __launch_bounds__(256, 8) void mat_prep_tiles_kernel(MatParams p, u32 nb_tiles, u32 nb_patch, bool group_tiles,
                                                                bool group_patch) {
  __shared__ uint2 s_lo[256];
  // word offsets for the blocks that resolve tiles, node offsets for those that write dimensions
  // (18 KiB of LDS in all: eight workgroups per compute unit)
  static_assert(kCheckOffsets * 4 <= (kOwnSumsMax + 1) * 8, "the lists' offsets");
  __shared__ u64 s_off[kOwnSumsMax + 1];
  if (blockIdx.x >= gridDim.x - kCheckBlocks) {  // the last blocks verify the order of the short lists
    check_lists(p, blockIdx.x - (gridDim.x - kCheckBlocks), kCheckBlocks, reinterpret_cast<u32*>(s_off));
    return;
  }
  __shared__ u32 s_tile[kOwnSums ? kOwnSumsMax + 1 : 1], s_src[kOwnSums ? kOwnSumsMax : 1];
  __shared__ u64 s_buf[17];
  PrepView<kOwnSums> v;
  if constexpr (kOwnSums) {
    const u32 G = p.d.n_graphs, tid = threadIdx.x;
    const bool nodes = blockIdx.x >= nb_tiles + nb_patch;
    constexpr u32 kPer = kOwnSumsMax / 256;
    u64 nw[kPer], nn[kPer], tw = 0, tn = 0, tt = 0;
    u32 from[kPer];
    const bool bad = graphs_sizes<kPer>(p, nw, nn, from);
#pragma unroll
    for (u32 i = 0; i < kPer; ++i) {
      if (i * 256 >= G) break;  // uniform
      const u32 g = i * 256 + tid;
      u64 e[3] = {nw[i], nn[i], tiles_of(nw[i])}, sum[3];
      block_excl_scan3(e, sum, s_buf);
      if (g < G) {
        s_off[g] = nodes ? tn + e[1] : tw + e[0];
        s_tile[g] = (u32)(tt + e[2]);
        s_src[g] = from[i];
      }
      tw += sum[0];
      tn += sum[1];
      tt += sum[2];
    }
    if (tid == 0) {
      s_off[G] = nodes ? tn : tw;
      s_tile[G] = (u32)tt;
    }
    __syncthreads();
    const bool ok = totals_ok(p, tw, tn, tt);
    v.out_word_off = v.out_node_off = s_off;
    v.tile_off = s_tile;
    v.src = s_src;
    v.n_tiles = ok ? (u32)tt : 0u;
    v.ok = ok ? 1u : 0u;
    if (blockIdx.x == 0) {
      if (bad) raise_status(p.d_status, FDY_ST_BAD_INDEX);
      if (tid == 0 && !ok) raise_status(p.d_status, FDY_ST_BAD_SIZE);
    }
  } else {
    v.out_word_off = p.ws.out_word_off;
    v.out_node_off = p.ws.out_node_off;
    v.tile_off = p.ws.tile_off;
    v.src = nullptr;
    v.n_tiles = p.ws.hdr->n_tiles;
    v.ok = p.ws.hdr->ok;
  }
  const u32 b = blockIdx.x;
  if (b < nb_tiles) {
    if (group_tiles) prep_tile_group(p, v, b * 8 + (threadIdx.x >> 5));
    else prep_tiles_block(p, v, b, s_lo);
  } else if (b < nb_tiles + nb_patch) {
    if (group_patch) prep_patch_group(p, v, (b - nb_tiles) * 32 + (threadIdx.x >> 3));
    else
      for (u64 i = (u64)(b - nb_tiles) * 256; i < (u64)v.n_tiles * p.d.n_ranks; i += (u64)nb_patch * 256)
        prep_patch(p, v, i + threadIdx.x);
  } else if (v.ok) {
    const u32 nb_dims = gridDim.x - kCheckBlocks - nb_tiles - nb_patch;
    for (u64 i = (u64)(b - nb_tiles - nb_patch) * 256; i < p.d.out_nodes_total; i += (u64)nb_dims * 256)
      write_dims(p, v, i + threadIdx.x);
  }
}

bool desc_ok(const fdy_mat_desc* d) {
  if (!d) return false;
  if (d->n_graphs > (1u << 20) || d->n_src_graphs > (1u << 20) || d->n_templates > (1u << 20))
    return false;
  if (d->n_maps > 65535u) return false;
  if (d->out_words_per_map >= (1ull << 40)) return false;
  return true;
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// The size that is asked for: that of tables for tiles of 2,048 words and 64-byte entries, as ever, so that a caller's
// sizes do not move, or what the tables take where that is more (248 ranks and more: up to 0.8 %, and an entry per rank).
size_t asked_bytes(const fdy_mat_desc* d) {
  const u64 tiles = (d->out_words_per_map + 2047) / 2048 + d->n_graphs;
  const size_t per_graph = align256(((size_t)d->n_graphs + 1) * 8);
  return align256(sizeof(MatHeader)) + 3 * per_graph + align256((size_t)tiles * 64) +
         align256((size_t)tiles * (d->map_rank ? d->n_ranks : 0) * sizeof(uint2));
}

// The tile table is last, and is rounded up to whole rounds of the eight XCDs where that takes no more (always up to 32
// ranks, from 40 tiles on): the entries beyond the tiles are marked unused like others in reserve, so that main, which a
// launch may want in whole rounds (see materialize_launch), has no bound to test.  With a test there main of the kernels
// of a load took 51.5 us for 67 graphs to 8 ranks, not 51.3.
size_t layout(const fdy_mat_desc* d, unsigned char* base, MatWs* ws) {
  const u64 max_tiles = (d->out_words_per_map + kMatTile - 1) / kMatTile + d->n_graphs;
  const u32 R = d->map_rank ? d->n_ranks : 0;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    unsigned char* p = base ? base + off : nullptr;
    off += align256(bytes);
    return p;
  };
  MatWs w;
  w.hdr = (MatHeader*)take(sizeof(MatHeader));
  w.out_word_off = (u64*)take(((size_t)d->n_graphs + 1) * 8);
  w.out_node_off = (u64*)take(((size_t)d->n_graphs + 1) * 8);
  w.tile_off = (u64*)take(((size_t)d->n_graphs + 1) * 8);
  w.tile_patch = (uint2*)take((size_t)max_tiles * R * sizeof(uint2));
  const u64 in_rounds = (max_tiles + 7) & ~7ull;
  const size_t asked = asked_bytes(d), least = off + align256((size_t)max_tiles * sizeof(MatTile));
  const size_t need = asked > least ? asked : least;
  const u64 n_entries = off + in_rounds * sizeof(MatTile) <= need ? in_rounds : max_tiles;
  w.tiles = (MatTile*)take((size_t)n_entries * sizeof(MatTile));
  w.max_tiles = (u32)max_tiles;
  w.n_entries = (u32)n_entries;
  if (ws) *ws = w;
  return need;
}

}  // namespace
}  // namespace fdy

using namespace fdy;

extern "C" size_t fdy_materialize_workspace_bytes(const fdy_mat_desc* h_desc) {
  if (!desc_ok(h_desc)) return 0;
  return layout(h_desc, nullptr, nullptr);
}

// Scratch of the entry point that allocates nothing (fdy_materialize_static): the tile table and
// the other per-call tables of a materialization, in device memory that belongs to the loaded
// library.  Each GPU holds its own copy at its own address, found once per device with
// hipGetSymbolAddress; host code uses that address, never the array's name.
// (The limit is on what is asked for; the tables themselves can take half as much again where thousands of ranks
// patch a graph of three tiles that would have been two of 2,048 words.)
constexpr size_t kStaticLimitBytes = 4u << 20, kStaticScratchBytes = 6u << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

static int materialize_launch(const fdy_mat_desc* h_desc, uint64_t* d_out_words, uint32_t* d_out_dims,
                              void* d_workspace, size_t workspace_bytes, uint32_t* d_status,
                              void* hip_stream);

extern "C" int fdy_materialize(const fdy_mat_desc* h_desc, uint64_t* d_out_words, uint32_t* d_out_dims,
                               void* d_workspace, size_t workspace_bytes, uint32_t* d_status,
                               void* hip_stream) {
  return materialize_launch(h_desc, d_out_words, d_out_dims, d_workspace, workspace_bytes, d_status, hip_stream);
}

extern "C" size_t fdy_materialize_static_limit(void) { return kStaticLimitBytes; }

extern "C" int fdy_materialize_static(const fdy_mat_desc* h_desc, uint64_t* d_out_words, uint32_t* d_out_dims,
                                      uint32_t* d_status, void* hip_stream) {
  if (!desc_ok(h_desc)) return FDY_ERR_INVALID_ARG;
  if (asked_bytes(h_desc) > kStaticLimitBytes) return FDY_ERR_WORKSPACE;  // beyond the fixed scratch
  constexpr int kMaxDevices = 64;
  static void* ptr_of_device[kMaxDevices] = {};
  static std::mutex mu;
  int dev = 0;
  FDY_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return FDY_ERR_INVALID_ARG;
  void* ptr = nullptr;
  {
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr_of_device[dev]) {  // first call on this device, which is current
      void* found = nullptr;
      FDY_HIP_TRY(hipGetSymbolAddress(&found, HIP_SYMBOL(scratch)));
      if (!found) return FDY_ERR_HIP;
      ptr_of_device[dev] = found;
    }
    ptr = ptr_of_device[dev];
  }
  return materialize_launch(h_desc, d_out_words, d_out_dims, ptr, kStaticScratchBytes, d_status, hip_stream);
}

static int materialize_launch(const fdy_mat_desc* h_desc, uint64_t* d_out_words, uint32_t* d_out_dims,
                              void* d_workspace, size_t workspace_bytes, uint32_t* d_status,
                              void* hip_stream) {
  if (!desc_ok(h_desc)) return FDY_ERR_INVALID_ARG;
  const fdy_mat_desc& d = *h_desc;
  if (d.n_graphs == 0 || d.n_maps == 0) return FDY_OK;
  if (!d.src_word_off || !d.src_reloc_off || !d.tmpl_graph || !d.graph_tmpl || !d.ovr_off ||
      !d.new_base)
    return FDY_ERR_INVALID_ARG;
  if (d.out_words_per_map && (!d_out_words || ((uintptr_t)d_out_words & 15) || !d.src_words ||
                              ((uintptr_t)d.src_words & 15)))
    return FDY_ERR_INVALID_ARG;
  if ((uintptr_t)d.relocs & 15 || (uintptr_t)d.patch & 15) return FDY_ERR_INVALID_ARG;
  if (d.map_rank && (d.n_ranks == 0 || !d.patch_off)) return FDY_ERR_INVALID_ARG;
  if (d_out_dims && (((uintptr_t)d_out_dims & 7) || !d.src_node_off || !d.govr_off ||
                     (d.out_nodes_total && !d.src_nodes)))
    return FDY_ERR_INVALID_ARG;
  MatParams p;
  p.d = d;
  if (!d.map_rank) p.d.n_ranks = 0;
  if (!d_out_dims) p.d.out_nodes_total = 0;
  const size_t need = layout(&d, nullptr, nullptr);
  if (!d_workspace || ((uintptr_t)d_workspace & 255) || workspace_bytes < need) return FDY_ERR_WORKSPACE;
  layout(&d, (unsigned char*)d_workspace, &p.ws);
  p.out_words = (u64*)d_out_words;
  p.out_dims = d_out_dims;
  p.d_status = d_status;
  p.map_group = 1;
  hipStream_t stream = (hipStream_t)hip_stream;
  (void)hipGetLastError();  // drop any stale error left by earlier, unrelated runtime calls

  // Base maps per workgroup: two.  A workgroup writes each of its maps in turn, and the further apart the maps that are
  // written at a time lie, the slower.  us of main with 1 / 2 / 3 / 4 / 8 maps, thirty passes warm: 67 graphs to 256 maps 342 / 257
  // / 285 / 298 / 306, 67 graphs to 8 ranks 57.5 / 51.1 / 50.8 / 52.3 / 56.4.  Four where the templates are more than the
  // Infinity Cache holds (16,384 tiles are 268 MB) and each group reads them from HBM: us of the call with two / four, 3 % of
  // the words relocated, 40 M words to 4 maps 388 / 351, 60 M to 3, 4, 8 489 / 404, 593 / 520, 1,182 / 1,018; 20 M 154 / 178.
  //
  // With rank patches, whose maps cost a workgroup three barriers each, a larger group is worth it where it lets the
  // launch resolve its own tiles, up to 4,608 tiles of all maps and sixteen maps: us of the call with two in two launches / more
  // in one, 449 tiles to 5, 6, 8 ranks 16.3 / 14.5 (four), 17.4 / 15.6 (four), 21.2 / 20.1 (four); 867 to 3, 4, 5 19.1 / 16.7,
  // 21.6 / 19.2 (four), 23.4 / 22.6 (eight), but to 8 30.3 / 31.8; 267 to 16 maps 22.0 / 20.7 (eight).  Beyond
  // sixteen maps only once groups of two are more workgroups than run at a time, and four at most: 24 tiles to 96 maps
  // 14.0 / 16.1, to 160 19.0 / 17.7, 7 to 512 18.4 / 19.9; 160 to 24 20.8 / 19.9, to 32 24.3 / 25.2 (six).  In two launches
  // four are better up to five maps (1,001 tiles to 3, 4, 5 ranks 20.4 / 19.3, 22.3 / 22.0, 26.6 / 24.7; 1,937 33.1 / 31.5,
  // 38.9 / 38.2, 44.5 / 43.6; to 8 60.6 / 61.5), where full groups of four all run at a time (667 to 8 26.3 / 25.5, 449 to
  // 12 maps 26.2 / 25.3; to 10 22.5 / 23.2), and where the templates are more than an L2 holds and come from afar for
  // each group (6 M words to 8, 16 ranks 116 / 98, 213 / 181, 12 M to 16 404 / 350, 200 graphs of 40 templates to 8, 16 114 /
  // 99, 212 / 177; of 10, 158 tiles, 90.4 / 92.5, 165 / 170; 2 M words to 8, 16 40.1 / 38.1, 66.0 / 67.6).
  const u64 self_limit = (u64)fdy__tune_get(FDY_TUNE_MAT_SELF_WGS);
  // (The line was placed with tiles of 2,048 words: 260,087 words, all relocated, to 16 maps, 129 tiles by eight groups,
  // 18.5 us in one launch, 25.7 in two; a quarter relocated 14.5 / 16.7.)
  const u64 distinct = (u64)p.ws.max_tiles * d.n_templates / d.n_graphs;  // tiles that the templates have
  const u64 line_tiles = (d.out_words_per_map + kMatBuf - 1) / kMatBuf + d.n_graphs;
  auto resolves_itself = [&](u32 group) {
    const u32 groups = (d.n_maps + group - 1) / group;
    return d.n_graphs <= kSelfGraphs && group <= kSelfMaxGroup && groups <= kSelfGroups && p.ws.max_tiles &&
           line_tiles * groups <= self_limit;
  };
  u32 mg = (u32)fdy__tune_get(FDY_TUNE_MAT_MAP_GROUP);
  if (mg == 0) {
    mg = distinct >= 16384 ? 4 : 2;
    if (d.map_rank && !resolves_itself(2)) {
      const u64 tiles = p.ws.max_tiles - d.n_graphs;  // at least (the entries in reserve aside)
      const bool few = d.n_maps <= 16, one_launch = (u64)p.ws.max_tiles * d.n_maps <= 4608;
      if (distinct >= 200 || d.n_maps <= 5 || (few && d.n_maps % 4 == 0 && tiles * (d.n_maps / 4) <= 1200)) mg = 4;
      if (one_launch && few && resolves_itself(8)) mg = 8;
      if (one_launch && (few || tiles * ((d.n_maps + 1) / 2) >= 1280) && resolves_itself(4)) mg = 4;
    }
  }
  if (mg > kMatMostMaps) mg = kMatMostMaps;
  p.map_group = mg < d.n_maps ? mg : d.n_maps;
  const u32 n_groups = (d.n_maps + p.map_group - 1) / p.map_group;
  // Where many maps are written, unused LDS keeps a compute unit to four workgroups instead of five: fewer places are
  // written at a time.  us of main with five / four, thirty passes warm: 772,000 words to 16 maps (8 groups) 21.0 / 21.3, 32
  // 37.7 / 36.2, 64 71.0 / 66.6, 128 137 / 129, 256 275 / 256; 5.9 M words to 8 maps 68.4 / 68.5, 32 282 / 260; 3.7 M words to
  // 32 maps 158 / 160, with rank patches, whose barriers need the fifth, 178 / 185.  (For some 60 passes after idle, while
  // the card's power settles, all are slower and five are the better: 256 maps 292 / 317.)  Not where five hold all workgroups at
  // a time and four do not: us of the call with five / four, 16 tiles to 124 maps (992 workgroups) 14.4 / 14.1, 128 (1,024, and
  // the entries in reserve) 14.4 / 16.2, 152 (1,216) 15.2 / 16.4; 6 tiles to 330 (990) 13.1 / 12.9, 340 (1,020) 13.4 / 14.9, 400
  // (1,200) 14.2 / 15.8; 72 tiles to 30 (1,080) 15.1 / 16.6, 36 (1,296) 17.6 / 17.1.
  const u64 n_wgs = (u64)(p.ws.max_tiles - d.n_graphs) * n_groups;  // at least (the entries in reserve aside)
  const bool four_per_cu = n_groups > 8 && !d.map_rank && (n_wgs <= 1000 || n_wgs > 1230);
  const size_t unused_lds = four_per_cu ? 160 * 1024 / 4 - kMatBuf * 8 - 512 : 0;
  p.stream_once = n_groups == 1 && p.ws.max_tiles >= (u32)fdy__tune_get(FDY_TUNE_MAT_ONCE_TILES) ? 1u : 0u;
  // A grid of 2^32 threads in one dimension and more is cut to its low 32 bits, and no error says so (16,778,216 blocks
  // of 256: 1,000 run).  Main goes out in several launches beyond this many tiles, 136 GB of output to a map; the prep
  // launch's blocks of patch slices and of launch dimensions take several rounds.
  const u32 most = (u32)fdy__tune_get(FDY_TUNE_MAT_MOST_BLOCKS);
  const u64 nb_dims_all = (d_out_dims && d.out_nodes_total) ? (d.out_nodes_total + 255) / 256 : 0;
  // Workgroups go to the eight XCDs in turn, one group of maps behind the other.  With a whole number of rounds to a group
  // a tile's groups share an XCD, whose L2 has its template and list then; else that depends on the number of tiles.  us
  // of the call, as they come / rounded up, graphs that are their own templates, tiles with those in reserve: a quarter of
  // the words relocated, to 64 maps 41 tiles 17.9 / 17.6, 81 26.7 / 25.2, 129 37.8 / 34.6, to 8 maps 395 23.4 / 19.7, 1,478
  // 59.5 / 55.2, 2,954 110.6 / 110.6; all relocated, to 64 maps 41 tiles 23.7 / 22.3, 81 40.6 / 32.6, to 16 maps 395 52.1 /
  // 38.3.  With tiles resolved here 113 to 16 maps 19.9 / 16.2, 81 11.2 / 11.1, but 65 10.3 / 10.9 and 25 9.1 / 11.0: rounds of
  // tiles and idle blocks come back to the same compute units.  Where graphs share templates, only beyond what
  // one L2 holds of them: 434 tiles of 16 templates of 40 graphs 19.7 / 19.5, of 4 19.6 / 19.75, 3,391 of 22 of 512 84.4 / 87.0.
  const u32 own_from = d.n_templates < d.n_graphs ? ~0u : resolves_itself(p.map_group) ? 80 : 40;
  const bool rounds = n_groups > 1 && (distinct >= 160 || p.ws.max_tiles >= own_from);
  // A launch small enough that all its workgroups run side by side resolves its tiles itself.
  if (resolves_itself(p.map_group) && p.ws.max_tiles <= most && nb_dims_all <= most / 2) {
    const u32 own_blocks = p.ws.max_tiles + (u32)nb_dims_all + kCheckBlocks;
    launch(FDY_PROF_MAT_MAIN, mat_main_kernel<true>,
           dim3(rounds ? (own_blocks + 7) & ~7u : own_blocks, n_groups), dim3(kMatBlock), 0, stream, p, 0u, p.ws.max_tiles,
           (u32)nb_dims_all);
    FDY_HIP_TRY(hipGetLastError());
    return FDY_OK;
  }

  if (!rounds) p.ws.n_entries = p.ws.max_tiles;
  const bool own_sums = d.n_graphs <= kOwnSumsMax;
  if (!own_sums) {
    launch(FDY_PROF_MAT_PREP_GRAPHS, mat_prep_graphs_kernel, dim3(1), dim3(1024), 0, stream, p);
    FDY_HIP_TRY(hipGetLastError());
  }
  const u64 pairs = (u64)p.ws.max_tiles * p.d.n_ranks;  // (0 ranks without a rank map)
  const u32 entries = p.ws.n_entries;
  const bool group_tiles = p.ws.max_tiles <= kGroupTiles, group_patch = pairs <= kGroupPairs;
  u32 nb_tiles = group_tiles ? (entries + 7) / 8 : (entries + kPrepTiles - 1) / kPrepTiles;
  const u64 nb_patch_all = group_patch ? (pairs + 31) / 32 : (pairs + 255) / 256;
  const u32 nb_patch = !group_patch && nb_patch_all > most ? most : (u32)nb_patch_all;
  const u32 nb_dims = nb_dims_all > most / 2 ? (most + 1) / 2 : (u32)nb_dims_all;
  if (own_sums && nb_tiles + nb_patch + nb_dims == 0) nb_tiles = 1;  // someone has to verify the totals
  if (nb_tiles + nb_patch + nb_dims) {
    const u32 nb = nb_tiles + nb_patch + nb_dims + kCheckBlocks;
    launch(FDY_PROF_MAT_PREP_TILES, own_sums ? mat_prep_tiles_kernel<true> : mat_prep_tiles_kernel<false>, dim3(nb),
           dim3(256), 0, stream, p, nb_tiles, nb_patch, group_tiles, group_patch);
    FDY_HIP_TRY(hipGetLastError());
  }
  for (u32 first = 0; first < entries;) {
    const u32 n = entries - first < most ? entries - first : most;
    launch(FDY_PROF_MAT_MAIN, mat_main_kernel<false>, dim3(n, n_groups), dim3(kMatBlock), unused_lds, stream, p, first,
           0u, 0u);
    FDY_HIP_TRY(hipGetLastError());
    first += n;
  }
  return FDY_OK;
}
