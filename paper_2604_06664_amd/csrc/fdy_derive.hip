// fdy_derive.hip - override derivation for gfx950: the SAVE side of templating.
//
// Section 4.2.1 / Section 5.3: graphs of one topology group "differ only in per-node
// parameters", so a non-template graph is stored as what differs from its template.  For
// graph g with template source graph s, every 32-bit half of g's argument words that is not
// equal to s's half at the same place becomes an fdy_ovr32 {byte offset, value}, ascending
// per graph, graphs in order: exactly the override lists fdy_materialize consumes.
//
//   tile  (tile of 2048 words) checks each graph against its template (index, word count) and
//                            prefix-sums the graphs' tile counts in LDS; compares its tile with
//                            the template's; leaves the tile's count and, if there are few, its
//                            entries in the workspace;
//   place (tile)             sums the counts of the tiles before it, moves the entries to their
//                            place (a tile with more than kDerSlot of them is compared again)
//                            and writes the offsets of the graphs that begin there.
// Archives of more than 1,024 graphs take the per-graph sums from a launch of one workgroup
// ahead (prep), those of more than kDerSelfTiles tiles the tiles' positions from one between
// (scan).  What bounds the call is launches and the dependent loads in front of each tile's
// words, not bytes: as prep, count, scan and write, each tile searching its graph in memory, the
// MoE archive (3.7 M words, 12,032 entries) took 31 us, 17 now.  Entries are few (a handful per
// tile), hence the slots: the archive is read once.  Ordering inside a tile comes from ballots
// over words in index order, low half before high half.
#include <type_traits>

#include "fdy_device.hpp"
#include "fdy_internal.h"

namespace fdy {
namespace {

constexpr int kDerTile = 2048;  // words per tile
constexpr int kDerBlock = 256;
constexpr int kDerRounds = kDerTile / kDerBlock;  // words per thread
// Entries of a tile that wait in the workspace (256 bytes per 16 KiB of words).  128 of them: 600
// graphs of 20,480 words with 31 differing halves in a tile 50 us instead of 57, equal with 4.
constexpr u32 kDerSlot = 32;
// Workgroups that compare, eight per compute unit: beyond, the sums are paid once each (6,600
// tiles: 39.8 us, one workgroup per tile 49.4).
constexpr u32 kDerGrid = 2048;
constexpr u32 kDerOwnGraphs = 1024;  // up to here every workgroup sums the graphs' tiles itself
// Up to here every workgroup sums the counts before its own (4 bytes each, from L2): half the
// square of them in all, 32 MiB at the limit.  us with the limit at 1,024 / 4,096 / 8,192: 2,000
// tiles 24.4 / 22.4 / 22.4, 6,600 with 31 entries each 57.1 / 56.7 / 58.2.
constexpr u32 kDerSelfTiles = 4096;

struct DerWs {
  u64* tile_off;   // [G+1] first tile of each graph
  u32* tile_cnt;   // [max_tiles]
  u32* tile_graph;  // [max_tiles]
  fdy_ovr32* slot;  // [max_tiles][kDerSlot] entries of tiles with few
  u64* tile_pos;   // [max_tiles] entries before the tile
  u32* n_tiles;    // tiles in use
  u32 max_tiles;
};

struct DerParams {
  const u64* words;
  const u64* word_off;
  u32 n_graphs;
  const u32* graph_tmpl;
  const u32* tmpl_graph;
  u32 n_templates;
  u64 n_words_total;
  fdy_ovr32* ovr;
  u64 capacity;
  u64* ovr_off;
  u32* d_status;
  DerWs ws;
};

// Words of graph g that take part: 0 for a graph that cannot be compared (status bits in flag).
struct DerGraph {
  u64 words;
  u32 src, flag;
};
__device__ __forceinline__ DerGraph comparable_words(const DerParams& p, u32 g) {
  DerGraph r{0, 0xffffffffu, 0};
  const u32 t = p.graph_tmpl[g];
  if (t < p.n_templates) r.src = p.tmpl_graph[t];
  if (r.src >= p.n_graphs) {
    r.flag = FDY_ST_BAD_INDEX;
    return r;
  }
  const u64 nw = p.word_off[g + 1] - p.word_off[g];
  if (p.word_off[r.src + 1] - p.word_off[r.src] != nw || (nw >> 29)) r.flag = FDY_ST_BAD_SIZE;  // byte offsets are 32-bit
  else r.words = nw;
  return r;
}

__global__ __launch_bounds__(1024) void derive_prep_kernel(DerParams p) {
  __shared__ u64 s_buf[17];
  const u32 G = p.n_graphs;
  u64 carry = 0;
  u32 flags = 0;
  for (u32 g0 = 0; g0 < G; g0 += 1024) {
    const u32 g = g0 + threadIdx.x;
    u64 nt = 0;
    if (g < G) {
      const DerGraph q = comparable_words(p, g);
      flags |= q.flag;
      nt = (q.words + kDerTile - 1) / kDerTile;
    }
    u64 total;
    const u64 e = block_excl_scan(nt, s_buf, total);
    if (g < G) p.ws.tile_off[g] = carry + e;
    carry += total;
  }
  if (flags) raise_status(p.d_status, flags);
  if (threadIdx.x == 0) {
    const bool ok = p.word_off[G] == p.n_words_total && carry <= p.ws.max_tiles;
    if (!ok) raise_status(p.d_status, FDY_ST_BAD_SIZE);
    p.ws.tile_off[G] = ok ? carry : 0;
    *p.ws.n_tiles = ok ? (u32)carry : 0u;
  }
}

// Where tile j lies.
struct DerTile {
  const u64 *a, *b;  // the graph's words and the template's
  u64 k0;
  u32 n;
};
__device__ __forceinline__ DerTile tile_at(const DerParams& p, u32 g, u32 s, u64 first_tile, u32 j) {
  DerTile t;
  const u64 a = uniform((u64)p.word_off[g]), b = uniform((u64)p.word_off[s]);
  const u64 nw = uniform((u64)p.word_off[g + 1]) - a;
  t.k0 = ((u64)j - uniform(first_tile)) * kDerTile;
  t.n = (u32)(nw - t.k0 < (u64)kDerTile ? nw - t.k0 : (u64)kDerTile);
  t.a = p.words + a + t.k0;
  t.b = p.words + b + t.k0;
  return t;
}

// Compares a tile and writes its entries, as far as `room` goes, to dst if there are at most
// `most`; returns their number (the same in every thread).  kKeep false, for tiles with few
// entries: only the differences stay in registers (64 per lane leave room for eight workgroups
// per compute unit, which cover the latency of each other's words) and the few words that
// differ are read again.  kKeep true: the words stay as well.  (Read again, 600 graphs of 20,480
// words with 400 differing halves in a tile took 76 us instead of 64.)
struct DerCounts {
  u32 n[kDerRounds][kDerBlock / 64];
};
template <bool kKeep>
__device__ __forceinline__ u32 compare_tile(const DerTile& t, DerCounts& s_cnt, fdy_ovr32* dst, u64 room, u32 most) {
  static_assert(kDerBlock == 256, "a round's counts are four");
  const u32 tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // All words are requested before one is looked at, in buffer loads without branches, as many rounds of them as a short
  // tile needs: us of the call, before / eight rounds always / now: 512 graphs of 11,520 words 23.6 / 22.2 / 22.2, 3.7 M words of 67
  // with scan and fingerprint 45.8 / 45.1 / 45.1; 5,000 graphs of 500 words 41.3 / 45.8 / 40.0, 900 of 700 13.0 / 14.0 / 13.3, of 1,500
  // 14.0 / 14.35 / 14.0; of 2,047 14.5 / 15.0 / 15.0.  Words in index order: round i covers words [256 i, 256 i + 256), one per thread
  u64 x[kDerRounds], va[kKeep ? kDerRounds : 1];
  v2u32 ra[kDerRounds], rb[kDerRounds];
  u32 at = tid * 8;
  asm volatile("" : "+v"(at));  // (the eight offsets are not kept from tile to tile)
  auto request = [&](auto rounds) __attribute__((always_inline)) {
    constexpr int kRounds = decltype(rounds)::value;
    const __amdgpu_buffer_rsrc_t from_a = buffer(t.a, t.n * 8), from_b = buffer(t.b, t.n * 8);
#pragma unroll
    for (int i = 0; i < kRounds; ++i) {
      ra[i] = __builtin_amdgcn_raw_buffer_load_b64(from_a, at + (u32)i * kDerBlock * 8, 0, 0);
      rb[i] = __builtin_amdgcn_raw_buffer_load_b64(from_b, at + (u32)i * kDerBlock * 8, 0, 0);
    }
#pragma unroll
    for (int i = kRounds; i < kDerRounds; ++i) ra[i] = rb[i] = v2u32{0, 0};
  };
  if (t.n <= 2 * kDerBlock) request(std::integral_constant<int, 2>{});
  else if (t.n <= 4 * kDerBlock) request(std::integral_constant<int, 4>{});
  else if (t.n <= 6 * kDerBlock) request(std::integral_constant<int, 6>{});
  else request(std::integral_constant<int, kDerRounds>{});
#pragma unroll
  for (int i = 0; i < kDerRounds; ++i) {
    const u64 a = pair64(ra[i].x, ra[i].y);
    x[i] = a ^ pair64(rb[i].x, rb[i].y);
    if constexpr (kKeep) va[i] = a;
  }
#pragma unroll
  for (int i = 0; i < kDerRounds; ++i) {
    const u32 c = __popcll(ballot((u32)x[i] != 0)) + __popcll(ballot((u32)(x[i] >> 32) != 0));
    if (lane == 0) s_cnt.n[i][wave] = c;
  }
  __syncthreads();
  u32 total = 0;
#pragma unroll
  for (int i = 0; i < kDerRounds; ++i) {
    const uint4 c = *reinterpret_cast<const uint4*>(s_cnt.n[i]);
    total += c.x + c.y + c.z + c.w;
  }
  if (total == 0 || total > most) return total;
  u32 before = 0;
#pragma unroll
  for (int i = 0; i < kDerRounds; ++i) {
    const uint4 c = *reinterpret_cast<const uint4*>(s_cnt.n[i]);
    const bool lo = (u32)x[i] != 0, hi = (u32)(x[i] >> 32) != 0;
    const u64 blo = ballot(lo), bhi = ballot(hi);
    if (lo || hi) {
      const u32 k = (u32)i * kDerBlock + tid, byte_off = (u32)((t.k0 + k) * 8);
      const u64 lt = lanemask_lt(), v = kKeep ? va[kKeep ? i : 0] : t.a[k];
      u32 to = before + __popcll(blo & lt) + __popcll(bhi & lt);
      to += (wave > 0 ? c.x : 0) + (wave > 1 ? c.y : 0) + (wave > 2 ? c.z : 0);
      if (lo) {
        if (to < room) dst[to] = fdy_ovr32{byte_off, (u32)v};
        ++to;
      }
      if (hi && to < room) dst[to] = fdy_ovr32{byte_off + 4, (u32)(v >> 32)};
    }
    before += c.x + c.y + c.z + c.w;
  }
  return total;
}

// kOwnSums: at most kDerOwnGraphs graphs; the per-graph sums are this workgroup's own, and the
// first one leaves them in the workspace and reports what they show.
template <bool kOwnSums>
__global__ __launch_bounds__(kDerBlock, 8) void derive_tile_kernel(DerParams p) {
  __shared__ __align__(16) DerCounts s_cnt;
  __shared__ u64 s_buf[17];
  __shared__ u32 s_first[kOwnSums ? kDerOwnGraphs + 1 : 1], s_src[kOwnSums ? kDerOwnGraphs : 1];
  const u32 tid = threadIdx.x, G = p.n_graphs;
  const bool reports = blockIdx.x == 0;
  u32 n_tiles;
  if constexpr (kOwnSums) {
    u32 flags = 0;
    u64 carry = 0;
    for (u32 q0 = 0; q0 < G; q0 += kDerBlock) {
      const u32 q = q0 + tid;
      u64 nt = 0, total;
      if (q < G) {
        const DerGraph d = comparable_words(p, q);
        flags |= d.flag;
        nt = (d.words + kDerTile - 1) / kDerTile;
        s_src[q] = d.src;
      }
      const u64 e = carry + block_excl_scan(nt, s_buf, total);
      if (q < G) {
        s_first[q] = (u32)e;
        if (reports) p.ws.tile_off[q] = e;
      }
      carry += total;
    }
    const bool ok = p.word_off[G] == p.n_words_total && carry <= p.ws.max_tiles;
    n_tiles = ok ? (u32)carry : 0u;
    if (reports) {
      if (flags) raise_status(p.d_status, flags);
      if (tid == 0) {
        if (!ok) raise_status(p.d_status, FDY_ST_BAD_SIZE);
        p.ws.tile_off[G] = n_tiles;
        *p.ws.n_tiles = n_tiles;
      }
    }
    __syncthreads();
  } else {
    n_tiles = *p.ws.n_tiles;
  }
  for (u32 j = blockIdx.x; j < n_tiles; j += gridDim.x) {
    // largest g whose first tile is not behind tile j
    u32 g = 0, hi = G;  // answer in [g, hi)
    while (hi - g > 1) {
      const u32 mid = g + (hi - g) / 2;
      if ((kOwnSums ? (u64)s_first[mid] : p.ws.tile_off[mid]) <= j) g = mid;
      else hi = mid;
    }
    u32 s;
    u64 first;
    if constexpr (kOwnSums) {
      first = s_first[g];
      s = s_src[g];
    } else {
      first = p.ws.tile_off[g];
      s = p.tmpl_graph[p.graph_tmpl[g]];  // valid: a graph that failed the checks has no tiles
    }
    u32 c = 0;
    if (s != g) {  // (a template does not differ from itself)
      c = compare_tile<false>(tile_at(p, g, s, first, j), s_cnt, p.ws.slot + (u64)j * kDerSlot, kDerSlot, kDerSlot);
      __syncthreads();  // the counts have been read
    }
    if (tid == 0) {
      p.ws.tile_cnt[j] = c;
      p.ws.tile_graph[j] = g;
    }
  }
}

// kSelf: at most kDerSelfTiles tiles; the position is this workgroup's own sum.
template <bool kSelf>
__global__ __launch_bounds__(kDerBlock, 6) void derive_place_kernel(DerParams p) {
  __shared__ __align__(16) DerCounts s_cnt;
  __shared__ u64 s_buf[17];
  const u32 j = blockIdx.x, tid = threadIdx.x, G = p.n_graphs, n = *p.ws.n_tiles;
  if (j >= n) {
    if (j == 0)  // nothing to compare: every list is empty
      for (u32 g = tid; g <= G; g += kDerBlock) p.ovr_off[g] = 0;
    return;
  }
  const u32 c = p.ws.tile_cnt[j], g = p.ws.tile_graph[j], before = j ? p.ws.tile_graph[j - 1] : 0;
  u64 pos;
  if constexpr (kSelf) {
    u64 sum = 0;
    for (u32 i = tid; i < j; i += kDerBlock) sum += p.ws.tile_cnt[i];
    (void)block_excl_scan(sum, s_buf, pos);
  } else {
    pos = p.ws.tile_pos[j];
  }
  // graphs that begin at this tile, those without tiles in front of them included
  for (u32 q = (j ? before + 1 : 0) + tid; q <= g; q += kDerBlock) p.ovr_off[q] = pos;
  if (j + 1 == n) {
    for (u32 q = g + 1 + tid; q <= G; q += kDerBlock) p.ovr_off[q] = pos + c;
    if (tid == 0 && pos + c > p.capacity) raise_status(p.d_status, FDY_ST_CAPACITY);
  }
  constexpr u64 kMost = 2 * kDerTile;  // entries of a tile
  const u64 left = pos < p.capacity ? p.capacity - pos : 0;
  const u32 room = (u32)(left < kMost ? left : kMost);
  if (c <= kDerSlot) {
    if (tid < c && tid < room) p.ovr[pos + tid] = p.ws.slot[(u64)j * kDerSlot + tid];
  } else {
    const u32 s = p.tmpl_graph[p.graph_tmpl[g]];
    compare_tile<true>(tile_at(p, g, s, p.ws.tile_off[g], j), s_cnt, p.ovr + pos, room, ~0u);
  }
}

__global__ __launch_bounds__(1024) void derive_scan_kernel(DerParams p) {
  __shared__ u64 s_buf[17];
  const u32 n = *p.ws.n_tiles;
  u64 carry = 0;
  for (u32 j0 = 0; j0 < n; j0 += 1024) {
    const u32 j = j0 + threadIdx.x;
    const u64 c = j < n ? p.ws.tile_cnt[j] : 0;
    u64 total;
    const u64 e = block_excl_scan(c, s_buf, total);
    if (j < n) p.ws.tile_pos[j] = carry + e;
    carry += total;
  }
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

size_t layout(u64 n_words_total, u32 n_graphs, unsigned char* base, DerWs* ws) {
  const u64 max_tiles = n_words_total / kDerTile + n_graphs;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    unsigned char* p = base ? base + off : nullptr;
    off += align256(bytes);
    return p;
  };
  DerWs w;
  w.n_tiles = (u32*)take(4);
  w.tile_off = (u64*)take(((size_t)n_graphs + 1) * 8);
  w.tile_cnt = (u32*)take((size_t)max_tiles * 4);
  w.tile_graph = (u32*)take((size_t)max_tiles * 4);
  w.slot = (fdy_ovr32*)take((size_t)max_tiles * kDerSlot * sizeof(fdy_ovr32));
  w.tile_pos = (u64*)take((size_t)max_tiles * 8);
  w.max_tiles = (u32)max_tiles;
  if (ws) *ws = w;
  return off;
}

bool sizes_ok(u64 n_words_total, u32 n_graphs) {
  return n_graphs <= (1u << 20) && n_words_total < (1ull << 40);
}

}  // namespace
}  // namespace fdy

using namespace fdy;

extern "C" size_t fdy_derive_workspace_bytes(uint64_t n_words_total, uint32_t n_graphs) {
  if (!sizes_ok(n_words_total, n_graphs)) return 0;
  return layout(n_words_total, n_graphs, nullptr, nullptr);
}

extern "C" int fdy_derive_overrides(const uint64_t* d_words, uint64_t n_words_total, const uint64_t* d_word_off,
                                    uint32_t n_graphs, const uint32_t* d_graph_tmpl,
                                    const uint32_t* d_tmpl_graph, uint32_t n_templates, fdy_ovr32* d_ovr,
                                    uint64_t ovr_capacity, uint64_t* d_ovr_off, void* d_workspace,
                                    size_t workspace_bytes, uint32_t* d_status, void* hip_stream) {
  if (!sizes_ok(n_words_total, n_graphs)) return FDY_ERR_INVALID_ARG;
  if (!d_word_off || !d_ovr_off) return FDY_ERR_INVALID_ARG;
  if (n_graphs && (!d_graph_tmpl || !d_tmpl_graph)) return FDY_ERR_INVALID_ARG;
  if (n_words_total && (!d_words || ((uintptr_t)d_words & 7))) return FDY_ERR_INVALID_ARG;
  if (ovr_capacity && (!d_ovr || ((uintptr_t)d_ovr & 7))) return FDY_ERR_INVALID_ARG;
  const size_t need = layout(n_words_total, n_graphs, nullptr, nullptr);
  if (!d_workspace || ((uintptr_t)d_workspace & 255) || workspace_bytes < need) return FDY_ERR_WORKSPACE;
  DerParams p;
  p.words = (const u64*)d_words;
  p.word_off = (const u64*)d_word_off;
  p.n_graphs = n_graphs;
  p.graph_tmpl = d_graph_tmpl;
  p.tmpl_graph = d_tmpl_graph;
  p.n_templates = n_templates;
  p.n_words_total = n_words_total;
  p.ovr = d_ovr;
  p.capacity = ovr_capacity;
  p.ovr_off = (u64*)d_ovr_off;
  p.d_status = d_status;
  layout(n_words_total, n_graphs, (unsigned char*)d_workspace, &p.ws);
  hipStream_t stream = (hipStream_t)hip_stream;
  (void)hipGetLastError();  // drop any stale error left by earlier, unrelated runtime calls
  const u32 tiles = p.ws.max_tiles ? p.ws.max_tiles : 1;  // one workgroup at least: the checks, the offsets
  const u32 resident = tiles < kDerGrid ? tiles : kDerGrid;
  if (n_graphs > kDerOwnGraphs) {
    hipLaunchKernelGGL(derive_prep_kernel, dim3(1), dim3(1024), 0, stream, p);
    FDY_HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(derive_tile_kernel<false>, dim3(resident), dim3(kDerBlock), 0, stream, p);
  } else {
    hipLaunchKernelGGL(derive_tile_kernel<true>, dim3(resident), dim3(kDerBlock), 0, stream, p);
  }
  FDY_HIP_TRY(hipGetLastError());
  if (tiles > kDerSelfTiles) {
    hipLaunchKernelGGL(derive_scan_kernel, dim3(1), dim3(1024), 0, stream, p);
    FDY_HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(derive_place_kernel<false>, dim3(tiles), dim3(kDerBlock), 0, stream, p);
  } else {
    hipLaunchKernelGGL(derive_place_kernel<true>, dim3(tiles), dim3(kDerBlock), 0, stream, p);
  }
  FDY_HIP_TRY(hipGetLastError());
  return FDY_OK;
}
