// fdy_lines.hpp - what lies below level 0 for tables that do not fit it: lines (eight entries of
// the table, 64 bytes or 32) and nodes (eight keys, the first bases of eight lines or nodes, 32
// bytes).  Packing, and finding a word's entry in them.  Plain arithmetic, also compiled for the
// host, where tests/level0/lines_host.hip compares every form with the definition.
//
// Nodes and lines hold distances from their first base, which they do not hold in full: whatever
// leads to them (a level-0 key, a node's distance) says it up to some low bits, and those are
// kept.  So level 0 samples the lines themselves where it can (up to 8 * 2^14 allocations): one
// request per candidate, where the base from an array of its own would be a second and a node
// between a third.
#pragma once
#include "fdy_device.hpp"
#include "fdy_level0.hpp"

namespace fdy {

constexpr u32 kMarked = 0xffffffffu;  // first word of a line that does not fit its form

// ---- units: what a level-0 key stands for, a line or the nodes above 8^k of them.  Keys are truncated: the last unit
// whose key is not above a word's may begin above the word, and so may several where units share the key (blocks of a
// few KiB and one region 2^46 bytes away: a key spans 64 KiB).  Exact first bases settle it, among the units with
// that key and the one before them.  us, 8.4 M words, a quarter pointers to blocks of 512 B to 8 KiB, one region
// 2^47 bytes away, whole table searched / settled: 100,000 blocks 156 / 76, 10^6 blocks 189 / 75.

// Whether the unit before u has the key of distance d as well: more than u may begin above the word.
__host__ __device__ __forceinline__ bool units_share(const FlatLevel& f, u64 d, u32 u) {
  return u && reinterpret_cast<const u32*>(f.keys)[u - 1] == (u32)(d >> f.key_shift);
}

// The last unit at or below u that begins at or below the word (0 if there is none), u being the last whose key is
// not above the word's.  units: exact first bases, and kUnitWindow more that may hold anything.  A power of four says
// how far back the units with the word's key reach at most, each request divides that by four, and the last is for
// neighbours, 32 bytes in a row (as four requests: 76 us above become 81).
constexpr u32 kUnitWindow = 4;
__host__ __device__ __forceinline__ u32 settle_unit(const FlatLevel& f, const u64* units, u64 d, u32 u) {
  const u64 w = d + f.span_lo;
  u32 reach = kUnitWindow;
  while (reach < u && reinterpret_cast<const u32*>(f.keys)[u - reach] == (u32)(d >> f.key_shift)) reach <<= 2;
  u32 r = u > reach ? u - reach : 0u;
  u64 b[kUnitWindow];
  for (u32 s = reach >> 2; s > 1; s >>= 2) {
    u32 m[4];
#pragma unroll
    for (u32 h = 0; h < 4; ++h) {
      m[h] = r + (h + 1) * s < u ? r + (h + 1) * s : u;
      b[h] = units[m[h]];
    }
#pragma unroll
    for (u32 h = 0; h < 4; ++h)
      if (b[h] <= w) r = m[h];
  }
  const u32 from = r + 1;
#pragma unroll
  for (u32 h = 0; h < kUnitWindow; ++h) b[h] = units[from + h];
#pragma unroll
  for (u32 h = 0; h < kUnitWindow; ++h)
    if (b[h] <= w && from + h <= u) r = from + h;
  return r;
}

// The same in few instructions, where it is rare: u itself is known to begin above the word.
__host__ __device__ __forceinline__ u32 settle_unit_rare(const FlatLevel& f, const u64* units, u64 d, u32 u) {
  const u64 w = d + f.span_lo;
  u32 reach = 4;
  while (reach < u && reinterpret_cast<const u32*>(f.keys)[u - reach] == (u32)(d >> f.key_shift)) reach <<= 1;
  u32 r = u > reach ? u - reach : 0u;
  while (u - r > 1) {
    const u32 mid = r + ((u - r) >> 1);
    if (units[mid] <= w) r = mid;
    else u = mid;
  }
  return r;
}

// ---- wide line: {distance >> s, size >> s} of each entry, 32 bits each, s the trailing zeros common to
// all sixteen (at most 31; allocators hand out aligned blocks, so regions far beyond 4 GiB fit).
// The first entry's distance is 0; its word holds s (low five bits) and the dropped part of the
// first base.
// ---- compact line: a word per entry, distance >> sd above size >> ss.  The first entry's distance
// bits hold the form (top bit) and the shifts:
//   0  12 bits of distance, 20 of size; sd 6 bits, ss 5 above them
//   1  13 and 19, the size's top bit meaning "shifted by kBigShift more": a line with a region of
//      gigabytes (whole 2 MiB pages and more) beside small ones; sd 6, ss 6
// Only lines whose first base needs no dropped part have it.
constexpr u32 kBigShift = 12;
constexpr u32 kMostDropped = 27;  // bits of a first base that a node or a wide line can keep

// The last of eight ascending values (v[0] first) that is not above x, given that v[0] counts as
// not above it.  (One after the other: as a tree, three compares and selections among the rest, the
// searches took a quarter longer.)
struct Place {
  u32 at, v;
};
__host__ __device__ __forceinline__ Place last_not_above(const u32 (&v)[8], u32 x) {
  Place r{0, v[0]};
#pragma unroll
  for (int h = 1; h < 8; ++h)
    if (v[h] <= x) {
      r.at = h;
      r.v = v[h];
    }
  return r;
}

struct PackedLine {
  u32 wide[16], compact[8];
};
// Line of entries e0 .. e0 + 7; told: what leads to the line says of its first base.
__host__ __device__ __forceinline__ void pack_line(const fdy_alloc* table, u64 e0, u64 n_alloc, u64 told, PackedLine& out) {
  bool fits = e0 + 8 <= n_alloc && (table[e0].base - told) >> kMostDropped == 0;  // (the last, partial line stays marked)
  bool form0 = fits, form1 = fits;
  if (fits) {
    u64 d[8], z[8], any_d = 0, any_z = 0, any_small = 0;
    const u64 b0 = table[e0].base;
    const u32 dropped = (u32)(b0 - told);
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      d[h] = table[e0 + h].base - b0;
      z[h] = table[e0 + h].size;
      any_d |= d[h];
      any_z |= z[h];
    }
    auto zeros = [](u64 v, u32 most) {
      const u32 n = v ? (u32)__builtin_ctzll(v) : 0u;
      return n < most ? n : most;
    };
    const u32 s = zeros(any_d | any_z, 31), sd = zeros(any_d, 63), ss = zeros(any_z, 31);
    out.wide[0] = s | dropped << 5;
    fits = out.wide[0] != kMarked;
    form0 = form1 = dropped == 0;
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      fits = fits && ((d[h] >> s) >> 32) == 0 && ((z[h] >> s) >> 32) == 0;
      if (h) out.wide[2 * h] = (u32)(d[h] >> s);
      out.wide[2 * h + 1] = (u32)(z[h] >> s);
      form0 = form0 && ((d[h] >> sd) >> 12) == 0 && ((z[h] >> ss) >> 20) == 0;
      out.compact[h] = (u32)(d[h] >> sd) << 20 | ((u32)(z[h] >> ss) & 0xfffffu);
    }
    out.compact[0] |= sd << 20 | ss << 26;
    if (!form0 && form1) {
      // the shift of those that fit without the extra one; the others must lose nothing by it
#pragma unroll
      for (int h = 0; h < 8; ++h)
        if (z[h] >> (ss + 18) == 0) any_small |= z[h];
      const u32 s1 = zeros(any_small, 31);
#pragma unroll
      for (int h = 0; h < 8; ++h) {
        const bool big = z[h] >> (s1 + 18) != 0;
        const u32 sh = s1 + (big ? kBigShift : 0u);
        const u64 m = z[h] >> sh;
        form1 = form1 && ((d[h] >> sd) >> 13) == 0 && (m >> 18) == 0 && m << sh == z[h];
        out.compact[h] = (u32)(d[h] >> sd) << 19 | ((u32)m & 0x3ffffu) | (big ? 1u << 18 : 0u);
      }
      out.compact[0] |= 1u << 31 | sd << 19 | s1 << 25;
    }
  }
  if (!fits) out.wide[0] = out.wide[2] = kMarked;
  if (!form0 && !form1) out.compact[0] = kMarked;
}

// The entry of the line that w falls at or behind: place in the line, exact base and size.  first:
// the line's first base, as far as it is known (what the line keeps is added).  False: the line is
// marked, or its first base lies above w (truncated keys can lead a line too far).
__host__ __device__ __forceinline__ bool pick_wide_line(const uint4 (&q)[4], u64 w, u64 first, u32& at, u64x2& e) {
  const u64 b = first + (q[0].x >> 5);
  const bool ok = q[0].x != kMarked & b <= w;
  const u32 s = q[0].x & 31u;
  const u64 x64 = (w - b) >> s;  // floor: entry h lies at or below w iff its distance <= x
  const u32 x = x64 >> 32 ? 0xffffffffu : (u32)x64;
  const u32 d[8] = {0u, q[0].z, q[1].x, q[1].z, q[2].x, q[2].z, q[3].x, q[3].z};
  const u32 z[8] = {q[0].y, q[0].w, q[1].y, q[1].w, q[2].y, q[2].w, q[3].y, q[3].w};
  const Place r = last_not_above(d, x);
  at = r.at;
  u32 zz = z[0];
#pragma unroll
  for (int h = 1; h < 8; ++h) zz = d[h] <= x ? z[h] : zz;
  e.x = b + ((u64)r.v << s);
  e.y = (u64)zz << s;
  return ok;
}

__host__ __device__ __forceinline__ bool pick_compact_line(const uint4 (&q)[2], u64 w, u64 first, u32& at, u64x2& e) {
  const u32 head = q[0].x;
  const bool ok = head != kMarked & first <= w;
  const u32 form = head >> 31, zbits = 20u - form, zmask = 0xfffffu >> form;
  const u32 sd = head >> zbits & 63u, ss = head >> (zbits + 6) & 63u;  // (form 0: the top bit is 0)
  const u64 x = (w - first) >> sd;
  // entry h lies at or below w iff its distance <= x, i.e. iff its whole word <= x's with all size
  // bits set
  const u32 xt = x >> ((32 - zbits) & 63u) ? 0xffffffffu : ((u32)x << zbits | zmask);
  const u32 v[8] = {head & zmask, q[0].y, q[0].z, q[0].w, q[1].x, q[1].y, q[1].z, q[1].w};
  const Place r = last_not_above(v, xt);
  at = r.at;
  const u32 d = r.v >> zbits, z = r.v & zmask;  // (v[0] has no distance bits)
  const u32 big = form & (z >> 18);
  e.x = first + ((u64)d << sd);
  e.y = (u64)(z ^ big << 18) << ((ss + big * kBigShift) & 63u);
  return ok;
}

// ---- node: seven distances from key 0 after a shift, 32 bits each (all ones: no such key; the last node of a
// level may have fewer than eight).  The shift is the distances' common trailing zeros, or, where they then do not
// fit, what they need: of a child's key the lost bits are then missing, which the child keeps.
// Word 0: shift (5 bits) and the dropped part of key 0.
// Node of the keys at entries k0, k0 + step, ...; told: what leads to the node says of key 0.
struct PackedNode {
  u32 w[8];
};
__host__ __device__ __forceinline__ void pack_node(const fdy_alloc* table, u64 k0, u64 step, u64 n_alloc, u64 told,
                                                   PackedNode& out) {
  const u64 b0 = table[k0].base, dropped = b0 - told;
  u64 d[8], any = 0;
#pragma unroll
  for (int h = 1; h < 8; ++h) {
    const u64 k = k0 + step * h;
    d[h] = k < n_alloc ? table[k].base - b0 : 0;
    any |= d[h];
  }
  u32 s = any ? (u32)__builtin_ctzll(any) : 0u;
  const u32 bits = any ? 64u - (u32)__builtin_clzll(any) : 0u;
  if (s > 31u) s = 31u;
  if (bits > s + 31u) s = bits - 31u;  // (31 bits: all ones stay free)
  const bool fits = s <= 31u && dropped >> kMostDropped == 0 && (s | (u32)dropped << 5) != kMarked;
  out.w[0] = fits ? s | (u32)dropped << 5 : kMarked;
#pragma unroll
  for (int h = 1; h < 8; ++h) out.w[h] = k0 + step * h < n_alloc ? (u32)(d[h] >> (s & 63u)) : 0xffffffffu;
}
// What the node of keys k0, k0 + step, ... says of the first key of the child at entry k0 + step * h.
__host__ __device__ __forceinline__ u64 told_of_child(const fdy_alloc* table, u64 k0, u64 step, u64 n_alloc, u32 h) {
  PackedNode n;
  pack_node(table, k0, step, n_alloc, table[k0].base, n);
  return table[k0].base + (h ? (u64)n.w[h] << (n.w[0] & 31u) : 0);
}

// The child that w falls into and what is told of its first key (child 0 if key 0 lies above w, which its
// line will show); first: what is told of the node's key 0.  False: the node is marked.
__host__ __device__ __forceinline__ bool pick_node(const uint4 (&q)[2], u64 w, u32& at, u64& first) {
  const u64 b = first + (q[0].x >> 5);
  const u32 s = q[0].x & 31u;
  const u64 x64 = b <= w ? (w - b) >> s : 0;
  const u32 x = x64 > 0xfffffffeull ? 0xfffffffeu : (u32)x64;
  const u32 d[8] = {0u, q[0].y, q[0].z, q[0].w, q[1].x, q[1].y, q[1].z, q[1].w};
  const Place r = last_not_above(d, x);
  at = r.at;
  first = b + ((u64)r.v << s);
  return q[0].x != kMarked;
}

// What became of a candidate, in 64 bits: {word of the sub-tile (9 bits), region, offset (the rest)}, all
// ones if no hit (no region is as large as its field).  An offset that does not fit (for 2^20
// allocations 16 GiB and more into a region) has a field of ones: whoever writes the entry takes
// word and base from memory.
struct Entries {
  u32 off_bits;
  __host__ __device__ __forceinline__ u64 none() const { return (1ull << off_bits) - 1; }
  __host__ __device__ __forceinline__ u64 pack(u32 word, u32 region, u64 off) const {
    return (u64)word << 55 | (u64)region << off_bits | (off < none() ? off : none());
  }
  __host__ __device__ __forceinline__ u32 word(u64 e) const { return (u32)(e >> 55); }
  __host__ __device__ __forceinline__ u32 region(u64 e) const { return (u32)(e << 9 >> 9 >> off_bits); }
  __host__ __device__ __forceinline__ u64 off(u64 e) const { return e & none(); }
};
// The most bits that the regions of a table leave: n_alloc < 2^(55 - off_bits).
inline u32 entry_off_bits(u64 n_alloc) {
  u32 bits = 55;
  while (n_alloc >> (55 - bits)) --bits;
  return bits;
}

// One behind the last entry of the line at entry lo (lo + 8 need not fit 32 bits).
__host__ __device__ __forceinline__ u32 line_end(u32 lo, u32 n_alloc) { return n_alloc - lo < 8u ? n_alloc : lo + 8u; }

// In the table itself, for the rare candidate whose line or a node above it is marked or begins above
// w: the last entry at or below w among [lo, hi).
__host__ __device__ __forceinline__ void find_exact(const fdy_alloc* table, u32 lo, u32 hi, u64 w, u32& n, u64x2& e) {
#pragma unroll 1
  while (hi - lo > 1) {
    const u32 mid = lo + ((hi - lo) >> 1);
    if (table[mid].base <= w) lo = mid;
    else hi = mid;
  }
  n = lo;
  e = *reinterpret_cast<const u64x2*>(&table[lo]);
  if (e.x > w) e.y = 0;  // no entry lies below w (an invalid table's first base may not be its least)
}

}  // namespace fdy
