// fdy_level0.hpp - level 0 of the table hierarchy: keys of sampled bases behind a bucket index,
// and, for tables whose every base has its key there, the whole interval search.  The functions
// are plain index arithmetic and are also compiled for the host, where
// tests/level0/level0_host.hip runs them over every small table under AddressSanitizer.
#pragma once
#include <type_traits>

#include "fdy_device.hpp"

namespace fdy {

// Level-0 keys are (base - span_lo) >> shift with the smallest shift that makes every key of
// the span fit key_bits bits (all-ones pads).  What the truncation leaves ambiguous is settled
// on the exact bases, so the shift affects speed only.
__host__ __device__ __forceinline__ u32 key_shift_for(u64 span_len, u32 key_bits) {
  const u64 m = span_len - 1;
  const u32 bits = m ? 64u - (u32)__builtin_clzll(m) : 0u;
  return bits > key_bits ? bits - key_bits : 0u;
}

// The level-0 key space is cut into 2^bucket_log2 equal buckets (key >> shift); the shift is the
// smallest that maps the span's largest key below the bucket count.
__host__ __device__ __forceinline__ u32 bucket_shift_for(u64 span_len, u32 key_shift, u32 bucket_log2) {
  const u64 max_key = (span_len - 1) >> key_shift;
  const u32 bits = max_key ? 64u - (u32)__builtin_clzll(max_key) : 0u;
  return bits > bucket_log2 ? bits - bucket_log2 : 0u;
}

// Level-0 entries: a power of two; those from `sampled` on are padding.  At least four, because the
// keys are staged in whole 16-byte pieces and the search reads every key of a piece: with two, half
// of the piece was memory that nobody had written.
inline u32 level0_entries(u32 sampled) {
  u32 n = 4;
  while (n < sampled) n <<= 1;
  return n;
}

// 32-bit key i of level 0 (every 2^sh0-th base), all ones behind the table's end.
__host__ __device__ __forceinline__ u32 level0_key(const fdy_alloc* table, u32 n_alloc, u32 sh0, u64 i, u64 span_lo,
                                                   u32 key_shift) {
  const u64 j = i << sh0;
  return j < n_alloc ? (u32)((table[j].base - span_lo) >> key_shift) : 0xffffffffu;
}

// First of the n sampled keys that is not below target, eight-way: a table cold in the caches costs
// a round trip per step, and five steps of seven loads beat fourteen of one (7.2 -> 4.3 us for
// 16,384 entries).
__host__ __device__ __forceinline__ u32 sampled_lower_bound(const fdy_alloc* table, u32 sh0, u32 n, u64 span_lo,
                                                            u32 key_shift, u64 target) {
  u32 lo = 0, hi = n;
  while (lo < hi) {
    const u32 len = hi - lo;
    u64 k[7];
    u32 at[7];
#pragma unroll
    for (u32 i = 0; i < 7; ++i) {
      at[i] = lo + (u32)(((u64)len * (i + 1)) >> 3);  // ascending; the same place twice in short ranges
      k[i] = (table[(u64)at[i] << sh0].base - span_lo) >> key_shift;
    }
    u32 nlo = lo, nhi = hi;
#pragma unroll
    for (u32 i = 0; i < 7; ++i)
      if (k[i] < target) nlo = at[i] + 1;
#pragma unroll
    for (int i = 6; i >= 0; --i)
      if (k[i] >= target) nhi = at[i];
    lo = nlo;
    hi = nhi;
  }
  return lo;
}

// ---- tables whose every base has its key in level 0
constexpr u32 kFlatPad = 8;  // keys behind the last one (all ones)

// What a workgroup stages and knows before its first word.
struct FlatLevel {
  const unsigned char* keys;  // u32 keys, addressed in bytes
  const unsigned short* bst;
  u64 span_lo, span_len;
  u32 key_shift, bucket_shift, last_at;  // last_at: byte offset of a key that is padding
};
__host__ __device__ __forceinline__ size_t flat_level_bytes(u32 top_n, u32 bucket_log2) {
  return (size_t)top_n * 4 + kFlatPad * 4 + ((((((size_t)1) << bucket_log2) + 1) * 2 + 15) & ~(size_t)15);
}

// The largest level 0 that is staged (plan_table keeps to it).
constexpr u32 kMostTopLog2 = 14, kMostBucketLog2 = 13;

// Where the keys are staged and what else a wave knows of them.  P: the launch's parameters (top, bstart, top_n,
// bucket_log2, table, n_alloc).
template <typename P>
__host__ __device__ __forceinline__ FlatLevel flat_level(const P& p, unsigned char* smem) {
  FlatLevel f;
  const u32 key_vec = p.top_n / 4;
  f.keys = smem;
  f.bst = reinterpret_cast<const unsigned short*>(smem + (size_t)(key_vec * 16 + kFlatPad * 4));
  f.last_at = key_vec * 16;
  f.span_lo = p.table[0].base;
  f.span_len = p.table[p.n_alloc - 1].base + p.table[p.n_alloc - 1].size - f.span_lo;
  f.key_shift = key_shift_for(f.span_len, 31);
  f.bucket_shift = bucket_shift_for(f.span_len, f.key_shift, p.bucket_log2);
  return f;
}

// Stages the keys and their index.  at_once: all pieces of the keys and
// their index are requested before the first arrives, and not each behind the one before.  For keys that a launch just
// before has written, which come from afar: us of a rebase with its preparation, piece by piece / at once, 16,384
// allocations, 100,003 words 11.7 / 10.2, 1.0 M 14.5 / 13.2, 5.0 M 26.9 / 25.4; 1,024 allocations 8.6 / 8.4, 11.4 / 11.3.  Keys of
// a table prepared before, which the caches hold, are better piece by piece below nodes: 1.0 M words, 4,096 allocations
// 8.8 / 9.05, 16,384 10.2 / 10.5, 5.0 M and 1,024 17.4 / 18.2; with nodes above the lines it is at once again, 1.0 M
// words and 10^6 allocations 18.8 / 17.9, 5.0 M and 300,000 34.9 / 34.1.  (The ordered scan's waves wait for their
// workgroup's ticket anyway: with all at once 0.4 us longer on 8,439 words, 1 us of 63 on 12.3 M words with lines, 1 us
// of 154 shorter with nodes.)
template <u32 kThreads, typename P>
__host__ __device__ __forceinline__ FlatLevel flat_stage(const P& p, unsigned char* smem, u32 tid, bool at_once) {
  const u32 n_bst = (1u << p.bucket_log2) + 1;
  const u32 key_vec = p.top_n / 4, bst_vec = (n_bst * 2 + 15) / 16;
  uint4* dst = reinterpret_cast<uint4*>(smem);
  const uint4 *ks = reinterpret_cast<const uint4*>(p.top), *bs = reinterpret_cast<const uint4*>(p.bstart);
  if (at_once) {
    constexpr u32 kMostPieces = (1u << kMostTopLog2) / 4 + (1u << kMostBucketLog2) / 8 + 1;
    constexpr u32 kBatch = (kMostPieces + kThreads - 1) / kThreads;
    const u32 pieces = key_vec + bst_vec;
    typedef u32 piece_t __attribute__((ext_vector_type(4)));
    const piece_t *kp = reinterpret_cast<const piece_t*>(p.top), *bp = reinterpret_cast<const piece_t*>(p.bstart);
    piece_t v[kBatch];
#pragma unroll
    for (u32 c = 0; c < kBatch; ++c) {
      if (c * kThreads >= pieces) break;  // (the same for all threads)
      // (beyond the last piece: the last again, no branch around the load)
      const u32 at = c * kThreads + tid, i = at < pieces ? at : pieces - 1;
      v[c] = *(i < key_vec ? kp + i : bp + (i - key_vec));
    }
#pragma unroll
    for (u32 c = 0; c < kBatch; ++c) {
      if (c * kThreads >= pieces) break;
      const u32 i = c * kThreads + tid;
      if (i < pieces) reinterpret_cast<piece_t*>(dst)[i < key_vec ? i : i + kFlatPad / 4] = v[c];
    }
  } else {
    for (u32 i = tid; i < key_vec; i += kThreads) dst[i] = ks[i];
    for (u32 i = tid; i < bst_vec; i += kThreads) dst[key_vec + kFlatPad / 4 + i] = bs[i];
  }
  if (tid < kFlatPad / 4) dst[key_vec + tid] = make_uint4(~0u, ~0u, ~0u, ~0u);
  return flat_level(p, smem);
}

// Level 0 for N distances d = word - span_lo per lane: byte offset of the last key not above each
// word's (key 0 is 0).
// The place among the keys of the bucket is found without branches: the step count is the one
// that the fullest of the wave's buckets needs, a step that leads past the bucket meets keys
// above the word's (keys ascend over the whole table) or the padding.
// any(b): whether b holds in some lane of the wave.
template <int N, typename Any>
__host__ __device__ __forceinline__ void flat_place(const FlatLevel& f, const u64 (&d)[N], u32 (&at)[N], Any any) {
  u32 kw[N], most = 0;  // at: byte offset of the first key not known to be at or below the word's
#pragma unroll
  for (int c = 0; c < N; ++c) {
    kw[c] = (u32)(d[c] >> f.key_shift);
    const u32 bk = kw[c] >> f.bucket_shift;
    const u32 lo = f.bst[bk], hi = f.bst[bk + 1];
    at[c] = lo * 4;
    most |= hi - lo;
  }
  u32 steps = 0;
  while (any((most >> steps) != 0)) ++steps;  // 2^steps > every lane's count
  for (; steps > 3; --steps) {
    const u32 step = 4u << (steps - 1);
    u32 k[N];
#pragma unroll
    for (int c = 0; c < N; ++c) k[c] = *reinterpret_cast<const u32*>(f.keys + (at[c] + step - 4 < f.last_at ? at[c] + step - 4 : f.last_at));
#pragma unroll
    for (int c = 0; c < N; ++c) at[c] += k[c] <= kw[c] ? step : 0u;
  }
  auto fixed = [&](auto step_c) __attribute__((always_inline)) {
    constexpr u32 step = decltype(step_c)::value;
    u32 k[N];
#pragma unroll
    for (int c = 0; c < N; ++c) k[c] = *reinterpret_cast<const u32*>(f.keys + at[c] + (step - 4));
#pragma unroll
    for (int c = 0; c < N; ++c) at[c] += k[c] <= kw[c] ? step : 0u;
  };
  if (steps >= 3) fixed(std::integral_constant<u32, 16>{});
  if (steps >= 2) fixed(std::integral_constant<u32, 8>{});
  if (steps >= 1) fixed(std::integral_constant<u32, 4>{});
#pragma unroll
  for (int c = 0; c < N; ++c) at[c] -= 4;
}

// Interval search where every base has its key in level 0: region, and the offset inside it if
// the entry holds the word (else any value at or above the entry's size: see hit).
template <int N, typename P, typename Any>
__host__ __device__ __forceinline__ void flat_search(const P& p, const FlatLevel& f, const u64 (&d)[N], u32 (&n)[N],
                                                     u64 (&off)[N], bool (&hit)[N], Any any) {
  u32 at[N];
  flat_place<N>(f, d, at, any);
  const unsigned char* table = reinterpret_cast<const unsigned char*>(p.table);
  u64x2 e[N];
#pragma unroll
  for (int c = 0; c < N; ++c) e[c] = *reinterpret_cast<const u64x2*>(table + at[c] * 4);
  // a base with the word's own truncated key may still lie above the word: one entry back, or,
  // where a run of blocks shares a key, a search among the exact bases.  A valid table's first
  // base is never above a candidate; an invalid one's may be (a span that wraps): a miss.
#pragma unroll
  for (int c = 0; c < N; ++c) {
    const u64 w = d[c] + f.span_lo;
    n[c] = at[c] >> 2;
    for (u32 step = 0; e[c].x > w; ++step) {
      if (n[c] == 0) {
        e[c].y = 0;
        break;
      }
      if (step < 4) {
        --n[c];
      } else {
        u32 a = 0, b = n[c];  // the last entry of [a, b) that is not above the word
        while (b - a > 1) {
          const u32 mid = a + ((b - a) >> 1);
          if (p.table[mid].base <= w) a = mid;
          else b = mid;
        }
        n[c] = a;
      }
      e[c] = *reinterpret_cast<const u64x2*>(&p.table[n[c]]);
    }
    off[c] = w - e[c].x;
    hit[c] = off[c] < e[c].y;
  }
}

}  // namespace fdy
