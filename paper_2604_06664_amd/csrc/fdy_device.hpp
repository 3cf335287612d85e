// Internal helpers shared by the HIP kernels of libfdy (gfx950, wave64).  Not installed.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include <atomic>

#include "fdy.h"
#include "fdy_internal.h"

#define FDY_WAVE 64

#define FDY_HIP_TRY(expr)                      \
  do {                                         \
    hipError_t e__ = (expr);                   \
    if (e__ != hipSuccess) return FDY_ERR_HIP; \
  } while (0)

namespace fdy {

typedef uint64_t u64;
typedef uint32_t u32;

__device__ __forceinline__ u32 lane_id() { return __lane_id(); }

__device__ __forceinline__ u64 lanemask_lt() {
  const u32 l = lane_id();
  return l == 0 ? 0ull : (~0ull >> (64 - l));
}

__device__ __forceinline__ u64 ballot(bool p) { return __ballot(p); }

// 16-byte vector load / store of two 64-bit words
struct __attribute__((aligned(16))) u64x2 {
  u64 x, y;
};

// Buffer accesses: lanes whose offset is not below the descriptor's bytes read zero and store nothing, so that
// loads and stores need no branches around them and stay together.  (Accesses lie wholly inside or wholly outside:
// what one does that straddles the end is not relied upon.)
typedef u32 v4u32 __attribute__((ext_vector_type(4)));
typedef u32 v2u32 __attribute__((ext_vector_type(2)));
constexpr int kNonTemporal = 2;        // cache policy of a buffer access
constexpr u32 kNowhere = 0x80000000u;  // an offset behind every descriptor's end
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void* base, u32 bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}
__device__ __forceinline__ u64 pair64(u32 lo, u32 hi) { return (u64)lo | (u64)hi << 32; }
// A value that is the same in all lanes, where the compiler cannot see that it is (a descriptor made of others is
// looped over).
__device__ __forceinline__ u32 uniform(u32 v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ u64 uniform(u64 v) { return pair64(uniform((u32)v), uniform((u32)(v >> 32))); }

__device__ __forceinline__ void raise_status(u32* d_status, u32 bit) {
  if (d_status) atomicOr(d_status, bit);
}

// Wave-cooperative lower bound.  key(i) must be non-decreasing over [lo, hi); every lane
// of the wave must call with the same arguments.  Returns the first index in [lo, hi] whose
// key is not below `target` (hi if none).  Each round probes 64 evenly spaced positions in
// parallel, so a range of n entries needs ceil(log64 n) dependent memory round trips
// instead of log2 n.
//
// The index space is 32-bit with hi <= 2^32 - 256 (every list this library searches is
// shorter), and the wave-uniform range is updated with 32-bit min/add only.  This is
// deliberate: hipcc 7.2 miscompiles a chain of two wave-uniform 64-bit compare+select
// steps for gfx950 (the second select reuses the first compare's SCC), which is exactly
// what a 64-bit version of this loop produces.
template <typename KeyFn>
__device__ __forceinline__ u32 wave_lower_bound(KeyFn key, u32 lo, u32 hi, u64 target) {
  const u32 l = lane_id();
  while (lo < hi) {
    const u32 n = hi - lo;
    const u32 stride = (n + 63u) >> 6;                 // ceil(n / 64) >= 1
    const u32 idx = lo + (l + 1u) * stride - 1u;       // this lane's probe, <= hi + 62
    u64 k = ~0ull;                                     // past the end: never below
    if (idx < hi) k = key(idx);
    const u32 c = (u32)__popcll(ballot(k < target));   // probes below the target (a prefix)
    // entries up to probe c-1 are below   => answer >= lo + c*stride
    // probe c, if it exists, is not below => answer <= lo + (c+1)*stride - 1
    const u32 nlo = min(lo + c * stride, hi);
    const u32 nhi = nlo + min(stride - 1u, hi - nlo);
    lo = nlo;
    hi = nhi;
  }
  return lo;
}

// What another lane holds, by the data-parallel primitives of the vector unit: a shift to the right by 1, 2, 4 or 8 within
// rows of 16 lanes, or the last lane of the row (of the half) before for the rows in kRows; `otherwise` in lanes that have no
// such neighbour.  All lanes of the wave take part.  (Through LDS, as __shfl_up goes, six steps of three 64-bit sums wait for
// each other and for those of the compute unit's other waves: 3 to 7 us of a prep launch for 512 graphs, 2 to 5 now.  us of
// whole passes, scans over a wave through LDS / so: load of 67 graphs 24.7 / 23.9, of 67 of 2,632 nodes for 8 ranks 88.8 /
// 87.3, of 512 graphs 61.9 / 60.4, save 45.1 / 43.1; the ordered fold of fingerprints 24.2 / 23.9, 87.6 / 87.3, 60.6 / 60.4,
// 43.3 / 43.0; for one graph of 512 nodes neither shows, 16.5 to 17.)
template <int kCtrl, int kRows = 0xf>
__device__ __forceinline__ u32 dpp(u32 v, u32 otherwise) {
  return (u32)__builtin_amdgcn_update_dpp((int)otherwise, (int)v, kCtrl, kRows, 0xf, false);
}
template <int kCtrl, int kRows = 0xf>
__device__ __forceinline__ u64 dpp(u64 v, u64 otherwise) {
  return pair64(dpp<kCtrl, kRows>((u32)v, (u32)otherwise), dpp<kCtrl, kRows>((u32)(v >> 32), (u32)(otherwise >> 32)));
}
constexpr int kShr1 = 0x111, kShr2 = 0x112, kShr4 = 0x114, kShr8 = 0x118;  // row_shr
constexpr int kOfRow = 0x142, kOfHalf = 0x143;                            // row_bcast:15 (rows 1 and 3), :31 (rows 2 and 3)

// Inclusive scan of a value per lane over a wave.
template <typename T>
__device__ __forceinline__ T wave_incl_scan(T v) {
  v += dpp<kShr1>(v, (T)0);
  v += dpp<kShr2>(v, (T)0);
  v += dpp<kShr4>(v, (T)0);
  v += dpp<kShr8>(v, (T)0);
  v += dpp<kOfRow, 0xa>(v, (T)0);
  v += dpp<kOfHalf, 0xc>(v, (T)0);
  return v;
}

// Exclusive scan of one u64 per thread over a workgroup of whole waves (at most 1024 threads);
// returns the exclusive prefix and sets `total` (same in every thread).  s_buf: 17 u64 of LDS.
__device__ inline u64 block_excl_scan(u64 v, u64* s_buf, u64& total) {
  const u32 l = lane_id(), w = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
  const u64 inc = wave_incl_scan(v);
  if (l == 63) s_buf[w] = inc;
  __syncthreads();
  if (w == 0) {
    const u64 x = l < n_waves ? s_buf[l] : 0;
    const u64 xi = wave_incl_scan(x);
    if (l < 16) s_buf[l] = xi - x;
    if (l == 15) s_buf[16] = xi;
  }
  __syncthreads();
  const u64 r = s_buf[w] + inc - v;
  total = s_buf[16];
  __syncthreads();
  return r;
}

// The current device and what the launches need to know about it.  Asking the runtime costs
// 0.2-0.4 us a question, which the latency-bound calls feel, so a device's compute-unit count is
// kept once known.  Devices beyond the cache are asked every time.
constexpr int kCachedDevices = 64;
inline int current_device(int* dev, int* n_cu) {
  static std::atomic<int> cached[kCachedDevices];
  FDY_HIP_TRY(hipGetDevice(dev));
  const bool cacheable = *dev >= 0 && *dev < kCachedDevices;
  int n = cacheable ? cached[*dev].load(std::memory_order_relaxed) : 0;
  if (n == 0) {
    FDY_HIP_TRY(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, *dev));
    if (cacheable) cached[*dev].store(n, std::memory_order_relaxed);
  }
  *n_cu = n;
  return FDY_OK;
}

// Lets `kernel` be launched with up to the whole LDS as dynamic shared memory (a limit, not a
// request); one runtime call per kernel and device.
template <typename Fn>
inline int allow_full_lds(Fn kernel, int dev, std::atomic<u64>& done) {
  const bool cacheable = dev >= 0 && dev < kCachedDevices;
  if (cacheable && (done.load(std::memory_order_relaxed) >> dev & 1)) return FDY_OK;
  hipFuncAttributes attr;
  FDY_HIP_TRY(hipFuncGetAttributes(&attr, (const void*)kernel));
  FDY_HIP_TRY(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)(160 * 1024 - attr.sharedSizeBytes)));
  if (cacheable) done.fetch_or(1ull << dev, std::memory_order_relaxed);
  return FDY_OK;
}

// One kernel launch on the caller's stream; when the bench has switched timing on for `slot`,
// the launch carries a pair of events that receive the kernel's own begin and end.
template <typename... KArgs, typename... Args>
inline void launch(int slot, void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds, hipStream_t stream,
                   Args&&... args) {
  static_assert(sizeof...(KArgs) == sizeof...(Args), "one argument per kernel parameter");
  void *a = nullptr, *b = nullptr;
  if (prof_take(slot, &a, &b))
    hipExtLaunchKernelGGL(kernel, grid, block, (uint32_t)lds, stream, (hipEvent_t)a, (hipEvent_t)b, 0u,
                          static_cast<KArgs>(args)...);
  else
    hipLaunchKernelGGL(kernel, grid, block, lds, stream, static_cast<KArgs>(args)...);
}

}  // namespace fdy
