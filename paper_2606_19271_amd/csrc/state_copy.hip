// state_copy.hip -- batched byte-range copies between device memory and pinned host memory.
//
// The paper's runtime suspends an idle session by copying its persistent state from GPU memory
// to host memory, and resumes it by restoring the state to the GPU chosen for it (Sec. 3.1,
// "GPU-CPU state offloading"); only the session's isolated state region moves (Sec. 6.1,
// "Session memory layout").  In a packed token-major batch a session's cached keys or values are
// one contiguous byte range, so suspend, resume and the compaction of a packed batch after
// sessions leave are all lists of range copies: dst[d, d + n) = src[s, s + n).
//
// Design: one launch copies up to kMaxCopyRanges ranges, passed by value in the kernel arguments
// (no device allocation, no host-to-device upload).  Every range is cut into chunks of one 256-thread
// workgroup's 16-byte accesses, all loads of a chunk in flight before its stores.  The chunk index
// space is dense: a prefix over the ranges' chunk counts maps a chunk to its range.  Pinned host
// memory is reached directly at its (unified) virtual address.  What bounds each direction, measured
// on 200 MB to 1.8 GB:
//  * device -> device, HBM: chunks of 16 KiB, one per workgroup, non-temporal on both sides where the
//    data is larger than the caches: 5.9 TB/s read + written.  Chunks of 32 KiB reach 4.2-4.4 TB/s with
//    or without non-temporal accesses, 16 KiB with plain ones 5.7.  Copies that the caches hold for
//    the next reader keep plain accesses (bypass_caches).
//  * device -> host, the link's writes: 32 workgroups walk the chunks together, so that the link sees
//    nearly consecutive writes: 55.6 GB/s, against 53.6 with a workgroup per chunk, whose order the
//    dispatcher scatters (8 workgroups 51.4, 16 55.0, 24 55.7, 48 55.3, 256 52.4).  Each loads its
//    next chunk before it stores the one before.
//  * host -> device, the link's reads: many outstanding requests, 32 KiB a workgroup: 57.1 GB/s
//    (16 KiB: 55.0; 16 or 32 workgroups in a walk: 57.0).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_launch.h"

namespace tsstate {

constexpr int kThreads = 256;
constexpr int kWalkers = 32;  // workgroups of a device -> host copy

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Chunk c of the copy: its vectors, of which the workgroup's thread t has t, t + 256, ...
template <int kVectors>
struct Chunk {
  const u32x4* src;
  u32x4* dst;
  int nvec;

  __device__ __forceinline__ Chunk(const char* s, char* d, const tsattn::CopyList& list, int64_t c) {
    // the range holding chunk c: last r with first_chunk[r] <= c (empty ranges own no chunk)
    int lo = 0, hi = list.n;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (list.first_chunk[mid] <= c) lo = mid; else hi = mid;
    }
    constexpr int64_t kBytes = (int64_t)kThreads * kVectors * 16;
    const int64_t off = (c - list.first_chunk[lo]) * kBytes, left = list.bytes[lo] - off;
    nvec = (int)((left < kBytes ? left : kBytes) >> 4);
    src = (const u32x4*)(s + list.src[lo] + off);
    dst = (u32x4*)(d + list.dst[lo] + off);
  }
  template <bool kNt>
  __device__ __forceinline__ void load(u32x4 (&r)[kVectors]) const {
#pragma unroll
    for (int u = 0; u < kVectors; ++u) {
      const int i = threadIdx.x + u * kThreads;
      if (i < nvec) r[u] = kNt ? __builtin_nontemporal_load(&src[i]) : src[i];
    }
  }
  template <bool kNt>
  __device__ __forceinline__ void store(const u32x4 (&r)[kVectors]) const {
#pragma unroll
    for (int u = 0; u < kVectors; ++u) {
      const int i = threadIdx.x + u * kThreads;
      if (i < nvec) {
        if (kNt) __builtin_nontemporal_store(r[u], &dst[i]);
        else dst[i] = r[u];
      }
    }
  }
};

// One chunk per workgroup: workgroup b takes chunk first + b.
template <int kVectors, bool kNtLoad, bool kNtStore>
__global__ void __launch_bounds__(kThreads)
state_copy_kernel(const char* __restrict__ src, char* __restrict__ dst, tsattn::CopyList list, int64_t first) {
  const Chunk<kVectors> c(src, dst, list, first + blockIdx.x);
  u32x4 r[kVectors];
  c.template load<kNtLoad>(r);
  c.template store<kNtStore>(r);
}

// Device -> host: workgroup b takes chunks b, b + gridDim.x, ...
__global__ void __launch_bounds__(kThreads)
state_suspend_kernel(const char* __restrict__ src, char* __restrict__ dst, tsattn::CopyList list) {
  constexpr int kVectors = tsattn::kCopyChunkBytes / (kThreads * 16);
  const int64_t chunks = list.first_chunk[list.n];
  int64_t i = blockIdx.x;
  if (i >= chunks) return;
  u32x4 r[kVectors], ahead[kVectors];
  Chunk<kVectors> c(src, dst, list, i);
  c.template load<false>(r);
  for (i += gridDim.x; i < chunks; i += gridDim.x) {
    const Chunk<kVectors> next(src, dst, list, i);
    next.template load<false>(ahead);
    c.template store<true>(r);
    c = next;
#pragma unroll
    for (int u = 0; u < kVectors; ++u) r[u] = ahead[u];
  }
  c.template store<true>(r);
}

}  // namespace tsstate

namespace tsattn {

hipError_t launch_state_copy(const void* src, void* dst, const CopyList& list, bool src_host,
                             bool dst_host, hipStream_t st) {
  const int64_t chunks = list.first_chunk[list.n];
  if (chunks <= 0) return hipSuccess;
  constexpr int kSmall = kCopyChunkBytes / (tsstate::kThreads * 16);
  constexpr int kLarge = kHostReadChunkBytes / (tsstate::kThreads * 16);
  const dim3 block(tsstate::kThreads);
  const char* s = (const char*)src;
  char* d = (char*)dst;
  if (dst_host && !src_host) {
    hipLaunchKernelGGL(tsstate::state_suspend_kernel,
                       dim3((unsigned)(chunks < tsstate::kWalkers ? chunks : tsstate::kWalkers)), block,
                       0, st, s, d, list);
    return hipGetLastError();
  }
  auto kern = src_host ? (dst_host ? tsstate::state_copy_kernel<kLarge, true, true>
                                   : tsstate::state_copy_kernel<kLarge, true, false>)
              : bypass_caches(chunks * kCopyChunkBytes) ? tsstate::state_copy_kernel<kSmall, true, true>
                                                        : tsstate::state_copy_kernel<kSmall, false, false>;
  // a grid holds fewer than 2^32 threads: 2^23 chunks a launch, 128 GiB of 16 KiB ones
  constexpr int64_t kLaunch = (int64_t)1 << 23;
  for (int64_t first = 0; first < chunks; first += kLaunch) {
    hipLaunchKernelGGL(kern, dim3((unsigned)(chunks - first < kLaunch ? chunks - first : kLaunch)), block, 0,
                       st, s, d, list, first);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace tsattn
