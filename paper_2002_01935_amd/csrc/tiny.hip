// Small-contraction kernel: one workgroup runs one group of connected small
// contractions (tables: tiny.h) with every intermediate in LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstring>

#include "kernels.h"
#include "plan.h"

namespace tn {

#define GMEM __attribute__((address_space(1)))
#define CMEM __attribute__((address_space(4)))
#define TN_WAVE_SYNC() __builtin_amdgcn_wave_barrier()
// A value the same in every lane of the wavefront, made known to the compiler as such.
#define TN_UNIFORM(x) __builtin_amdgcn_readfirstlane(x)

#include "rowops.h"

#include "tiny_kernel.h"

template <int BYTES>
struct alignas(16) TinyArg {
  Ctx ctx;
  char pad[(64 - sizeof(Ctx) % 64) % 64];
  char blob[BYTES];
};

// One workgroup per group and in-flight slice.  Bound by latency: a chain of
// launch, table and operand loads, then about 1 us per level of the group (LDS
// reads and a barrier), against 4.4 us and more per contraction as launches of
// their own (95 % of a circuit's contractions, in trees 10 to 15 levels deep).
// Whole calls on MI355X, before and after: 122 contractions of a 3 x 3 circuit
// 332 -> 95 us, 509 of a 5 x 6 circuit with gradients 12.7 -> 4.75 ms, a
// random graph of 120 tensors 2.10 -> 1.15 ms.  The tables travel as a kernel
// argument: a captured graph keeps them in its own memory, so a replay uploads
// nothing and the caller's workspace holds none of them.
template <typename T, int BYTES>
__global__ __launch_bounds__(512) void tiny_tree_kernel(TinyArg<BYTES> arg) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int z = blockIdx.y;
  const int64_t sid = slice_id(arg.ctx, z);
  if (sid < 0) return;
  // the argument is read in place, in the kernel argument segment
  const uint64_t blob = reinterpret_cast<uint64_t>(__builtin_amdgcn_kernarg_segment_ptr()) + offsetof(TinyArg<BYTES>, blob);
  tiny_group<T>(arg.ctx, blob, blockIdx.x, z, sid, smem);
}

template <typename T, int BYTES>
static hipError_t launch_tiny_n(const Ctx& ctx, const TinyLaunch& L, hipStream_t s) {
  TinyArg<BYTES> arg;
  arg.ctx = ctx;
  std::memcpy(arg.blob, L.blob.data(), L.blob.size());
  hipLaunchKernelGGL((tiny_tree_kernel<T, BYTES>), dim3(L.n_groups, ctx.n_batch), dim3(L.threads), L.lds_bytes, s, arg);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_tiny_t(const Ctx& ctx, const TinyLaunch& L, hipStream_t s) {
  if (L.blob.size() <= kTinyBlobSmall) return launch_tiny_n<T, kTinyBlobSmall>(ctx, L, s);
  if (L.blob.size() <= kTinyBlobMid) return launch_tiny_n<T, kTinyBlobMid>(ctx, L, s);
  if (L.blob.size() <= kTinyBlobLarge) return launch_tiny_n<T, kTinyBlobLarge>(ctx, L, s);
  return hipErrorInvalidValue;
}

// Gradient copies of small leaves, a wavefront per 64 values (blockIdx.y): the
// in-flight slices are added one after another, so the sum does not depend on
// how many there are.  That chain, about 0.5 us per slice, is the time of the
// launch: one wavefront per leaf, walking its values too, took 128 us for 16
// slices of leaves of 2^10 values, 8 us now.
template <typename T, int BYTES>
__global__ __launch_bounds__(64) void scatter_kernel(TinyArg<BYTES> arg) {
  using V = typename C2<T>::t;
  const Ctx& ctx = arg.ctx;
  const uint64_t blob = reinterpret_cast<uint64_t>(__builtin_amdgcn_kernarg_segment_ptr()) + offsetof(TinyArg<BYTES>, blob);
  const ScatterEntry e = cload(reinterpret_cast<CMEM const ScatterEntry*>(blob) + blockIdx.x);
  const uint64_t base = reinterpret_cast<CMEM const uint64_t*>(ctx.ws + ctx.ptrtab_off)[e.slot];
  const uint32_t i = blockIdx.y * 64 + threadIdx.x;
  if (i < (1u << e.n_bits)) {
    uint32_t at = 0;
#pragma unroll
    for (int j = 0; j < 10; j++)
      if (j < e.n_bits) at |= ((i >> j) & 1u) << e.pos[j];
    for (int z = 0; z < ctx.n_batch; z++) {
      const int64_t sid = slice_id(ctx, z);
      if (sid < 0) continue;
      uint64_t off = 0;
#pragma unroll
      for (int j = 0; j < kMaxSliceTerms; j++)
        if (j < e.n_slice) off |= uint64_t((sid >> e.slice_bit[j]) & 1) << e.slice_pos[j];
      const V s = ld(reinterpret_cast<GMEM const V*>(ctx.ws + ctx.arena_off + uint64_t(z) * ctx.arena_stride + 256 * uint64_t(e.src)) + i);
      GMEM V* D = reinterpret_cast<GMEM V*>(base) + off + at;
      V v = ld(D);
      v.x += s.x;
      v.y += s.y;
      st(D, v);
    }
  }
}

template <typename T, int BYTES>
static hipError_t launch_scatter_n(const Ctx& ctx, const TinyLaunch& L, hipStream_t s) {
  TinyArg<BYTES> arg;
  arg.ctx = ctx;
  std::memcpy(arg.blob, L.blob.data(), L.blob.size());
  int bits = 0;
  for (uint32_t g = 0; g < L.n_groups; g++) {
    ScatterEntry e;
    std::memcpy(&e, L.blob.data() + g * sizeof e, sizeof e);
    bits = std::max(bits, (int)e.n_bits);
  }
  hipLaunchKernelGGL((scatter_kernel<T, BYTES>), dim3(L.n_groups, 1u << std::max(0, bits - 6)), dim3(64), 0, s, arg);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_scatter_t(const Ctx& ctx, const TinyLaunch& L, hipStream_t s) {
  if (L.blob.size() <= kTinyBlobSmall) return launch_scatter_n<T, kTinyBlobSmall>(ctx, L, s);
  if (L.blob.size() <= kTinyBlobLarge) return launch_scatter_n<T, kTinyBlobLarge>(ctx, L, s);
  return hipErrorInvalidValue;
}

hipError_t launch_scatter(const Ctx& ctx, const TinyLaunch& L, bool f64, hipStream_t s) {
  if (L.n_groups == 0) return hipErrorInvalidValue;
  return f64 ? launch_scatter_t<double>(ctx, L, s) : launch_scatter_t<float>(ctx, L, s);
}

// Zeroes arrays of the pointer table, one workgroup each: words[i] 8-byte
// words at slot first + i.
struct ZeroArg {
  uint64_t ptrtab;
  uint32_t first, pad;
  uint32_t words[kZeroArrays];
};
__global__ __launch_bounds__(256) void zero_kernel(ZeroArg arg) {
  GMEM uint64_t* p = reinterpret_cast<GMEM uint64_t*>(reinterpret_cast<CMEM const uint64_t*>(arg.ptrtab)[arg.first + blockIdx.x]);
  const uint32_t n = arg.words[blockIdx.x];
  for (uint32_t i = threadIdx.x; i < n; i += 256) p[i] = 0;
}

hipError_t launch_zero(const Ctx& ctx, int first_slot, const uint32_t* words, int n, hipStream_t s) {
  if (n < 1 || n > kZeroArrays) return hipErrorInvalidValue;
  ZeroArg arg;
  std::memset(&arg, 0, sizeof arg);
  arg.ptrtab = ctx.ws + ctx.ptrtab_off;
  arg.first = (uint32_t)first_slot;
  std::memcpy(arg.words, words, sizeof(uint32_t) * (size_t)n);
  hipLaunchKernelGGL(zero_kernel, dim3(n), dim3(256), 0, s, arg);
  return hipGetLastError();
}

hipError_t launch_tiny(const Ctx& ctx, const TinyLaunch& L, bool f64, hipStream_t s) {
  if (L.n_groups == 0 || L.threads > 512 || L.lds_bytes > 65536) return hipErrorInvalidValue;
  return f64 ? launch_tiny_t<double>(ctx, L, s) : launch_tiny_t<float>(ctx, L, s);
}

}  // namespace tn
