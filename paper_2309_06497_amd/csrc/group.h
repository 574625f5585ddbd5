// Launches that serve several buckets of blocks at once.
//
// A parameter set whose sizes the block size does not divide has up to a dozen buckets (blocks of equal shape), most of them
// with few blocks: one launch per bucket and stage leaves the GPU idle for most of a launch and costs the host a few
// microseconds each.  Buckets do not depend on one another, so every stage is one launch for all of them: the kernel's
// arguments are a table with one entry per bucket, a workgroup finds its entry by its index and works on it as if it were
// alone.  A step, bucket by bucket and so: three transformer layers of 1000 in blocks of 512 (ten buckets), filtered bf16
// gradients, 2245 and 1200 us; one layer of 331 in blocks of 1024 (five), float32 gradients, 2078 and 624 us; ResNet-50 with
// convolution tensors 1130 and 890 us.  One bucket alone: the same time.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <algorithm>

namespace shampoo {

// entries in a launch: what fits the 4 KB of a kernel's arguments beside RESERVE bytes of others
template <typename Args, int RESERVE = 0> constexpr int group_max() { return std::min<int>(32, (4096 - 16 - RESERVE) / ((int)sizeof(Args) + 4) - 1); }

template <typename Args, int RESERVE = 0> struct Group {
  int32_t count;
  int32_t first[group_max<Args, RESERVE>()];    // first workgroup of an entry (a multiple of 8: the XCD of a workgroup is its index modulo 8)
  Args a[group_max<Args, RESERVE>()];
};

// The compiler knows that a pointer among a kernel's arguments is one to global memory, but not of one that it finds by an
// index; loads and stores through it would be flat ones, which also wait for LDS.
template <typename T> __device__ __forceinline__ void to_global(T *&p) {
  p = (T *)(__attribute__((address_space(1))) T *)reinterpret_cast<uintptr_t>(p);
}
// the same of a pointer that comes out of a table in memory
template <typename T> __device__ __forceinline__ T *global_ptr(const void *p) {
  T *q = (T *)const_cast<void *>(p);
  to_global(q);
  return q;
}
template <typename T, typename... Rest> __device__ __forceinline__ void to_global(T *&p, Rest *&...rest) { to_global(p); to_global(rest...); }

// Between accesses to memory by lanes of one wavefront that depend on one another: the memory keeps their order by itself, the compiler must.
// No instruction.
__device__ __forceinline__ void wavefront_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The entry of this workgroup, and its index among the entry's workgroups.  A copy, read once: what stays behind a
// reference is read again wherever it is used.  The first entry is requested together with the count, so that a launch for one
// bucket starts after one round trip.
template <typename Args, int RESERVE> __device__ __forceinline__ Args group_pick(const Group<Args, RESERVE> &g, int &wg) {
  Args a = g.a[0];
  int k = 0;
  while (k + 1 < g.count && (int)blockIdx.x >= g.first[k + 1]) ++k;
  if (k > 0) a = g.a[k];
  wg = (int)blockIdx.x - (k > 0 ? g.first[k] : 0);
  a.globals();
  return a;
}

}  // namespace shampoo
