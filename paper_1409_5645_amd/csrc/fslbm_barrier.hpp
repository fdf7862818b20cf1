// Barriers of kernels whose workgroups wait for one another.  Such a kernel's
// grid has to be on the device as a whole: each keeps to a few workgroups, a
// fraction of the 256 compute units, so that several of them (one per hardware
// queue) fit beside one another, and all other work on the device ends.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fslbm {

// Waits until the wavefront's stores have reached the L2 (every memory access
// before it in the program comes before it).
__device__ __forceinline__ void drain_stores() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); }

// Barrier of the whole grid on one counter (zero at launch): the low word
// counts arrivals, the upper two 16-bit fields the flags raised at even and at
// odd barriers (a workgroup that is ahead can be at most one barrier on, so it
// cannot disturb the field that a late one still reads; RESIDENT_STEPS steps of
// at most 64 workgroups fit a field).  Returns whether any workgroup raised its
// flag.
struct GridBarrier {
  unsigned long long* p;
  unsigned target, index, seen[2];
  __device__ explicit GridBarrier(unsigned long long* q) : p(q), target(0), index(0), seen{0, 0} {}
  __device__ bool meet(bool flag) {
    __shared__ unsigned long long got;
    // Every wavefront waits for its stores to reach the L2 its workgroup
    // shares; one lane then writes that L2 back, and invalidates the caches
    // for the workgroup afterwards (a write-back by every wavefront cost four
    // times the barrier itself).
    drain_stores();
    const int any = __syncthreads_or(flag ? 1 : 0);
    const unsigned field = index & 1u;
    target += gridDim.x;
    if (threadIdx.x == 0) {
      const unsigned long long add = 1ull + (any ? (field ? 1ull << 48 : 1ull << 32) : 0ull);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      __hip_atomic_fetch_add(p, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      unsigned long long v;
      while ((unsigned)(v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < target)
        __builtin_amdgcn_s_sleep(1);
      got = v;
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    const unsigned now = (unsigned)(got >> (field ? 48 : 32)) & 0xffffu;
    const bool raised = now != seen[field];
    seen[field] = now;
    ++index;
    return raised;
  }
};

// Barrier of one workgroup between passes whose data goes through memory: the
// stores have reached the L2, and nothing older than them is read from the
// vector cache after it.
__device__ __forceinline__ void block_meet() {
  drain_stores();
  __syncthreads();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// A value that other workgroups add to.
__device__ __forceinline__ int peek(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace fslbm
