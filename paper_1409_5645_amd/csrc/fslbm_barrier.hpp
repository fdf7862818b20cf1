// Barriers of kernels whose workgroups wait for one another.  A workgroup may
// wait for those only that are on the device: nothing says that a whole grid
// gets there at once (other streams and processes have kernels of this kind
// too, and each may hold part of the device).  So a kernel first forms a team of
// the workgroups that have started, within a bounded wait, and goes on with
// these; one that starts later finds the team closed and exits.  With a team of
// one the kernel's work is done by one workgroup.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fslbm {

// Waits until the wavefront's stores have reached the L2 (every memory access
// before it in the program comes before it).
__device__ __forceinline__ void drain_stores() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); }

// A launch has BAR_WORDS words, zero at its start: the barrier's (GridBarrier)
// and, TEAM_WORD further, the team's.
constexpr int BAR_WORDS = 2, TEAM_WORD = 1;
// Looks of a team's first workgroup at the number of arrivals before it closes
// the team, each some tenths of a microsecond after the last: a grid that finds
// room starts well within one look.
constexpr int TEAM_WAIT = 256;

struct Team {
  unsigned rank, size;  // size 0: the workgroup is not in it and exits
};

// Every workgroup of the launch that is to do the work calls this once.  The
// word's low half counts arrivals, its upper half is the team's size from the
// moment it is closed.  The first workgroup to arrive closes it: at `most`
// arrivals, or after `wait` looks with those that have arrived.  It calls before
// just ahead of that (thread 0; stores of its own that the team is to see).
// The ranks are the order of arrival (that of the launch in its place: 20^3 cells
// FP32 with conversions 15.9 -> 16.8 us a step).
template <class B>
__device__ __forceinline__ Team join_team(unsigned long long* word, unsigned most, int wait, B before) {
  __shared__ Team mine;
  if (threadIdx.x == 0) {
    Team t{0u, 0u};
    unsigned long long v = __hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    t.rank = (unsigned)v;
    if ((v >> 32) == 0ull && t.rank < most) {
      if (t.rank == 0u) {
        before();
        v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int look = 0; look < wait && (unsigned)v < most; ++look) {
          __builtin_amdgcn_s_sleep(1);
          v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        for (;;) {  // (a second time only where another workgroup has arrived meanwhile)
          t.size = min((unsigned)v, most);
          const unsigned long long w = atomicCAS(word, v, v | (unsigned long long)t.size << 32);
          if (w == v) break;
          v = w;
        }
      } else {
        while (((v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> 32) == 0ull)
          __builtin_amdgcn_s_sleep(1);
        t.size = (unsigned)(v >> 32);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      }
    }
    mine = t;
  }
  __syncthreads();
  // (the same in every thread: scalar registers)
  return Team{(unsigned)__builtin_amdgcn_readfirstlane((int)mine.rank),
              (unsigned)__builtin_amdgcn_readfirstlane((int)mine.size)};
}

// Barrier of a team on one counter (zero at launch): the low word counts
// arrivals, the upper two 16-bit fields the flags raised at even and at odd
// barriers (a workgroup that is ahead can be at most one barrier on, so it
// cannot disturb the field that a late one still reads; RESIDENT_STEPS steps of
// at most 64 workgroups fit a field).  Returns whether any workgroup raised its
// flag.
struct GridBarrier {
  unsigned long long* p;
  Team team;
  unsigned target, seen0, seen1;  // values of the fields last seen
  bool odd;
  __device__ GridBarrier(unsigned long long* q, Team t) : p(q), team(t), target(0), seen0(0), seen1(0), odd(false) {}
  __device__ bool meet(bool flag) {
    __shared__ unsigned long long got;
    // Every wavefront waits for its stores to reach the L2 its workgroup
    // shares; one lane then writes that L2 back, and invalidates the caches
    // for the workgroup afterwards (a write-back by every wavefront cost four
    // times the barrier itself).
    drain_stores();
    const int any = __syncthreads_or(flag ? 1 : 0);
    if (threadIdx.x == 0) {
      const unsigned long long add = 1ull + (any ? (odd ? 1ull << 48 : 1ull << 32) : 0ull);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      __hip_atomic_fetch_add(p, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      target += team.size;
      asm("" : "+v"(target));
      unsigned long long v;
      while ((unsigned)(v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < target)
        __builtin_amdgcn_s_sleep(1);
      got = v;
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    const unsigned now = (unsigned)(got >> (odd ? 48 : 32)) & 0xffffu;
    const bool raised = __builtin_amdgcn_readfirstlane((int)(now != (odd ? seen1 : seen0))) != 0;
    seen0 = odd ? seen0 : now;
    seen1 = odd ? now : seen1;
    asm("" : "+v"(seen0), "+v"(seen1));  // (vector registers: the kernels spill scalar ones)
    odd = !odd;
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
