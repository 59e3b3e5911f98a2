// Which of several workgroups that share a piece of work ends last, without a launch that clears a counter first.
//
// A counter is 64 bits in the caller's workspace, which may hold anything: the number of the call, which no other call of the
// process has (56 bits, next_call), above 8 bits that count arrivals.  At its start a workgroup puts the number there if it finds 0, and waits for
// nothing; when it has written what it leaves for the others it adds one.  Only where neither 0 nor the call's number stood
// there (a workspace's first use) does it put the number there before.  An exchange that fails means that another workgroup of
// the call was first, so none is tried twice and nothing ever waits.  The last to arrive leaves 0, which is what the next call,
// or the next replay of a captured one, finds.  That what a workspace holds by chance is the number of a call has a likelihood
// of 2^-56 a counter.
//
// What is left for others, and what the last one reads of it, goes past the caches of one die: stores and loads at agent scope,
// and a workgroup arrives when its stores are acknowledged.  (A release at agent scope in their place writes back all that the
// die's L2 holds.)  Counters that were compared and exchanged until it succeeded cost as many round trips as workgroups met:
// 32 units of 64 tiles in 8 parts 14.3 us, 7.9 so.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rlda {

uint64_t next_call();                                        // a number that no other call of the process has, of any operation

namespace {

constexpr int MAX_ARRIVALS = 255;

// by one thread, at the start; the result goes to arrive()
__device__ __forceinline__ uint64_t claim(uint64_t* counter, uint64_t call) {
  uint64_t seen = 0;
  __hip_atomic_compare_exchange_strong(counter, &seen, call << 8, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return seen;
}
// by the same thread, after a barrier that follows stores_done() of all threads: whether it is the last of n
__device__ __forceinline__ bool arrive(uint64_t* counter, uint64_t call, uint64_t seen, int n) {
  if (seen != 0 && seen >> 8 != call)
    __hip_atomic_compare_exchange_strong(counter, &seen, call << 8, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const bool last = (int)(__hip_atomic_fetch_add(counter, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 255) + 1 == n;
  if (last) __hip_atomic_store(counter, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return last;
}
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// a pair of floats for others
__device__ __forceinline__ void put(uint64_t* p, float x, float y) {
  __hip_atomic_store(p, (uint64_t)__float_as_uint(y) << 32 | __float_as_uint(x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 get(const uint64_t* p) {
  const uint64_t v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}

}  // namespace
}  // namespace rlda
