// A value handed from one workgroup to another while both run: 16 bytes of device memory that carry it and a tag.
//
// The value is published as two agent-scope atomic words (value bits, value bits XOR tag); a reader polls the slots it needs
// until both words of the present exchange have landed.  Tags are made of a number that no other launch of the process has
// (dsbd_launch_nonce), so nothing an earlier launch left in the memory passes for a value of this one and nobody clears it.
// A launch that a graph replays repeats its arguments, tags included: such launches need something else to tell them apart.
#pragma once
#include "common.h"

struct Slot { unsigned long long w0, w1; };

__host__ __device__ __forceinline__ unsigned long long exchange_tag(unsigned long long epoch) {
  return epoch * 0x9E3779B97F4A7C15ull;
}

__device__ __forceinline__ void slot_post(Slot* s, double v, unsigned long long tag) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  __hip_atomic_store(&s->w0, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(&s->w1, b ^ tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits until the slot carries the tag; gives up after `limit` ticks of the wall clock (returns false).
__device__ __forceinline__ bool slot_wait(Slot* s, unsigned long long tag, double& v, long long limit) {
  long long t0 = 0;
  for (int spin = 0;; ++spin) {
    const unsigned long long w0 = __hip_atomic_load(&s->w0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long w1 = __hip_atomic_load(&s->w1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((w0 ^ w1) == tag) { v = __longlong_as_double((long long)w0); return true; }
    if (spin == 0) t0 = wall_clock64();
    else if ((spin & 15) == 0 && wall_clock64() - t0 > limit) return false;
    __builtin_amdgcn_s_sleep(1);
  }
}

// The same for two slots at once (their loads in flight together).
__device__ __forceinline__ bool slot_wait2(Slot* s0, Slot* s1, unsigned long long tag, double& v0, double& v1, long long limit) {
  long long t0 = 0;
  bool h0 = false, h1 = false;
  for (int spin = 0;; ++spin) {
    unsigned long long a0 = 0, a1 = 0, b0 = 0, b1 = 0;
    if (!h0) { a0 = __hip_atomic_load(&s0->w0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); a1 = __hip_atomic_load(&s0->w1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    if (!h1) { b0 = __hip_atomic_load(&s1->w0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); b1 = __hip_atomic_load(&s1->w1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    if (!h0 && (a0 ^ a1) == tag) { v0 = __longlong_as_double((long long)a0); h0 = true; }
    if (!h1 && (b0 ^ b1) == tag) { v1 = __longlong_as_double((long long)b0); h1 = true; }
    if (h0 && h1) return true;
    if (spin == 0) t0 = wall_clock64();
    else if ((spin & 15) == 0 && wall_clock64() - t0 > limit) return false;
    __builtin_amdgcn_s_sleep(1);
  }
}
