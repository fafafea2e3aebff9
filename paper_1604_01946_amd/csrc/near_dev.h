// Device-side helpers of the kernels whose workgroups exchange values that are their own flags (persistent_tiny.hip,
// persistent_near_fwd.hip, persistent_near_bwd.hip): an exchange slot holds the empty pattern until it is written, once, and whoever needs it reads it until no
// word shows the pattern any more.
#pragma once
#include "persistent_dev.h"

namespace lstm {
namespace {

constexpr unsigned kEmpty = 0xFFFFFFFFu;  // "not written yet": a NaN that arithmetic never produces, and the largest word

__device__ __forceinline__ float poll_load(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// near: every reader is on this XCD, whose L2 is as far as the value has to go
__device__ __forceinline__ void publish(float* p, float v, bool near) {
  unsigned b = __float_as_uint(v);
  if (b == kEmpty) b = 0x7FC00000u;
  if (near) __hip_atomic_store(reinterpret_cast<unsigned*>(p), b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else __hip_atomic_store(reinterpret_cast<unsigned*>(p), b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Four words of a slot of n floats at a wave-uniform address, for values that another XCD writes.
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uintx4 remote_load4(const float* p, int n, int at) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), (short)0, 4 * n, 0x00020000);
  asm volatile("" ::: "memory");  // (asked for again, it is read again)
  return __builtin_amdgcn_raw_buffer_load_b128(r, 4 * at, 0, 16);  // sc1: as an agent-scope load
}

// True in every lane if `v` is true in every lane of the wave (the wave is whole), as a scalar.
__device__ __forceinline__ bool every_lane(bool v) { return __builtin_amdgcn_ballot_w64(!v) == 0; }

// 16 bytes at float `at` of a slot of n floats.  sc1: as an agent-scope load, which sees what other CUs have written.
template <bool SC1>
__device__ __forceinline__ floatx4 slot_load4(const float* slot, int n, int at) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(slot), (short)0, 4 * n, 0x00020000);
  return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, 4 * at, 0, SC1 ? 16 : 0));
}
// The largest word of a number of 16-byte pieces: kEmpty if any of them is.  (Two instructions a piece.)
__device__ __forceinline__ unsigned umax3(unsigned a, unsigned b, unsigned c) { return max(max(a, b), c); }
__device__ __forceinline__ unsigned top4(floatx4 v, unsigned m) {
  return umax3(umax3(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2])), __float_as_uint(v[3]), m);
}
__device__ __forceinline__ float canonical(float v) { return __float_as_uint(v) == kEmpty ? __uint_as_float(0x7FC00000u) : v; }
// near: plain stores, which end in the L2 that the readers share; else through it to memory
__device__ __forceinline__ void slot_store4(float* slot, int n, int at, floatx4 v, bool near) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(slot, (short)0, 4 * n, 0x00020000);
  const uintx4 b = __builtin_bit_cast(uintx4, floatx4{canonical(v[0]), canonical(v[1]), canonical(v[2]), canonical(v[3])});
  if (near) __builtin_amdgcn_raw_buffer_store_b128(b, r, 4 * at, 0, 0);
  else __builtin_amdgcn_raw_buffer_store_b128(b, r, 4 * at, 0, 16);
}
__device__ __forceinline__ void slot_store1(float* slot, int n, int at, float v, bool near) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(slot, (short)0, 4 * n, 0x00020000);
  const unsigned b = __float_as_uint(canonical(v));
  if (near) __builtin_amdgcn_raw_buffer_store_b32(b, r, 4 * at, 0, 0);
  else __builtin_amdgcn_raw_buffer_store_b32(b, r, 4 * at, 0, 16);
}

// Polls: one round after the other, without a pause (backward, L = 1, H = 256, T = 500: none 0.56 ms, 128 cycles before the first
// round 0.57, 256 0.60, 512 0.66).  What a round costs grows with the bytes that all waves together ask for, so the waves of a
// workgroup poll a share of the slot each and hand the shares to each other through LDS.
struct NearWaiter {
  int* watchdog;
  int limit;
  bool dead;
  __device__ __forceinline__ bool give_up(int& spins) {
    if (dead) return true;
    if (++spins > limit) {
      dead = true;
      __hip_atomic_store(watchdog, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      return true;
    }
    return false;
  }
  // One value per lane.
  __device__ __forceinline__ float poll1(const float* p) {
    int spins = 0;
    while (true) {
      const float v = poll_load(p);
      if (__all(__float_as_uint(v) != kEmpty) || give_up(spins)) return v;
    }
  }
};

// Whether all workgroups of a group run on one XCD: each leaves its XCD's number in the group's table (a word per member, at most
// 64, the empty pattern before the launch) and reads the others'.  All read the same words, so all come to the same answer.
__device__ __forceinline__ void leave_xcd(float* table, int member, int lane) {
  if (lane == 0) publish(table + member, __int_as_float(xcd_id()), false);
}
__device__ __forceinline__ bool all_on_one_xcd(NearWaiter& w, const float* table, int members, int lane) {
  const float v = w.poll1(table + (lane < members ? lane : 0));
  return __all(__float_as_int(v) == xcd_id());
}

}  // namespace
}  // namespace lstm
