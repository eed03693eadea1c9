// Step barriers of the XCD-local recurrence kernels: the check that a block's
// workgroups share one XCD, the signal and the wait within it, and the
// schedule's active counts (see lstm_xcd.hip for the design).
#pragma once

#include "am_device.h"
#include "am_internal.h"
#include "poll_budget.h"

namespace am {
namespace {

constexpr int NX = 8;                    // XCDs
constexpr unsigned SPIN_LIMIT = 1u << 22;

__device__ __forceinline__ unsigned xcc_id() {
  unsigned v;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(v));
  return v & 0xfu;
}

// One-time check that the workgroups of this block share one XCD: each
// publishes its XCD (+1; the launch's sync slot starts zeroed) in its word
// of the block's line, and one wave waits for all members and compares.
// Only the block's members take part, with plain device-scope loads and
// stores: no read-modify-write, no cache write-back or invalidation.  Every
// member of a block returns the same answer; y.fenced forces the fenced
// exchange regardless (so that tests can run it).
__device__ bool check_local(const XcdSync& y, int blk, int us, int members, int* bad_sh) {
  unsigned* line = reinterpret_cast<unsigned*>(y.xcc) + blk * 32;
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    if (lane == 0) __hip_atomic_store(line + us, xcc_id() + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned v = 0, spins = 0;
    for (;;) {
      v = lane < members ? __hip_atomic_load(line + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 1u;
      if (__all(v != 0)) break;
      if (++spins > SPIN_LIMIT) {
        if (lane == 0) __hip_atomic_store(y.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
      __builtin_amdgcn_s_sleep(2);
    }
    const unsigned first = __shfl(v, 0, 64);
    const bool bad = __any(lane < members && v != first);
    if (lane == 0) *bad_sh = bad || y.fenced ? 1 : 0;
  }
  __syncthreads();
  return *bad_sh == 0;
}

// One poll of a flag word from the XCD's L2: a non-temporal load, which
// does not keep the line in the CU's L1 (an agent-coherent load, sc1, goes
// past the L2 to memory).
__device__ __forceinline__ unsigned poll_l2(const unsigned* p) {
  unsigned v;
  asm volatile("global_load_dword %0, %1, off nt\n\ts_waitcnt vmcnt(0)" : "=v"(v) : "v"(p) : "memory");
  return v;
}

// This workgroup's stores of the step have completed: publish its count of
// completed steps in its own word of the block's flag line (one 128-byte
// line of 32 words, word us for member us).  The store reaches the XCD's L2
// after the data stores it follows have completed there, so a poller that
// sees the count then reads the data from L2.  When a block spans XCDs the
// store is device-scope (it goes on to memory) after a release fence (a
// write-back of this XCD's L2); within one XCD the word stays in the L2,
// where the polls read it (a device-scope access would go past the L2 to
// memory: 1.5-3 % slower recurrences).
// Separate words need no atomic read-modify-write, which the L2 would
// serialise over the block's members.
__device__ __forceinline__ void xsignal(const XcdSync& y, bool local, int blk, int us,
                                        unsigned count) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    if (local) {
      __hip_atomic_store(y.flags + blk * 32 + us, count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    } else {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      __hip_atomic_store(y.flags + blk * 32 + us, count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// Wait until every member of the block has published a count >= target.
// Wave `poller` polls: lane m < members reads member m's word (one request
// for the line; from the XCD's L2 with a non-temporal load, or with a
// device-scope load when the block spans XCDs) and the wave votes.  The other workgroups' exchanged rows are then read from
// the shared L2 (local) or after an acquire that invalidates this CU's
// caches (block spans XCDs).  Each poll waits for every load its wave has
// in flight, so the poller should be a wave with none outstanding.
__device__ __forceinline__ void xwait(const XcdSync& y, bool local, int blk, int members,
                                      unsigned target, int poller = 0) {
  if ((int)(threadIdx.x >> 6) == poller) {
    const int lane = threadIdx.x & 63;
    const unsigned* line = y.flags + blk * 32;
    unsigned spins = 0;
    for (;;) {
      const unsigned v = lane >= members ? target
                         : local ? poll_l2(line + lane)
                                 : __hip_atomic_load(line + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__all(v >= target)) break;
      if (++spins > SPIN_LIMIT) {
        if (lane == 0) __hip_atomic_store(y.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    if (!local) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  __syncthreads();
}

// Block of sequences served by this workgroup: workgroup i runs on XCD
// i % 8 and serves block i % 8 + 8 (i / 8 / members), so with two blocks per
// XCD both of them sit on the XCD of their workgroups.
__device__ __forceinline__ int xcd_block(int members) {
  return (int)(blockIdx.x % NX) + NX * (int)(blockIdx.x / NX / members);
}

// Sequences longer than t steps, from those at t - 1 (active_down) or t + 1
// (active_up), walked through the sorted lengths one load after another; or,
// COUNTS, read from ps.lens[t].
template <bool COUNTS = false>
__device__ __forceinline__ int active_down(const PersistSchedule& ps, int nb, int t) {
  if constexpr (COUNTS) return ps.lens[t];
  if (!ps.varlen) return ps.B;
  while (nb > 0 && (int)ps.lens[nb - 1] <= t) --nb;
  return nb;
}
template <bool COUNTS = false>
__device__ __forceinline__ int active_up(const PersistSchedule& ps, int nb, int t) {
  if constexpr (COUNTS) return ps.lens[t];
  if (!ps.varlen) return ps.B;
  while (nb < ps.B && (int)ps.lens[nb] > t) ++nb;
  return nb;
}

}  // namespace
}  // namespace am
