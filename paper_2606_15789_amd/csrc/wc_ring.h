#pragma once

// wc_ring.h -- decode steps of one LDS round trip, for launches of few 64-lane
// chunks.  Included by wc_decoder.h.
//
// Paper: Alg. 2 (slot = state mod 2^b, table lookup of (symbol, freq, cumfreq),
// state update f * floor(x / 2^b) + slot - cum, renormalisation from one
// interleaved word stream).
//
// What bounds such a launch: a wave's steps are one serial chain, and few chains
// leave the compute units idle.  A step that looks the table up, ballots the lanes
// that renormalise and then reads their words is two dependent LDS round trips:
// 72 ns when few waves share a compute unit (a loop of bare steps).  Here the
// words are table entries before a lane needs them, so a step is one round trip
// (45 ns): a lane's next entry lies at its slot's place in the table when it keeps
// its state, and at its word's place in a ring of entries when it takes a word.
//  * With x = (xn << 16) | w after renormalisation, the slot is w mod 2^12 and
//    floor(x / 2^12) = 16 xn + (w >> 12), so w's entry is
//    {16 f | symbol << 24, f (w >> 12) + slot - cum} with the multiplier xn itself,
//    where a table entry {f | symbol << 24, slot - cum} takes floor(x / 2^12): w is
//    not needed any more.  16 f <= 2^16 and xn < 2^16 fit the 24-bit multiply.
//  * Nothing but the address stands between an entry's arrival and the next read:
//    the multiplier is made while that entry is on its way.
//  * A second wave of the workgroup, the feeder, makes the entries: loads the
//    words, looks their table entries up and writes the ring, on issue slots that
//    are idle otherwise.  Done by the decoding wave itself this took 0.28 us per
//    256 words, a fifth of the 8B int4 layer's launch.

#include <hip/hip_runtime.h>

#include "wc_internal.h"

namespace {

// The ring: kRingEntries entries of 8 bytes, the first kMirror again past its end
// (a step reads at most 64 from its position on), then two counters, both in
// bytes of entries since the chunk's start: written by the feeder, and consumed.
constexpr uint32_t kRingEntries = 1024, kMirror = 64, kUnitEntries = 128;
constexpr uint32_t kRingBytes = 8 * kRingEntries, kUnitBytes = 8 * kUnitEntries;
constexpr uint32_t kRingWritten = kRingBytes + 8 * kMirror, kRingConsumed = kRingWritten + 4;
constexpr uint32_t kRingWaveBytes = kRingWritten + 16;
constexpr uint32_t kRingDone = 0xFFFFFFFFu;  // consumed: the chunk's decoder has left

typedef uint32_t ru2 __attribute__((ext_vector_type(2)));
typedef uint32_t ru4 __attribute__((ext_vector_type(4)));

// LDS by byte address (the low 32 bits of an LDS pointer).  The counters are
// accessed as volatile; a wave's LDS accesses are performed in order, so entries
// written before the counter are there for whoever has read it.
typedef __attribute__((address_space(3))) ru2 lds_u2;
typedef __attribute__((address_space(3))) ru4 lds_u4;
typedef __attribute__((address_space(3))) volatile uint32_t lds_counter;
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}
__device__ __forceinline__ ru2 lds_load2(uint32_t a) { return *(lds_u2*)(uintptr_t)a; }
__device__ __forceinline__ void lds_store4(uint32_t a, ru4 v) { *(lds_u4*)(uintptr_t)a = v; }
__device__ __forceinline__ uint32_t counter(uint32_t a) {
  return __builtin_amdgcn_readfirstlane(*(lds_counter*)(uintptr_t)a);
}
__device__ __forceinline__ void set_counter(uint32_t a, uint32_t v) {
  asm volatile("" ::: "memory");
  if (__lane_id() == 0) *(lds_counter*)(uintptr_t)a = v;
  asm volatile("" ::: "memory");
}

// m's lane bit ? a : b, as one v_cndmask on the mask the ballot left in scalar
// registers.
__device__ __forceinline__ uint32_t select(uint64_t m, uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(r) : "v"(b), "v"(a), "s"(m));
  return r;
}

// The decoding wave's side.
struct Ring {
  uint32_t ring;   // LDS address
  uint32_t cur;    // bytes of entries consumed
  uint32_t limit;  // the feeder is looked at when cur passes this
  ru2 e;           // this lane's next entry: {multiplicand | symbol << 24, addend}
  uint32_t h;      // and its multiplier
  uint32_t low;    // the state interval's lower end

  // Before the workgroup's barrier.
  __device__ __forceinline__ void reset() {
    set_counter(ring + kRingWritten, 0u);
    set_counter(ring + kRingConsumed, 0u);
  }

  // Tell the feeder how far the decode is and wait until the next two steps' 128
  // entries are there.  It ends: with less than a unit between the two counters
  // the feeder finds room for a unit and writes it (feed).
  __device__ __forceinline__ void wait() {
    set_counter(ring + kRingConsumed, cur);
    uint32_t written = counter(ring + kRingWritten);
    while (written - cur < kUnitBytes) {
      __builtin_amdgcn_s_sleep(1);
      written = counter(ring + kRingWritten);
    }
    limit = written - kUnitBytes;
    asm volatile("" ::: "memory");
  }
  // Every second step: they consume at most 128 entries.
  __device__ __forceinline__ void check() {
    if (__builtin_expect(cur > limit, 0)) wait();
  }

  // The first entries, and the lane's own, from its state x.
  __device__ __forceinline__ void start(uint32_t x) {
    low = wc::kStateLow;
    asm("" : "+s"(low));  // kept in its register
    cur = 0;
    wait();
    h = x >> wc::kProbBits;
    e = lds_load2((x & (wc::kTableSize - 1)) << 3);
  }

  // One step; returns the entry's low word (symbol in byte 3).  With kAll every
  // lane decodes a symbol; otherwise those with `active` set do, and the others
  // keep their state and get 0.
  template <bool kAll>
  __device__ __forceinline__ uint32_t step(bool active) {
    const uint32_t lo = e.x;
    const uint32_t xn = __umul24(e.x, h) + e.y;
    const uint32_t a = (xn & (wc::kTableSize - 1)) << 3;
    const bool need = (kAll || active) && xn < low;
    const uint64_t m = __ballot(need);
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
        (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    const uint32_t at = ring + (cur & (kRingBytes - 8u)) + 8u * rank;
    const uint32_t taken = (uint32_t)__popcll(m);
    asm("s_lshl3_add_u32 %0, %1, %0" : "+s"(cur) : "s"(taken) : "scc");
    if constexpr (kAll) {
      // the address first, the multiplier while its entry is read
      e = lds_load2(select(m, at, a));
      __builtin_amdgcn_sched_barrier(0);
      h = select(m, xn, xn >> wc::kProbBits);
      return lo;
    } else {
      const ru2 en = lds_load2(need ? at : a);
      e.x = active ? en.x : e.x;
      e.y = active ? en.y : e.y;
      h = active ? (need ? xn : xn >> wc::kProbBits) : h;
      return active ? lo : 0u;
    }
  }

  // The lane's state, from its next entry: a table entry (f, the symbol's
  // frequency) holds slot - cum, one from the ring (16 f) f (w >> 12) + slot - cum.
  __device__ __forceinline__ uint32_t state(uint32_t f, uint32_t cum) const {
    const bool ring_entry = (e.x & 0xFFFFFFu) != f;
    const uint32_t q = e.y / max(f, 1u);
    const uint32_t hi = ring_entry ? 16u * h + q : h;
    return (hi << wc::kProbBits) + cum + (ring_entry ? e.y - q * f : e.y);
  }

  // The decoding wave leaves: so does its feeder.
  __device__ __forceinline__ void done() { set_counter(ring + kRingConsumed, kRingDone); }
};

// The feeder: the words at byte `words` of the record rs to entries in the ring at
// LDS address `ring`, a unit of 128 words at a time, until the decoding wave has
// left (done, which it reaches after the chunk's steps or at once).  Loads run
// kAhead units ahead; past the record they give zeros.  build: the workgroup's
// table, with a barrier.
template <class Build>
__device__ __forceinline__ void feed(__amdgpu_buffer_rsrc_t rs, uint32_t words, uint32_t ring,
                                     uint32_t lane, Build build) {
  constexpr int kAhead = 8;
  uint32_t w[kAhead];
  uint32_t off = words + 4u * lane;
#pragma unroll
  for (int u = 0; u < kAhead; u++) {
    w[u] = __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
    off += 2u * kUnitEntries;
  }
  build();
  uint32_t written = 0;
  for (;;) {
#pragma unroll
    for (int u = 0; u < kAhead; u++) {
      const ru2 g0 = lds_load2((w[u] & 0xFFFu) << 3), g1 = lds_load2((w[u] >> 13) & 0x7FF8u);
      const ru4 v = {__umul24(g0.x, 15u) + g0.x, __umul24(g0.x, (w[u] >> 12) & 15u) + g0.y,
                     __umul24(g1.x, 15u) + g1.x, __umul24(g1.x, w[u] >> 28) + g1.y};
      w[u] = __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
      off += 2u * kUnitEntries;
      // room for the unit, once the decode has left its place in the ring
      for (;;) {
        const uint32_t consumed = counter(ring + kRingConsumed);
        if (consumed == kRingDone) return;
        if (written + kUnitBytes - consumed <= kRingBytes) break;
        __builtin_amdgcn_s_sleep(1);
      }
      const uint32_t at = ring + (written & (kRingBytes - 1u)) + 16u * lane;
      lds_store4(at, v);
      if ((written & (kRingBytes - 1u)) == 0 && lane < kMirror / 2) lds_store4(at + kRingBytes, v);
      written += kUnitBytes;
      set_counter(ring + kRingWritten, written);
    }
  }
}

}  // namespace
