#pragma once

// wc_ring.h -- decode steps of one LDS round trip, for 64-lane chunks of which few
// share a compute unit: decodes of few chunks (FedRing) and the shared fused GEMM
// (OwnRing).  Included by wc_decoder.h.
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
//  * Where the workgroup has waves to spare, a second wave, the feeder, makes the
//    entries (FedRing): loads the words, looks their table entries up and writes the
//    ring, on issue slots that are idle otherwise.  Done by the decoding wave itself
//    this took 0.28 us per 256 words, a fifth of the 8B int4 layer's launch.
//  * The shared fused GEMM's workgroup is full with eight waves that decode and eight
//    that multiply: there the decoding wave makes them itself (OwnRing).

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
__device__ __forceinline__ uint32_t lds_load1(uint32_t a) {
  return *(__attribute__((address_space(3))) uint32_t*)(uintptr_t)a;
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

// A lane's next entry and what it multiplies, and the step.
struct Entry {
  ru2 e;         // {multiplicand | symbol << 24, addend}
  uint32_t h;    // the multiplier
  uint32_t low;  // the state interval's lower end

  __device__ __forceinline__ void begin(uint32_t x) {
    low = wc::kStateLow;
    asm("" : "+s"(low));  // kept in its register
    h = x >> wc::kProbBits;
    e = lds_load2((x & (wc::kTableSize - 1)) << 3);
  }

  // One step; returns the entry's low word (symbol in byte 3).  The next word's
  // entry is at LDS address `at`; `words` gets 8 bytes for every word taken.  With
  // kAll every lane decodes a symbol; otherwise those with `active` set do, and
  // the others keep their state and get 0.
  template <bool kAll>
  __device__ __forceinline__ uint32_t step(bool active, uint32_t at, uint32_t& words) {
    const uint32_t lo = e.x;
    const uint32_t xn = __umul24(e.x, h) + e.y;
    const uint32_t a = (xn & (wc::kTableSize - 1)) << 3;
    const bool need = (kAll || active) && xn < low;
    const uint64_t m = __ballot(need);
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
        (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    const uint32_t word = at + 8u * rank;
    const uint32_t taken = (uint32_t)__popcll(m);
    asm("s_lshl3_add_u32 %0, %1, %0" : "+s"(words) : "s"(taken) : "scc");
    if constexpr (kAll) {
      // the address first, the multiplier while its entry is read
      e = lds_load2(select(m, word, a));
      __builtin_amdgcn_sched_barrier(0);
      h = select(m, xn, xn >> wc::kProbBits);
      return lo;
    } else {
      const ru2 en = lds_load2(need ? word : a);
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
};

// A unit of 128 words as entries, two a lane, from the lane's words w and their
// table entries: {16 f | symbol << 24, f (w >> 12) + slot - cum}.
__device__ __forceinline__ ru4 word_entries(uint32_t w, ru2 g0, ru2 g1) {
  return ru4{__umul24(g0.x, 15u) + g0.x, __umul24(g0.x, (w >> 12) & 15u) + g0.y,
             __umul24(g1.x, 15u) + g1.x, __umul24(g1.x, w >> 28) + g1.y};
}
__device__ __forceinline__ void word_lookups(uint32_t w, ru2& g0, ru2& g1) {
  g0 = lds_load2((w & 0xFFFu) << 3);
  g1 = lds_load2((w >> 13) & 0x7FF8u);
}

// The decoding wave's side of a ring that a feeder fills.
struct FedRing : Entry {
  uint32_t ring;   // LDS address
  uint32_t cur;    // bytes of entries consumed
  uint32_t limit;  // the feeder is looked at when cur passes this

  // Before the workgroup's barrier.
  __device__ __forceinline__ void open(uint32_t lds, __amdgpu_buffer_rsrc_t, ru4, uint32_t,
                                       uint32_t) {
    ring = lds;
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
  // After group j of two steps: the next two consume at most 128 entries.
  template <int j>
  __device__ __forceinline__ void check() {
    if (__builtin_expect(cur > limit, 0)) wait();
  }

  // The first entries, and the lane's own, from its state x.
  __device__ __forceinline__ void start(uint32_t x) {
    cur = 0;
    wait();
    begin(x);
  }

  template <bool kAll>
  __device__ __forceinline__ uint32_t next(bool active) {
    return step<kAll>(active, ring + (cur & (kRingBytes - 8u)), cur);
  }

  __device__ __forceinline__ uint32_t words() const { return cur / 8u; }

  // The decoding wave leaves: so does its feeder.
  __device__ __forceinline__ void close() { set_counter(ring + kRingConsumed, kRingDone); }
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
      ru2 g0, g1;
      word_lookups(w[u], g0, g1);
      const ru4 v = word_entries(w[u], g0, g1);
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

// A ring that its decoding wave fills itself, for workgroups with no waves to spare
// for feeders.  A unit is kBlocks blocks of 128 words (one load of a dword a lane
// each); the ring is two units long and its first unit is written a second time past
// its end, so p runs on without a wrap while a unit is read and goes back when the
// second unit is replaced.  Units pass four stages so that no commit waits for what
// it uses: memory -> LDS staging (loads straight to LDS, kStage units), staging ->
// registers, registers -> table entries, entries -> ring; each commit moves the
// units behind it one stage on.  Two blocks to a unit commit half as often, one leaves
// LDS for a second workgroup (the shared GEMM has both).
constexpr uint32_t kBlockWordBytes = 256, kBlockRing = 1024;

template <uint32_t kBlocks, uint32_t kStage>
struct OwnRing : Entry {
  static constexpr uint32_t kUnitRing = kBlockRing * kBlocks;
  static constexpr uint32_t kUnitWords = kBlockWordBytes * kBlocks;  // bytes
  static constexpr uint32_t kStaging = 3 * kUnitRing;                // offset of the staging
  static constexpr uint32_t kSlots = kStage * kUnitWords;
  static constexpr uint32_t kBytes = kStaging + kSlots;

  ru4 record;       // buffer descriptor of the chunk's record
  uint32_t ring;    // LDS address
  uint32_t ring_v;  // this lane's place in a block of the ring's first unit
  uint32_t lane4;   // and in a block of staged words
  uint32_t next_v;  // record offset of this lane's words of the next unit to load
  uint32_t p;       // LDS address of the next word's entry
  uint32_t thr;     // commit a unit when p passes this
  uint32_t wraps;   // times p went back to the ring's start
  uint32_t slot;    // staging offset of the unit after the next one to commit
  ru2 g[2 * kBlocks];                    // the next unit's table entries
  uint32_t w[kBlocks], wn[kBlocks];   // this lane's words (two a block) of the next
                                            // unit and of the one after
  uint32_t first[4 * kBlocks];           // the chunk's first four units

  // A staging offset below 2 kSlots, around the staging's end.
  __device__ static __forceinline__ uint32_t around(uint32_t x) {
    if constexpr ((kSlots & (kSlots - 1)) == 0) return x & (kSlots - 1);
    return x >= kSlots ? x - kSlots : x;
  }

  // The next unit's words to staging offset `to`; past the record they are zeros.
  // The loads have no destination register; the wave waits on vmcnt before it
  // reads the words (commit), and before it ends (close).
  __device__ __forceinline__ void stage(uint32_t to) {
#pragma unroll
    for (uint32_t b = 0; b < kBlocks; b++) {
      asm volatile("s_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                   :
                   : "{m0}"(ring + kStaging + to + b * kBlockWordBytes), "v"(next_v),
                     "s"(record)
                   : "memory");
      next_v += kBlockWordBytes;
    }
  }

  // Before the workgroup's barrier: the chunk's first words on their way, four
  // units to registers and the next kStage - 1 to staging.
  __device__ __forceinline__ void open(uint32_t lds, __amdgpu_buffer_rsrc_t rs, ru4 rec,
                                       uint32_t words_at, uint32_t lane) {
    ring = lds;
    record = rec;
    ring_v = ring + 16u * lane;
    lane4 = 4u * lane;
    next_v = words_at + lane4;
#pragma unroll
    for (uint32_t k = 0; k < 4 * kBlocks; k++)
      first[k] = __builtin_amdgcn_raw_buffer_load_b32(rs, next_v + k * kBlockWordBytes, 0, 0);
    next_v += 4 * kUnitWords;
#pragma unroll
    for (uint32_t u = 4; u < 3 + kStage; u++) stage((u * kUnitWords) % kSlots);
    slot = 4 * kUnitWords % kSlots;
  }

  __device__ __forceinline__ void lookups() {
#pragma unroll
    for (uint32_t b = 0; b < kBlocks; b++) word_lookups(w[b], g[2 * b], g[2 * b + 1]);
  }

  // Units 0 and 1 into the ring, the next ones into their stages, and the lane's
  // first entry, from its state x.
  __device__ __forceinline__ void start(uint32_t x) {
    p = ring;
    thr = ring + kUnitRing;
    wraps = 0;
#pragma unroll
    for (uint32_t u = 0; u < 3; u++) {
#pragma unroll
      for (uint32_t b = 0; b < kBlocks; b++) w[b] = first[u * kBlocks + b];
      lookups();
      if (u == 2) break;
#pragma unroll
      for (uint32_t b = 0; b < kBlocks; b++)
        lds_store4(ring_v + u * kUnitRing + b * kBlockRing,
                   word_entries(w[b], g[2 * b], g[2 * b + 1]));
    }
#pragma unroll
    for (uint32_t b = 0; b < kBlocks; b++) wn[b] = first[3 * kBlocks + b];
    begin(x);
  }

  // After every kBlocks groups j of two steps: they consume at most a unit until the
  // next call, and at least a unit is left after it.
  template <int j>
  __device__ __forceinline__ void check() {
    if constexpr (j % kBlocks == kBlocks - 1) {
      if (__builtin_expect(p > thr, 0)) commit();
    }
  }
  __device__ __forceinline__ void commit() {
    const bool head = thr == ring + kUnitRing;  // the ring's first unit is next
#pragma unroll
    for (uint32_t b = 0; b < kBlocks; b++) {
      const ru4 v = word_entries(w[b], g[2 * b], g[2 * b + 1]);
      lds_store4(ring_v + (head ? 0u : kUnitRing) + b * kBlockRing, v);
      if (head) lds_store4(ring_v + 2 * kUnitRing + b * kBlockRing, v);
    }
    p -= head ? 0u : 2 * kUnitRing;
    wraps += head ? 0u : 1u;
    thr = 2 * ring + 3 * kUnitRing - thr;
#pragma unroll
    for (uint32_t b = 0; b < kBlocks; b++) w[b] = wn[b];
    lookups();
    // the unit at `slot` has landed once at most the kStage - 2 units after it
    // are in flight; the slot before it is free, its words are in w
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kBlocks * (kStage - 2)) : "memory");
#pragma unroll
    for (uint32_t b = 0; b < kBlocks; b++)
      wn[b] = lds_load1(ring + kStaging + slot + b * kBlockWordBytes + lane4);
    stage(around(slot + kSlots - kUnitWords));
    slot = around(slot + kUnitWords);
    // keep the words in their registers: no copies on the path without a commit
#pragma unroll
    for (uint32_t b = 0; b < kBlocks; b++) asm volatile("" : "+v"(w[b]), "+v"(wn[b]));
  }

  template <bool kAll>
  __device__ __forceinline__ uint32_t next(bool active) {
    return step<kAll>(active, p, p);
  }

  __device__ __forceinline__ uint32_t words() const {
    return (wraps * 2 * kUnitRing + (p - ring)) / 8u;
  }

  // No load may be in flight to the wave's LDS when it ends.
  __device__ __forceinline__ void close() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
};

}  // namespace
