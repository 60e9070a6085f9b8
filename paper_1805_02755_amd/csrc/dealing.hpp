// Dealing of many small pieces of uneven work to the workgroups of one launch,
// and inside a workgroup to its waves.
//
// The pieces are dealt in levels: a level hands an eighth of what is left to the
// launch's T workgroups in claims of equal size, the last levels a few parts
// each. So a run takes some tens of claims per workgroup from the counter in HBM
// instead of one per piece (an atomic on it takes 12.5 ns, one after another),
// and what is uneven in the claims of one level is evened out by the next.
// Workgroup t starts with claim t of level 0 without asking. The pieces of a
// claim are T apart, rotated from one to the next, so that they do not all come
// from one place.
//
// There are four counters, each with every fourth workgroup and every fourth
// piece: one counter still bounded small batches (16 jobs of 9 million pixels,
// packages of one and two tiles: 294 and 306 us, with 4 counters 221 and 238, 2
// jobs of 2 million 160 and 178, now 128 and 145), while with 16 or 32 the work
// of the banks differs by more than that gains (1,024 jobs: 9.40 ms with one
// counter, 9.43 with 4, 9.57 and 9.91).
//
// The batch of 256 escape-time jobs (157 million pixels, tiles of 16 x 16) with
// packages of 1, 2, 4 and 8 tiles taken from the counter one by one, a barrier
// after each: 7.55, 3.91, 2.68 and 2.73 ms; dealt, 2.68, 2.52, 2.54 and 2.64. With a half of what is
// left in each level 3.05, 2.92, 3.03, 3.04, with a quarter 2.89, 2.71, 2.65,
// 2.71 (a workgroup's first claim may hold far more than its share of the work);
// with claims of fixed size and no counter 3.35, 3.43, 3.53, 3.90.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_divide.hpp"

namespace ce {

constexpr uint32_t kDealLevels = 64;
constexpr uint32_t kDealLeastParts = 8;  // of a claim, two per wave
constexpr uint32_t kDealBanks = 4;
constexpr uint32_t kDealBankWords = 16;  // a counter's own 128 bytes
constexpr size_t kDealCounterBytes = (size_t)kDealBanks * kDealBankWords * sizeof(uint64_t);

struct Deal {
  uint64_t whole;               // pieces of `parts` parts
  uint32_t rest;                // parts of the one after them
  uint32_t banks;
  Divisor groups;               // workgroups of a bank
  Divisor parts;                // waves' parts of a piece
  uint32_t turn;                // pieces the assignment is rotated by
  uint32_t levels;
  uint64_t start[kDealLevels];  // first of a bank's pieces in a level
  uint32_t size[kDealLevels];   // pieces of one of its claims
  uint64_t* counters;           // kDealCounterBytes, zero: a bank's claims after level 0, and its workgroups that left

  __host__ Deal(uint64_t n_parts, uint32_t workgroups, uint32_t parts_per_piece, uint64_t* c)
      : whole(n_parts / parts_per_piece), rest((uint32_t)(n_parts % parts_per_piece)), banks(workgroups % kDealBanks ? 1u : kDealBanks), groups(workgroups / banks), parts(parts_per_piece),
        turn((uint32_t)(groups.d * 5ull / 8) | 1u), levels(0), counters(c) {
    const uint32_t least = (kDealLeastParts + parts_per_piece - 1) / parts_per_piece;
    const uint64_t pieces = whole + (rest != 0), all = pieces / banks + (pieces % banks != 0);
    // an eighth, or as little more as the table has room for (2^14 pieces per workgroup)
    for (uint64_t share = 8; share >= 1; --share) {
      uint64_t at = 0;
      for (levels = 0; at < all && levels < kDealLevels; ++levels) {
        const uint64_t part = (all - at) / (share * groups.d) + (share == 1);
        start[levels] = at;
        size[levels] = (uint32_t)(part > least ? part : least);
        at += (uint64_t)size[levels] * groups.d;
      }
      if (at >= all) break;
    }
  }
};

#ifdef __HIPCC__
// A workgroup's dealing state in LDS: the claim in the high half, its next part
// in the low one.
struct DealState {
  unsigned long long claim_part;
};

__device__ __forceinline__ uint64_t* deal_counter(const Deal& d) {
  return d.counters + (blockIdx.x & (d.banks - 1)) * kDealBankWords;
}

__device__ __forceinline__ void deal_begin(const Deal& d, DealState& s) {
  if (threadIdx.x == 0) s.claim_part = (unsigned long long)(blockIdx.x / d.banks) << 32;
  __syncthreads();
}

// The wave's next part of work: false when there is none left. All of a wave's
// lanes call it and get the same.
__device__ __forceinline__ bool deal_next(const Deal& d, DealState& s, uint64_t* piece, uint32_t* part) {
  const bool first = __lane_id() == 0;
  for (;;) {
    unsigned long long got = 0;
    if (first) got = __hip_atomic_fetch_add(&s.claim_part, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    const uint32_t claim = __builtin_amdgcn_readfirstlane((uint32_t)(got >> 32));
    const uint32_t i = __builtin_amdgcn_readfirstlane((uint32_t)got);
    uint32_t place, rotated;
    const uint32_t level = d.groups.split(claim, &place);
    if (level >= d.levels) return false;
    const uint32_t all = d.size[level] * d.parts.d;
    if (i == all) {  // this wave takes the next claim for the workgroup, and waits for nobody
      if (first) {
        const uint64_t c = d.groups.d + __hip_atomic_fetch_add(deal_counter(d), (uint64_t)1, __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&s.claim_part, (unsigned long long)c << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      continue;
    }
    if (i > all) {  // another wave is taking it
      __builtin_amdgcn_s_sleep(2);
      continue;
    }
    const uint32_t j = d.parts.split(i, part);
    d.groups.split(j * d.turn, &rotated);
    place += rotated;
    const uint64_t own = d.start[level] + (uint64_t)j * d.groups.d + (place < d.groups.d ? place : place - d.groups.d);
    *piece = own * d.banks + (blockIdx.x & (d.banks - 1));
    if (__builtin_expect(*piece < d.whole, 1) || (*piece == d.whole && *part < d.rest)) return true;
    // nothing left in this piece: on to the next (unless the claim is over), not
    // part by part, since a caller's piece may have millions
    if (first)
      __hip_atomic_fetch_max(&s.claim_part, (unsigned long long)claim << 32 | (j + 1) * d.parts.d, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}

// The last workgroup of a bank re-arms its counter for the next launch (no
// memset node is needed when the launch is replayed from a graph).
__device__ __forceinline__ void deal_end(const Deal& d) {
  __syncthreads();
  if (threadIdx.x != 0) return;
  uint64_t* const c = deal_counter(d);
  const uint64_t out = __hip_atomic_fetch_add(&c[1], (uint64_t)1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
  if (out + 1 == d.groups.d) {
    __hip_atomic_store(&c[0], (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&c[1], (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}
#endif

}  // namespace ce
