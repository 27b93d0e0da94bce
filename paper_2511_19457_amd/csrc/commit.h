// Count commit of an output measurement fused into a producer kernel: the
// work-groups' zero counts and nonzero-block counts reach the sparoa_counts of
// the output without one same-address atomic per work-group.
#pragma once

#include <hip/hip_runtime.h>

#include "sparoa.h"

namespace sparoa {

// Words of the grouped count commit: kOmGroups groups x 2 counters, one
// 128-byte line each.
constexpr int kOmGroups = 8;
constexpr int kOmDirectMax = 64;   // grids up to this many work-groups commit directly
static_assert(2 * kOmGroups * 128 == SPAROA_COMMIT_WORDS_BYTES, "commit word layout");
// Packed commit: both counts and the ticket in one word, 16 groups of one
// word each (the same lines): ticket from bit 52, zeros from bit 24, nonzero
// blocks below.  One returning atomic per work-group instead of two, and half
// the members on a word.
constexpr int kOmPackedGroups = 2 * kOmGroups;

// The words argument of om_commit for an output of numel elements measured by
// nwg work-groups: bit 0 marks the packed commit, taken where no field can
// overflow (a group's zeros < 2^28, its blocks of 8 < 2^24, its members <
// 2^12).
inline unsigned long long *om_words_for(unsigned long long *words, int64_t numel, int64_t nwg) {
  const bool packed = numel < ((int64_t)1 << 27) && nwg / kOmPackedGroups < 4095;
  return words && packed ? reinterpret_cast<unsigned long long *>(
                               reinterpret_cast<uintptr_t>(words) | 1u)
                         : words;
}

// Sum of v over the 64 lanes of a wave, in lane 63.  Six adds whose operand
// moves between lanes in the vector unit (row shifts, then row broadcasts):
// the same sum by shuffles goes through LDS six times, one latency each.  (The
// commit is the tail of every measuring kernel: with the parts below read at
// once it takes 1.45 us of a 14 x 14 layer, 1.7 with shuffles and one LDS read
// per wave; the rest is the atomics.  8 groups instead of 16: 0.05 to 0.3 us
// slower, 4: 0.3 to 0.7.)
__device__ __forceinline__ uint32_t wave_sum_63(uint32_t v) {
#define SPAROA_DPP_ADD(ctrl, rows) \
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xf, true)
  SPAROA_DPP_ADD(0x111, 0xf);   // row_shr:1, :2, :4, :8
  SPAROA_DPP_ADD(0x112, 0xf);
  SPAROA_DPP_ADD(0x114, 0xf);
  SPAROA_DPP_ADD(0x118, 0xf);
  SPAROA_DPP_ADD(0x142, 0xa);   // row_bcast:15 into rows 1 and 3
  SPAROA_DPP_ADD(0x143, 0xc);   // row_bcast:31 into rows 2 and 3
#undef SPAROA_DPP_ADD
  return v;
}

// Adds a work-group's zero count and nonzero-block count into counts
// (zero_blocks starts at nb).  Same-address atomics serialise device-wide
// (13-17 ns per work-group measured with one atomic per counter), so with
// `words` (the caller's zeroed count-commit words) work-group b of nwg is
// a member of group b % kOmGroups: each member adds (1 << 40) + its count to
// its group's word with one returning atomic, and the member whose add
// completes the group adds the group's total to counts and clears the word
// for the next call (om_words_for: both counts in one word where they fit).
// Without `words`, or for a grid of at most
// kOmDirectMax work-groups: one atomic per counter per work-group (the words
// are left untouched).
__device__ __forceinline__ void om_commit(uint32_t zeros, uint32_t nz, sparoa_counts *counts,
                                          unsigned long long *words, int64_t b, int64_t nwg) {
  __shared__ __attribute__((aligned(16))) uint32_t part[2][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  zeros = wave_sum_63(zeros);
  nz = wave_sum_63(nz);
  if (lane == 63) {
    part[0][wave] = zeros;
    part[1][wave] = nz;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    // every slot is read (in a few wide reads, all in flight at once), those
    // past the last wave's dropped
    unsigned long long z = 0, n = 0;
    const int waves = (int)(blockDim.x >> 6);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const uint32_t pz = part[0][i], pn = part[1][i];
      z += i < waves ? pz : 0u;
      n += i < waves ? pn : 0u;
    }
    // small grids commit directly: the ticket's returning atomic is a memory
    // round trip on every work-group's path (about 1 us), more than up to 64
    // work-groups' serialised same-address atomics (measured: 64 work-groups
    // 1 us faster direct, 98 work-groups 0.25 us slower)
    if (!words || nwg <= kOmDirectMax) {
      if (z) atomicAdd((unsigned long long *)&counts->zeros, z);
      if (n) atomicAdd((unsigned long long *)&counts->zero_blocks, 0ull - n);
      return;
    }
    if (reinterpret_cast<uintptr_t>(words) & 1u) {
      constexpr int kT = 52, kZ = 24;
      const int64_t g = b % kOmPackedGroups;
      const unsigned long long members = (unsigned long long)(
          nwg / kOmPackedGroups + (g < nwg % kOmPackedGroups ? 1 : 0));
      unsigned long long *w = reinterpret_cast<unsigned long long *>(
                                  reinterpret_cast<uintptr_t>(words) & ~(uintptr_t)1) +
                              g * 16;
      const unsigned long long mine = (1ull << kT) + (z << kZ) + n;
      const unsigned long long old = atomicAdd(w, mine);
      if ((old >> kT) == members - 1) {
        const unsigned long long t = old + mine;
        const unsigned long long tz = (t >> kZ) & ((1ull << (kT - kZ)) - 1);
        const unsigned long long tn = t & ((1ull << kZ) - 1);
        if (tz) atomicAdd((unsigned long long *)&counts->zeros, tz);
        if (tn) atomicAdd((unsigned long long *)&counts->zero_blocks, 0ull - tn);
        atomicExch(w, 0ull);
      }
      return;
    }
    constexpr unsigned long long kTicket = 1ull << 40;  // sums < 2^40, members < 2^24
    const int64_t g = b % kOmGroups;
    const unsigned long long members =
        (unsigned long long)(nwg / kOmGroups + (g < nwg % kOmGroups ? 1 : 0));
    unsigned long long *wz = words + g * 32, *wn = words + g * 32 + 16;
    const unsigned long long oz = atomicAdd(wz, kTicket + z);
    const unsigned long long on = atomicAdd(wn, kTicket + n);
    if ((oz >> 40) == members - 1) {
      const unsigned long long tz = (oz & (kTicket - 1)) + z;
      if (tz) atomicAdd((unsigned long long *)&counts->zeros, tz);
      atomicExch(wz, 0ull);
    }
    if ((on >> 40) == members - 1) {
      const unsigned long long tn = (on & (kTicket - 1)) + n;
      if (tn) atomicAdd((unsigned long long *)&counts->zero_blocks, 0ull - tn);
      atomicExch(wn, 0ull);
    }
  }
}

}  // namespace sparoa
