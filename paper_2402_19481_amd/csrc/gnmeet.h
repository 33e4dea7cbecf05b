// What the workgroups of gn_meet_kernel (groupnorm.hip) go by when they hand each other sums: rules of a few integers, for the host as well, so
// that all interleavings of a launch can be tried there.
#pragma once
#include "kernels.h"

namespace df {

// The patch's own cached sums [B, G, 2] may be refreshed in place (sums_out inside stale).  Two statistic modes read the old entry, in every
// workgroup of a slab; one that is late to start must not find the new one there.
__host__ __device__ inline bool gn_reads_own(int stat_mode) { return stat_mode == DF_GN_EQ2 || stat_mode == DF_GN_STALE; }

// Which workgroup of a slab writes the patch's own sums (all of them know the totals).  `counted`: each has added one to the slab's counter behind
// its read of the cached sums and found `arrived` there; no other launch counts meanwhile and every launch adds P, so the last to arrive, waited
// for or not, knows that all have read.  Not counted: nobody reads what is written.
__host__ __device__ inline bool gn_meet_writes(bool counted, unsigned int arrived, int P, int part) {
  return counted ? (arrived & (unsigned int)(P - 1)) == (unsigned int)(P - 1) : part == 0;
}

// Without a counter of its own (the library's words serve calls that overlap) a launch that would overwrite cached sums that it reads takes them from
// a copy, made by a launch before it (1.9 us: 1024 x 1280 bf16 recorded 9.3 us, 7.4 without, two launches 10.0).  `n` floats of a patch; the own entry
// alone, where the mode does not read it, needs none.
inline bool gn_meet_copies(const float* stale, const float* sums_out, long long n, int patch_idx, int N, int stat_mode) {
  if (!stale || !sums_out) return false;
  const uintptr_t s = (uintptr_t)stale, o = (uintptr_t)sums_out, entry = (uintptr_t)n * sizeof(float);
  if (o >= s + N * entry || s >= o + entry) return false;
  return gn_reads_own(stat_mode) || o != s + patch_idx * entry;
}

// The number that a launch's words carry.  A word counts with the right number only, so no other launch whose words may lie there has the same.
//   - Words of one plan (id 0): its launches do not overlap, each takes P tickets, so a ticket's multiple of P is the launch's; older words are always
//     the previous launch's.
//   - The library's words serve calls that overlap, and tickets that are dealt out in turns say nothing there: of two launches a replay can find
//     half of a multiple its own and half the replay's before.  The call has a number of its own instead; an eager one gets it back after 2^31
//     others.  A recorded one keeps it for all replays (so those have numbers that no eager call has), and its words are cleared by a launch
//     before it: others on the same words can take a word away, not bring back the replay's before (1.5 us: 494 x 1280 float 6.6 us recorded, 5.1
//     eager, a workgroup per group 6.2; 4096 x 640 float 8.8, two launches 13.4).  Two replays of it at once are the same sums of the same x.
__host__ __device__ inline unsigned int gn_meet_number(unsigned int id, unsigned int ticket, int lgP) { return id ? id : (ticket >> lgP) + 1u; }
inline unsigned int gn_call_id(unsigned long long n, bool recorded) {
  return (unsigned int)(n % 0x7fffffffull) + 1u + (recorded ? 0x80000000u : 0u);   // (never 0: words that nobody has written)
}

}  // namespace df
