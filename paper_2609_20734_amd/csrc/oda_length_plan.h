// Split length of a Full call planned from the selected requests' lengths.
// Used by the attention kernels (every workgroup plans its call by itself, on
// wavefront-uniform values) and, without a GPU, by the plan's test: nothing
// here is HIP's but the function qualifiers.
#ifndef ODA_LENGTH_PLAN_H_
#define ODA_LENGTH_PLAN_H_

#include <stdint.h>

#if defined(__HIPCC__)
#define ODA_PLAN_FN __host__ __device__ __forceinline__
#else
#define ODA_PLAN_FN inline
#endif

namespace oda {

constexpr uint32_t kPlanCus = 256;        // workgroups of one round (one per CU)
constexpr uint32_t kPlanWaves = 8;        // shortest split: a block per wavefront
constexpr uint32_t kLengthBlocks = 128;   // shortest split that the plan adds rounds for
constexpr uint32_t kLengthRounds = 16;    // rounds of workgroups it considers
constexpr uint32_t kLongBlocks = 1024;    // blocks per CU from which its splits are kLongSplit blocks
constexpr uint32_t kLongSplit = 512;

ODA_PLAN_FN uint32_t plan_min(uint32_t x, uint32_t y) { return x < y ? x : y; }
ODA_PLAN_FN uint32_t plan_max(uint32_t x, uint32_t y) { return x > y ? x : y; }
ODA_PLAN_FN uint32_t even_up(uint32_t x) { return (x + 1) & ~1u; }

// ceil(n / c), c from 1, for n up to 2^26 and quotients up to 2^20 (a larger
// one comes out above 2^19: callers bound it by a request's blocks), with inv = 1 / c to within 2^-22 of it: n * inv
// rounded is the quotient's floor or ceiling (its error stays below a half), and
// one product tells which.  A third of the instructions of a 32-bit division, on
// the way to every workgroup's first load.
ODA_PLAN_FN uint32_t ceil_quotient(uint32_t n, uint32_t c, float inv) {
  const uint32_t q = (uint32_t)((float)n * inv + 0.5f);
  return q * c < n ? q + 1 : q;
}
ODA_PLAN_FN uint32_t ceil_quotient(uint32_t n, uint32_t c) {
#if defined(__HIP_DEVICE_COMPILE__)
  return ceil_quotient(n, c, __builtin_amdgcn_rcpf((float)c));
#else
  return ceil_quotient(n, c, 1.f / (float)c);
#endif
}

// The shortest even split length c in [least, whole], to within 1/16 of it,
// whose (request, split) pairs are at most `pairs` (pairs >= count; `total`
// blocks in `count` requests; pairs_of(c) = the sum of max(1, ceil(blocks / c))
// over the requests, which falls as c grows).  Below total / pairs nothing
// fits; from total / (pairs - count) everything does, since a request's count
// is at most blocks / c + 1.  The bisection between them takes at most five
// steps unless pairs is within a few of count.
template <class PairsOf>
ODA_PLAN_FN uint32_t shortest_fit(uint32_t total, uint32_t count, uint32_t least, uint32_t whole, uint32_t pairs,
                                  const PairsOf& pairs_of) {
  uint32_t lo = plan_min(whole, plan_max(least, even_up(ceil_quotient(total, pairs))));
  uint32_t hi = whole;
  if (pairs > count) hi = plan_max(lo, plan_min(whole, even_up(ceil_quotient(total, pairs - count))));
  uint32_t c = lo;
  for (;;) {
    if (pairs_of(c) <= pairs) {
      if (c == lo) return c;      // only the first try: later ones lie strictly between lo and hi
      hi = c;
    } else {
      lo = c;
    }
    if (hi - lo <= plan_max(2, lo / 16)) return hi;
    c = ((lo + hi) / 2) & ~1u;
  }
}

// Blocks per split for `count` (at most 64) selected requests of `total` blocks
// together, the longest of `longest` (at most 2^20), with `units` (layer, KV
// head) units apiece, at most max_splits splits each and at most `slots`
// (request, split) pairs (>= count).
//   - eight units per CU, whole units that fill their rounds of one workgroup
//     per CU within 5%, or one round whose longest unit takes no longer alone
//     (0.18 us a 128-wide block) than all blocks on a busy HBM (0.29 us a block
//     and CU) and the merge (8 us), or two rounds and more without the work
//     for one more: whole units.  24 requests of 200-2,000 positions: 27.9 us,
//     35.8 split;
//   - kLongBlocks blocks per CU: splits of kLongSplit blocks, whatever rounds
//     that makes.  Many uneven rounds beat few even ones, whose workgroups
//     start and wait for their first blocks together: one layer of 32
//     requests of 8K-64K positions 721 us, in eight even rounds
//     812, with the longest request's splits for all 913;
//   - else, for m = 1, 2, ... rounds, the shortest splits whose (request,
//     split) pairs fit m rounds; the first m at which they spread the blocks
//     over the CUs within 10% of evenly, else the m with the least m * bps.
//     Rounds past the first feasible one are tried only while splits keep
//     kLengthBlocks blocks.
template <class PairsOf>
ODA_PLAN_FN uint32_t length_bps(uint32_t total, uint32_t longest, uint32_t count, uint32_t units, uint32_t max_splits,
                                uint32_t slots, uint32_t head_dim, const PairsOf& pairs_of) {
  const uint32_t whole = even_up(plan_max(longest, 2));
  const uint64_t work = (uint64_t)total * units;
  const uint32_t rounds = (count * units + kPlanCus - 1) / kPlanCus;   // of whole units: the first feasible m
  if (rounds >= 8 || work * 20 >= (uint64_t)rounds * whole * kPlanCus * 19) return whole;
  if (rounds == 1 && (uint64_t)whole * 5 * kPlanCus <= 8 * work + 240 * 128 / head_dim * kPlanCus) return whole;
  if (rounds > 1 && work < (uint64_t)kLengthBlocks * (rounds + 1) * kPlanCus) return whole;
  // no split shorter than a block per wavefront, no more splits than partial slots
  const uint32_t least = even_up(plan_max(kPlanWaves, ceil_quotient(longest, max_splits)));
  if (work >= (uint64_t)kLongBlocks * kPlanCus) {
    const uint32_t c = plan_min(whole, plan_max(least, kLongSplit));
    return pairs_of(c) <= slots ? c : shortest_fit(total, count, least, whole, slots, pairs_of);
  }
  uint32_t best = whole, best_m = 0;
  for (uint32_t m = rounds; m <= kLengthRounds; ++m) {
    if (best_m != 0 && work < (uint64_t)kLengthBlocks * m * kPlanCus) break;
    const uint32_t pairs = ceil_quotient(kPlanCus * m - units + 1, units);   // the floor of kPlanCus * m / units
    const uint32_t c = shortest_fit(total, count, least, whole, plan_min(pairs, slots), pairs_of);
    if (best_m == 0 || m * c < best_m * best) {
      best = c;
      best_m = m;
    }
    if (work * 10 >= (uint64_t)m * c * kPlanCus * 9) break;
  }
  return best;
}

}  // namespace oda

#endif  // ODA_LENGTH_PLAN_H_
