// Partitioned bulk build of the iceberg table (Section III-C).
//
// The radix passes and the bin placement are the cuckoo table's: pairs are
// grouped by the bin of their primary bucket, and a bin's primaries are
// filled on chip, each up to t pairs (the placement without eviction).  A
// pair that meets a primary already holding t pairs is written back to the
// front of its bin's input range and continues at its two secondary
// choices in the insertion kernel below, which is the concurrent iceberg
// insertion started after the primary step: first every pair whose primary
// is below t takes it, then the rest run the secondary step concurrently.
// The threshold rule holds exactly: a pair reaches the secondary level only
// once its primary holds t pairs.
#pragma once
#include "bht_partition.hpp"
#include "bht_schemes.hpp"

namespace bht {

struct IcebergOverflowArgs {
  SchemeArgs32 g;                // keys / vals = the partitioned arrays
  PartMeta M;
  uint32_t nbins;
  uint32_t parts;                // work items per bin
  uint32_t* counts;              // one per secondary bucket (counted kernel)
};

template <int B, int B2, int W>
__global__ __launch_bounds__(kBlock) void iceberg_overflow_kernel(IcebergOverflowArgs a) {
  uint32_t flags = 0, probes = 0, evicted = 0;
  for_items(a.M.head, a.nbins * a.parts, [&](uint32_t it) {
    const uint32_t bin = it / a.parts, part = it % a.parts;
    const Range r = part_of(a.M.bin_start[bin], a.M.ovf_len[bin], part, a.parts);
    evicted += (uint32_t)(r.end - r.cursor);
    if (r.cursor < r.end) flags |= iceberg_build_range<B, B2, W, true, true>(a.g, r, &probes);
  });
  if (flags) atomicOr(a.g.status, flags);
  add_overflow_stats(a.M.stats, a.g.status, evicted, probes);
}

// The same phase with one counter per secondary bucket, of two-level tables
// (as p2_count_build_kernel: a pair reads the counts of its two secondary
// buckets, raises the smaller one from the value read, ties to s0, and
// stores itself in the slot that value names).  With both secondaries full
// the pair goes to its primary past the t pairs there, as above.
template <int B, int B2>
__global__ __launch_bounds__(kBlock) void iceberg_count_overflow_kernel(IcebergOverflowArgs a) {
  constexpr uint32_t kStride = p2_count_stride(B2);
  const SchemeArgs32& g = a.g;
  const uint32_t lane = __lane_id();
  const uint32_t t = g.threshold < (uint32_t)B ? g.threshold : (uint32_t)B;
  uint32_t flags = 0, probes = 0, evicted = 0;
  for_items(a.M.head, a.nbins * a.parts, [&](uint32_t it) {
    const uint32_t bin = it / a.parts, part = it % a.parts;
    const Range r = part_of(a.M.bin_start[bin], a.M.ovf_len[bin], part, a.parts);
    evicted += (uint32_t)(r.end - r.cursor);
    uint64_t i = r.cursor + lane;
    uint32_t k_next = i < r.end ? g.keys[i] : 0u, v_next = i < r.end ? g.vals[i] : 0u;
    for (; i < r.end; i += 64) {
      const uint32_t key = k_next, val = v_next;
      if (i + 64 < r.end) {
        k_next = g.keys[i + 64];
        v_next = g.vals[i + 64];
      }
      const uint64_t pair = ((uint64_t)val << 32) | key;
      const uint32_t s0 = hash32(g.H2, 1, key), s1 = hash32(g.H2, 2, key);
      uint32_t l0 = __hip_atomic_load(a.counts + (uint64_t)s0 * kStride, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
      uint32_t l1 = __hip_atomic_load(a.counts + (uint64_t)s1 * kStride, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
      probes += 2;
      bool placed = false;
      // at most 2 B2 tries: each failed one has raised a count seen
      for (;;) {
        const bool first = l0 <= l1;
        const uint32_t s = first ? s0 : s1, slot = first ? l0 : l1;
        if (slot >= (uint32_t)B2) break;
        uint32_t seen = slot;
        if (__hip_atomic_compare_exchange_strong(a.counts + (uint64_t)s * kStride, &seen, slot + 1,
                                                 __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT)) {
          g.slots2[(uint64_t)s * B2 + slot] = pair;
          placed = true;
          break;
        }
        if (first || s0 == s1) l0 = seen;
        if (!first || s0 == s1) l1 = seen;
      }
      if (!placed) {
        uint64_t* const primary = g.slots + (uint64_t)hash32(g.H, 0, key) * B;
        for (uint32_t slot = t; slot < (uint32_t)B && !placed; ++slot)
          placed = cas64(primary + slot, kEmptyPair, pair) == kEmptyPair;
        if (!placed) flags |= kFlagFailed;
      }
    }
  });
  if (flags) atomicOr(a.g.status, flags);
  add_overflow_stats(a.M.stats, a.g.status, evicted, probes);
}

}  // namespace bht
