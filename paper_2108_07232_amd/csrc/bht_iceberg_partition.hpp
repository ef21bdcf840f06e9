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

}  // namespace bht
