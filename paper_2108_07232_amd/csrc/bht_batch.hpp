// Batched mode: many independent cuckoo tables of uneven sizes built and
// then queried by persistent kernels that pull (table, range) work items
// from device-side queues (a wave's first item is its own, further ones come
// from up to 16 counters on separate lines).  Each wave takes an item, runs the same per-lane insertion or query loop as the
// single-table kernels on that table's range, and takes the next item, so
// thousands of small tables cost a few launches instead of thousands, and
// large tables still spread over the whole device.
//
// Phases are separate kernels (reset -> build -> find): on gfx950 each XCD
// has its own L2, and the kernel boundary is what makes one table's
// inserts, performed by atomics, visible to plain bucket loads of queries
// running on any XCD.
#pragma once
#include "bht_kernels.hpp"
#include "bht_partition.hpp"

namespace bht {

struct BatchTable {
  uint64_t* slots;
  uint64_t words;
  const uint32_t* keys;
  const uint32_t* vals;
  uint64_t n_keys;
  const uint32_t* queries;
  uint32_t* out_v;
  uint8_t* out_f;
  uint64_t n_queries;
  Hash32 H;
  uint32_t max_chain;
  uint32_t rng_seed;
};

struct BatchItem {
  uint32_t table;
  uint32_t pad;
  uint64_t start;
  uint64_t count;
};

// Clears the heads of the build's and the queries' queue and every table's
// status word (no memset nodes, so the sequence can be captured in a graph
// and replayed).
__global__ void batch_reset_kernel(unsigned int* __restrict__ heads,
                                   uint32_t* __restrict__ status, uint32_t n_tables) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  clear_heads(heads, i);
  clear_heads(heads + kQueueHeads * kAtomicLine, i);
  for (uint32_t t = i; t < n_tables; t += gridDim.x * blockDim.x) status[t] = 0;
}

// Section III: every bucket of every table starts empty.  Item = a range of
// 64-bit words of one table's slot array.
__global__ __launch_bounds__(kBlock) void batch_fill_kernel(const BatchTable* __restrict__ tables,
                                                           const BatchItem* __restrict__ items,
                                                           uint64_t n_items) {
  for (uint64_t it = blockIdx.x; it < n_items; it += gridDim.x) {
    const BatchItem item = items[it];
    uint64_t* const p = tables[item.table].slots;
    for (uint64_t w = item.start + threadIdx.x; w < item.start + item.count; w += blockDim.x)
      p[w] = kEmptyPair;
  }
}

template <int B, int W>
__global__ __launch_bounds__(kBlock) void batch_build_kernel(const BatchTable* __restrict__ tables,
                                                            const BatchItem* __restrict__ items,
                                                            uint32_t n_items,
                                                            unsigned int* __restrict__ heads,
                                                            uint32_t* __restrict__ status) {
  const uint32_t salt = lane_salt();
  for_items(heads, n_items, [&](uint32_t it) {
    const BatchItem item = items[it];
    const BatchTable& T = tables[item.table];
    BuildArgs32 g;
    g.slots = T.slots;
    g.keys = T.keys;
    g.vals = T.vals;
    g.n = T.n_keys;
    g.status = status + item.table;
    g.probe_total = nullptr;
    g.H = T.H;
    g.max_chain = T.max_chain;
    g.rng_seed = T.rng_seed;
    Range r;
    r.cursor = item.start;
    r.end = item.start + item.count;
    uint32_t probes = 0;
    const uint32_t flags =
        cuckoo_build_range<B, W, false>(g, r, g.rng_seed ^ salt ^ (it * 0x85EBCA6Bu), &probes);
    if (flags) atomicOr(g.status, flags);
  });
}

// How the listed ranges of queries are cut into work items: 2^shift pieces
// of `size` queries each (the last ones of a short range are empty).  The
// cutting is left to the waves because the list is made and copied on the
// host when the batch is created: 101 M queries in items of 256 took 5.0 ms
// to list one by one, 0.5 ms in ranges of 8,192.
struct FindCut {
  uint32_t size, shift;
};

template <int B, int W, int Q = 1>
__global__ __launch_bounds__(kBlock) void batch_find_kernel(const BatchTable* __restrict__ tables,
                                                           const BatchItem* __restrict__ items,
                                                           uint32_t n_items, FindCut cut,
                                                           uint32_t queues,
                                                           unsigned int* __restrict__ heads) {
  for_items(heads, n_items << cut.shift, [&](uint32_t it) {
    const BatchItem item = items[it >> cut.shift];
    const uint64_t skip = (uint64_t)(it & ((1u << cut.shift) - 1)) * cut.size;
    if (skip >= item.count) return;
    const BatchTable& T = tables[item.table];
    FindArgs32 g;
    g.slots = T.slots;
    g.queries = T.queries;
    g.n = T.n_queries;
    g.out_v = T.out_v;
    g.out_f = T.out_f;
    g.probes = nullptr;
    g.H = T.H;
    Range r;
    r.cursor = item.start + skip;
    r.end = item.start + (item.count - skip < cut.size ? item.count : skip + cut.size);
    cuckoo_find_chunk_range<B, W, false, Q>(g, r);
  }, queues);
}

// ---------------------------------------------- partitioned batched build
//
// The partitioned build of bht_partition.hpp for all tables of a batch at
// once, with one radix pass per table: a table's pairs are grouped by the
// bin (8,192 slots; 2,048 where that leaves no table more than 1,024 bins) of
// their first bucket within that table, so pairs of
// different tables never mix and every table needs at most 1,024 bins.
// Bins of all tables are numbered globally (table t owns bins
// [bin_off_t, bin_off_t + nbins_t)); placement and overflow insertion run
// over the global bins.  Work items of the counting and scatter kernels are
// (table, chunk of at most 64 K pairs, 16 K in smaller batches); the partitioned pairs live in a
// workspace where table t's pairs start at key_off_t.

struct BatchPart {
  unsigned long long key_off;    // first workspace position of the table's pairs
  unsigned long long hist_off;   // first counter of the table's chunk histograms
  uint32_t bin_off;              // first global bin of the table
  uint32_t nbins;                // bins of the table (at most kMaxFan)
};

struct BatchChunk {
  uint32_t table;
  uint32_t local;                // chunk index within the table
  unsigned long long start;      // first pair of the chunk, within the table's input
  unsigned long long count;
};

struct BatchPartArgs {
  const BatchTable* tables;
  const BatchPart* parts;
  const BatchChunk* chunks;
  const uint32_t* bin_table;     // global bin -> table
  uint32_t n_chunks;
  uint32_t count;                // tables
  uint32_t nbins;                // global bins
  uint32_t bin_shift;            // bins of 2^bin_shift buckets
  uint32_t splits;               // overflow work items per bin
  uint32_t* hist;
  unsigned long long* total;     // per global bin
  unsigned long long* cursor;
  unsigned long long* bin_start;
  unsigned long long* bin_len;
  uint32_t* ovf_len;
  uint32_t* keys;                // workspace
  uint32_t* vals;
  unsigned int* head;            // overflow queue
  uint32_t* status;              // per table
};

__global__ void batch_part_clear_kernel(BatchPartArgs a) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  for (uint32_t j = i; j < a.nbins; j += gridDim.x * blockDim.x) a.total[j] = 0;
  clear_heads(a.head, i);
}

__global__ __launch_bounds__(kPassBlock) void batch_part_hist_kernel(BatchPartArgs a) {
  const BatchChunk c = a.chunks[blockIdx.x];
  const BatchTable& T = a.tables[c.table];
  const BatchPart P = a.parts[c.table];
  const Hash32 H = T.H;
  const uint32_t shift = a.bin_shift;
  const bool sentinel =
      hist_range<8>(T.keys, c.start, c.start + c.count, P.nbins,
                 [&](uint32_t k) { return hash32(H, 0, k) >> shift; },
                 a.hist + P.hist_off + (uint64_t)c.local * P.nbins, a.total + P.bin_off);
  if (sentinel) atomicOr(a.status + c.table, kFlagSentinel);
}

// One block per table: the table's bin totals become workspace ranges.
__global__ __launch_bounds__(kPartBlock) void batch_part_scan_kernel(BatchPartArgs a) {
  __shared__ unsigned long long wt[kPartBlock / 64];
  __shared__ unsigned long long base[kMaxFan];
  const BatchPart P = a.parts[blockIdx.x];
  const unsigned long long* tot = a.total + P.bin_off;
  block_exclusive_scan<kPartBlock, unsigned long long>(tot, base, P.nbins, wt);
  for (uint32_t d = threadIdx.x; d < P.nbins; d += kPartBlock) {
    const uint64_t g = (uint64_t)P.bin_off + d;
    a.cursor[g] = P.key_off + base[d];
    a.bin_start[g] = P.key_off + base[d];
    a.bin_len[g] = tot[d];
  }
}

__global__ __launch_bounds__(kPassBlock, kScatterBlocksPerCU) void batch_part_scatter_kernel(BatchPartArgs a) {
  const BatchChunk c = a.chunks[blockIdx.x];
  const BatchTable& T = a.tables[c.table];
  const BatchPart P = a.parts[c.table];
  const Hash32 H = T.H;
  const uint32_t shift = a.bin_shift;
  scatter_range<16>(T.keys, T.vals, c.start, c.start + c.count, P.nbins,
                [&](uint32_t k) { return hash32(H, 0, k) >> shift; },
                a.hist + P.hist_off + (uint64_t)c.local * P.nbins, a.cursor + P.bin_off, a.keys,
                a.vals);
}

// One block per global bin.
template <int B, int S>
__global__ __launch_bounds__(kBinBlock) void batch_place_kernel(BatchPartArgs a) {
  const uint32_t g = blockIdx.x;
  const uint32_t t = a.bin_table[g];
  const BatchTable& T = a.tables[t];
  const uint32_t R = 1u << a.bin_shift;
  const uint64_t first = (uint64_t)(g - a.parts[t].bin_off) * R;
  const uint32_t nb = (uint64_t)T.H.m - first < (uint64_t)R ? (uint32_t)(T.H.m - first) : R;
  const uint32_t ovf = place_bin<B, true, S>(T.slots, a.keys, a.vals, T.H, R, first, nb, a.bin_start[g],
                                    a.bin_len[g], T.max_chain, T.rng_seed, g, (uint32_t)B,
                                    a.status + t);
  if (threadIdx.x == 0) a.ovf_len[g] = ovf;
}

// Pairs evicted during placement continue at their next buckets (cuckoo
// insertion, Section III-A).
template <int B, bool BOTH>
__global__ __launch_bounds__(kBlock) void batch_overflow_kernel(BatchPartArgs a) {
  const uint32_t salt = lane_salt();
  for_items(a.head, a.nbins * a.splits, [&](uint32_t it) {
    const uint32_t g = it / a.splits, part = it % a.splits;
    const Range r = part_of(a.bin_start[g], a.ovf_len[g], part, a.splits);
    if (r.cursor >= r.end) return;
    const uint32_t t = a.bin_table[g];
    const BatchTable& T = a.tables[t];
    BuildArgs32 b;
    b.slots = T.slots;
    b.keys = a.keys;
    b.vals = a.vals;
    b.n = 0;
    b.status = a.status + t;
    b.probe_total = nullptr;
    b.H = T.H;
    b.max_chain = T.max_chain;
    b.rng_seed = T.rng_seed;
    uint32_t probes = 0;
    const uint32_t flags = cuckoo_continue_range<B, BOTH>(
        b, r, T.rng_seed ^ salt ^ (g * 0x85EBCA6Bu), &probes);
    if (flags) atomicOr(a.status + t, flags);
  });
}

// Small coalesced query launches pass their request descriptors as kernel
// arguments (no staging copy, no queue reset): a launch is then as cheap as
// a single-table query.  Work items are implicit: request r owns items
// [first_item[r], first_item[r+1]), each item_size queries long, and waves
// take items round-robin.
struct FindTable {
  const uint64_t* slots;
  const uint32_t* queries;
  uint32_t* out_v;
  uint8_t* out_f;
  uint64_t n;
  Hash32 H;
};

constexpr int kInlineRequests = 24;

struct InlineFind {
  FindTable t[kInlineRequests];
  uint32_t first_item[kInlineRequests + 1];
  uint32_t count;
  uint32_t item_size;
};

// The request and the range of its queries of work item `it`.
__device__ __forceinline__ FindArgs32 inline_item(const InlineFind& a, uint32_t it, Range* rg) {
  uint32_t r = 0;
  while (r + 1 < a.count && a.first_item[r + 1] <= it) ++r;
  const FindTable& T = a.t[r];
  FindArgs32 g;
  g.slots = T.slots;
  g.queries = T.queries;
  g.n = T.n;
  g.out_v = T.out_v;
  g.out_f = T.out_f;
  g.probes = nullptr;
  g.H = T.H;
  rg->cursor = (uint64_t)(it - a.first_item[r]) * a.item_size;
  rg->end = rg->cursor + a.item_size < T.n ? rg->cursor + a.item_size : T.n;
  return g;
}

template <int B, int W>
__global__ __launch_bounds__(kBlock) void inline_find_kernel(InlineFind a) {
  const uint32_t wave = (uint32_t)(((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  const uint32_t nwaves = (uint32_t)(((uint64_t)gridDim.x * blockDim.x) >> 6);
  const uint32_t total = a.first_item[a.count];
  for (uint64_t it = wave; it < total; it += nwaves) {
    Range rg;
    const FindArgs32 g = inline_item(a, (uint32_t)it, &rg);
    cuckoo_find_chunk_range<B, W, false>(g, rg);
  }
}

// For few queries in all: an item of at most 64 per wave, read per lane as
// by cuckoo_find_lane_kernel (16 requests, 90,000 queries: 7.8 -> 6.8 us).
template <int B>
__global__ __launch_bounds__(kBlock) void inline_find_lane_kernel(InlineFind a) {
  const uint32_t wave = __builtin_amdgcn_readfirstlane(
      (uint32_t)(((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6));
  if (wave >= a.first_item[a.count]) return;
  Range rg;
  const FindArgs32 g = inline_item(a, wave, &rg);
  const uint64_t idx = rg.cursor + __lane_id();
  if (idx < rg.end) cuckoo_find_lane<B, false>(g, idx);
}

}  // namespace bht
