// Build of a small cuckoo table (BCHT, and the one-slot table) by a single
// workgroup: the whole table is built in LDS and written out once, so the
// insertion makes no global atomic and the build is one launch (no reset).
//
// The schedule is the partitioned build's (bht_partition.hpp): every pair
// claims the next slot of its first bucket, a pair that meets it full
// exchanges itself with a random resident there, and the evicted pairs take
// the first of their next two buckets with room or evict again.
#pragma once
#include "bht_kernels.hpp"

namespace bht {

constexpr int kSmallBlock = 1024;
constexpr int kSmallList = kSmallBlock;        // evicted pairs under way at once, one per thread

// Slots of a table built this way, at most: slots, one load counter per
// bucket and the list of evicted pairs fit the 160 KB of LDS.
template <int B>
constexpr int small_slots() { return B == 1 ? 12288 : 16384; }

// One workgroup.  A chain step costs LDS latencies (about 1 us per round of
// all evicted pairs, most of it the three hash evaluations) where the
// concurrent build pays dependent memory atomics (0.5 us each, and up to B
// of them for the claims of a bucket's first pairs, which all start at
// slot 0 of the empty table).  LF 0.9, concurrent (with 2 us of reset) and
// this build, us: 5,000 pairs 50 and 11, 10,000 52 and 18, 14,000 52 and 20;
// the partitioned build's six launches take 42 to 53.
template <int B>
__global__ __launch_bounds__(kSmallBlock) void small_build_kernel(BuildArgs32 g) {
  constexpr int S = small_slots<B>();
  constexpr int PER = S / kSmallBlock;
  __shared__ u64x2 tbl2[S / 2];
  __shared__ uint32_t load[S / B];
  __shared__ unsigned long long list[kSmallList];
  __shared__ uint32_t listed, flags_all;
  unsigned long long* tbl = reinterpret_cast<unsigned long long*>(tbl2);
  const uint32_t tid = threadIdx.x;
  const Hash32& H = g.H;
  const uint32_t m = H.m, words = m * B, n = (uint32_t)g.n;
  const u64x2 e2 = {kEmptyPair, kEmptyPair};
  for (uint32_t i = tid; i < (words + 1) / 2; i += kSmallBlock) tbl2[i] = e2;
  for (uint32_t i = tid; i < m; i += kSmallBlock) load[i] = 0;
  if (tid == 0) flags_all = 0;
  uint32_t rng = g.rng_seed ^ (tid * 0x9E3779B9u);
  if (rng == 0) rng = 0x2545F491u;
  uint32_t flags = 0, k[PER], v[PER], full[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const uint32_t i = j * kSmallBlock + tid;
    k[j] = kEmptyKey;
    v[j] = 0;
    full[j] = ~0u;
    if (j * kSmallBlock < (int)n) {              // uniform
      k[j] = g.keys[i < n ? i : n - 1];
      v[j] = g.vals[i < n ? i : n - 1];
    }
  }
  __syncthreads();
  // claims in first buckets
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    if (j * kSmallBlock + tid < n) {
      if (k[j] == kEmptyKey) {
        flags |= kFlagSentinel;
      } else {
        const uint32_t b = hash32(H, 0, k[j]);
        const uint32_t s = atomicAdd(&load[b], 1u);
        if (s < (uint32_t)B) tbl[b * B + s] = ((unsigned long long)v[j] << 32) | k[j];
        else full[j] = b;
      }
    }
  }
  __syncthreads();
  // exchanges in full first buckets (every claimed slot is written)
  bool held = false;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    if (full[j] != ~0u) {
      if (g.max_chain == 0) {
        flags |= kFlagFailed;
        full[j] = ~0u;
      } else {
        rng = xorshift32(rng);
        const unsigned long long old = atomicExch(&tbl[full[j] * B + rng % (uint32_t)B],
                                                  ((unsigned long long)v[j] << 32) | k[j]);
        k[j] = (uint32_t)old;
        v[j] = (uint32_t)(old >> 32);
        held = true;
      }
    }
  }
  // The evicted pairs' chains, one list of at most a pair per thread after
  // the other (few builds need a second list: 6% of the pairs at LF 0.9).
  while (__syncthreads_or(held)) {
    if (tid == 0) listed = 0;
    __syncthreads();
    held = false;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      if (full[j] != ~0u) {
        const uint32_t pos = atomicAdd(&listed, 1u);
        if (pos < (uint32_t)kSmallList) {
          list[pos] = ((unsigned long long)v[j] << 32) | k[j];
          full[j] = ~0u;
        } else {
          held = true;
        }
      }
    }
    __syncthreads();
    bool active = tid < (listed < (uint32_t)kSmallList ? listed : (uint32_t)kSmallList);
    uint32_t key = 0, val = 0, chain = 1;
    Choices c = {0u, 0u, false, false};
    if (active) {
      key = (uint32_t)list[tid];
      val = (uint32_t)(list[tid] >> 32);
      c = next_choices(H, key, 0u, true);
    }
    for (;;) {
      if (active && !c.full) {
        // a bucket with room takes the pair; exchanges never touch it, since
        // they are made in full buckets only
        uint32_t b = c.at, s = atomicAdd(&load[b], 1u);
        if (s >= (uint32_t)B && c.has_alt) {
          b = c.alt;
          s = atomicAdd(&load[b], 1u);
        }
        if (s < (uint32_t)B) {
          tbl[b * B + s] = ((unsigned long long)val << 32) | key;
          active = false;
        }
      }
      if (!__syncthreads_or(active)) break;
      if (active) {
        if (chain >= g.max_chain) {
          flags |= kFlagFailed;
          active = false;
        } else {
          rng = xorshift32(rng);
          const unsigned long long old = atomicExch(&tbl[c.at * B + rng % (uint32_t)B],
                                                    ((unsigned long long)val << 32) | key);
          key = (uint32_t)old;
          val = (uint32_t)(old >> 32);
          ++chain;
          c = next_choices(H, key, c.at, false);
        }
      }
    }
  }
  if (flags) atomicOr(&flags_all, flags);
  __syncthreads();
  u64x2* dst2 = reinterpret_cast<u64x2*>(g.slots);
  for (uint32_t i = tid; i < words / 2; i += kSmallBlock) dst2[i] = tbl2[i];
  if ((words & 1) && tid == 0) g.slots[words - 1] = tbl[words - 1];
  if (tid < 8) g.status[tid] = tid == 0 ? flags_all : 0u;
}

}  // namespace bht
