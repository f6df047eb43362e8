// bf_partition.hpp -- partitioned construction: bulk add without global
// atomics on the filter.
//
// On gfx950 a device-scope atomic OR is executed beyond the XCD's L2, and
// the device sustains only ~20 G such requests per second from HBM; direct
// construction (one atomic group per key) is bound by that rate.  This path
// instead groups the keys by filter chunk -- a range of blocks whose words
// fit in LDS -- and lets one workgroup own each chunk: it loads the chunk
// into LDS, ORs the patterns of its keys with LDS atomics, and writes the
// chunk back with plain coalesced stores.  The filter words it writes are
// exactly those of the direct path (OR is commutative and idempotent).
//
// Grouping (bf_group.hpp) is a radix partition of the chunk index in one or
// two digits (the CPU filter the paper compares with partitions keys by
// radix for the same reason, Sec. V-A):
//   group    keys -> hashed records, each step of 8,192 sorted by the high
//            digit: block << 32 | lo32;                     [8 B in, 8 out]
//   regroup  the records of one high digit -> steps sorted by chunk, as
//            lo32 and the block within the chunk;           [8 in, 6 out]
//   apply    per chunk: LDS load, LDS atomic OR of the records of its runs,
//            store.                                         [6 in + chunk]
// A filter of at most kChunkDigits chunks (64 MiB) needs one digit: the
// first pass sorts its steps by chunk, and the second pass is skipped.
// No step depends on how the keys are distributed: repeated keys only make
// longer runs.  Measured on MI355X, 2^28 keys into 1 GiB of 256-bit blocks:
// group 0.81, plan and scan 0.016, regroup 0.87, apply 0.90 ms (with fixed
// capacity buckets instead of sorted steps 1.13, 1.15 and 0.84 ms).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bf_group.hpp"
#include "bf_hash.hpp"
#include "bf_kernels.hpp"
#include "bf_variant_kernels.hpp"

namespace bfhip {

constexpr int kClassicThreads = 512;
constexpr int kApplyThreads = 1024;                 // apply: 16 waves share one chunk
constexpr int kApplyList = 1536;                    // unit entries listed at once (LDS for two workgroups per CU)
constexpr int kChunkBytes = 64 * 1024;              // LDS bytes owned per chunk
constexpr int kMaxDigits = 1024;                    // digit fan-out limit of the first pass
constexpr int kMaxDigits2 = 512;                    // ... and of the second (chunks per high digit)
constexpr int kMaxChunks = kMaxDigits * kMaxDigits2;  // of a partitioned filter
constexpr int kWideDigits2 = 1024;                  // second digits of one filter beyond 16 GiB
constexpr int kChunkDigits = kMaxDigits;            // chunks up to which the first pass sorts by chunk
constexpr int kVecPerThread = kChunkBytes / 16 / kApplyThreads;  // 16-byte chunk vectors per apply thread
static_assert(kVecPerThread * 16 * kApplyThreads == kChunkBytes, "apply covers a chunk exactly");

// Slice `split` of `nsplit` of the records of chunk `bucket`, which are in
// the output of second-pass items [item0, item1).
struct PartWork {
  uint32_t bucket;
  uint16_t split;
  uint16_t nsplit;
  uint32_t item0;
  uint32_t item1;
};

struct ApplyArgs {
  // the single filter (nfilters == 1) or a table of filters sharing one
  // layout and k
  void* words;
  uint64_t num_blocks;
  const PartFilter* filters;
  const uint32_t* chunk_owner;  // global chunk -> filter
  // records and their table of runs, by chunk (one pass) or by second digit
  const uint32_t* table;
  uint64_t stride;
  const uint32_t* lo;
  const uint16_t* blk;
  const uint32_t* slot0;        // two passes: first output step of every item
  const PartWork* work;         // plans: the workgroups' chunks
  uint32_t nfilters;
  uint32_t k;
  uint32_t steps;               // one pass: table entries per chunk (else 0)
  uint32_t per_digit;           // two passes: items per first digit
  uint32_t chunk_shift;         // log2(blocks per chunk)
  uint32_t low_bits;            // bits of the second digit
  // slices of every chunk (> 1 for filters of few chunks, so the grid still
  // fills the device)
  uint32_t split;
};

struct PartArgs {
  GroupArgs g;
  RegroupArgs r;     // two digits only
  ApplyArgs p;
  uint64_t chunks;
  uint32_t nranges;  // plans: first-pass workgroups
  uint32_t nwork;    // plans: apply workgroups
  bool one_pass;
  bool short_units;  // second pass in units of kShortUnit slots
};

template <typename W>
__device__ __forceinline__ void lds_or(W* p, W v) {
  if constexpr (sizeof(W) == 8)
    atomicOr(reinterpret_cast<unsigned long long*>(p), static_cast<unsigned long long>(v));
  else
    atomicOr(reinterpret_cast<unsigned int*>(p), static_cast<unsigned int>(v));
}

// LDS position of word f (of width 4 * PER bytes) of chunk-local block lb:
// word f ^ key(lb) of the block.  With 64 four-byte banks, a block of
// S_WORDS * PER banks starts in one of G = 64 / (S_WORDS * PER) bank groups,
// chosen by the low log2(G) bits of lb.  One LDS instruction of an apply
// touches word f of 64 random blocks.  Unswizzled, they all sit in the G
// banks word f can occupy; keyed by lb mod s, the word within the group is
// still a function of the same low bits, so they reach only max(G, s) banks
// (8 for 8 x 32-bit blocks; measured on MI355X: 82 % of LDS-active cycles
// in bank conflicts).  Keyed by the bits above the group bits,
// key = (lb >> log2 G) mod s, the group and the word within it are
// independent and the lanes spread over all banks (also over 32 banks).
constexpr int log2_floor(int v) { return v > 1 ? 1 + log2_floor(v / 2) : 0; }
template <int S_WORDS, int PER = 1>
__device__ __forceinline__ uint32_t lds_key(uint32_t lb) {
  constexpr int kGroups = 64 / (S_WORDS * PER) > 1 ? 64 / (S_WORDS * PER) : 1;
  return (lb >> log2_floor(kGroups)) & (S_WORDS - 1);
}
template <int S_WORDS, int PER = 1>
__device__ __forceinline__ uint32_t lds_word(uint32_t lb, uint32_t f) {
  return (lb * S_WORDS) | (f ^ lds_key<S_WORDS, PER>(lb));
}
// The same for a 32-bit index t into the chunk image (W of width 4 * PER).
template <int S_WORDS, int PER>
__device__ __forceinline__ uint32_t lds_u32(uint32_t t) {
  const uint32_t e = t / PER;
  return lds_word<S_WORDS, PER>(e / S_WORDS, e & (S_WORDS - 1)) * PER + t % PER;
}

// What a record does to its block held in LDS, per layout: Z = 0 is the
// sectorized filter (every word of the block gets its pattern), Z > 0 the
// cache-sectorized filter with Z groups (one word per group; `k` then
// carries the bits per selected word).
template <typename W, int S_WORDS, int K, int Z>
struct BlockRule {
  CsbfLane<W, S_WORDS, Z, K, 1> ln;
  __device__ __forceinline__ BlockRule() : ln(0) {}
  __device__ __forceinline__ void add_lds(W* lds, uint32_t lb, uint32_t lo, uint32_t k) const {
#pragma unroll
    for (int i = 0; i < Z; ++i)
      lds_or<W>(&lds[lds_word<S_WORDS, sizeof(W) / 4>(lb, ln.word(i, lo))], ln.pattern(i, lo, k));
  }
};

template <typename W, int S_WORDS, int K>
struct BlockRule<W, S_WORDS, K, 0> {
  LanePatterns<W, S_WORDS, K, 1, S_WORDS> lp;
  __device__ __forceinline__ BlockRule() : lp(0) {}
  __device__ __forceinline__ void add_lds(W* lds, uint32_t lb, uint32_t lo, uint32_t k) const {
    if constexpr (sizeof(W) == 4 && S_WORDS >= 2) {
      // Words f and f + 1 (f even) sit at positions f ^ key and (f ^ key) ^ 1
      // of the block: one aligned 8-byte pair, so one 64-bit LDS atomic
      // covers both (their order within it flips with the key's low bit).
      const uint32_t key = lds_key<S_WORDS, 1>(lb);
#pragma unroll
      for (int f = 0; f < S_WORDS; f += 2) {
        const uint64_t p0 = lp.word(0, f, lo, k), p1 = lp.word(0, f + 1, lo, k);
        const uint64_t v = (key & 1u) ? (p0 << 32 | p1) : (p1 << 32 | p0);
        if (v) lds_or<uint64_t>(reinterpret_cast<uint64_t*>(lds + lb * S_WORDS + ((f ^ key) & ~1u)), v);
      }
    } else {
#pragma unroll
      for (int f = 0; f < S_WORDS; ++f) {
        const W pat = lp.word(0, f, lo, k);
        if (pat) lds_or<W>(&lds[lds_word<S_WORDS, sizeof(W) / 4>(lb, static_cast<uint32_t>(f))], pat);
      }
    }
  }
};

// Z = -1: the classic filter (Sec. II-A-1) seen as blocks of one 32-bit
// word; its records are (word << 32 | bit), one per pattern bit, so the
// rule sets a single bit.
template <typename W, int S_WORDS, int K>
struct BlockRule<W, S_WORDS, K, -1> {
  static_assert(sizeof(W) == 4 && S_WORDS == 1, "classic records address 32-bit words");
  __device__ __forceinline__ BlockRule() {}
  __device__ __forceinline__ void add_lds(W* lds, uint32_t lb, uint32_t bit, uint32_t) const {
    lds_or<W>(&lds[lb], W(1) << bit);
  }
};

// First pass of the classic filter: each key gives K records, one per
// position p (word p / 32, bit p mod 32); a thread hashes kPer / K keys
// per step.  a.n and the steps count keys.
template <int K, bool POW2, int D, int ROWS, bool SPLIT>
__global__ __launch_bounds__(kClassicThreads) void group_classic_kernel(GroupArgs a) {
  constexpr int kPer = kStep / kClassicThreads;  // records per thread per step
  constexpr int kKeys = kPer / K;                // keys per thread per step
  constexpr int kRecs = kKeys * K;               // records of them
  static_assert(kKeys >= 1, "at most kPer positions per key");
  __shared__ __attribute__((aligned(16))) GroupLds<D, ROWS> l;
  const uint32_t tid = threadIdx.x;
  for (uint32_t d = tid; d < D; d += kClassicThreads) l.cnt[d] = 0;
  __syncthreads();
  constexpr uint64_t kStepKeys = static_cast<uint64_t>(kClassicThreads) * kKeys;
  const uint32_t t0 = blockIdx.x * a.wg_steps;
  const uint32_t t1 = t0 + a.wg_steps < a.steps ? t0 + a.wg_steps : a.steps;
  for (uint32_t t = t0; t < t1; ++t) {
    const uint64_t s = t * kStepKeys;
    const uint32_t vkeys = static_cast<uint32_t>(a.n - s < kStepKeys ? a.n - s : kStepKeys);
    bool ok[kKeys];
    uint64_t r[kPer];
    uint32_t dg[kPer], rank[kPer];
#pragma unroll
    for (int u = 0; u < kKeys; ++u) {
      const uint32_t idx = tid + u * kClassicThreads;
      ok[u] = idx < vkeys;
      const uint64_t key = ok[u] ? a.keys[s + idx] : 0;
      const uint64_t h = xxh64_u64(key, a.hash_init);
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const uint64_t p = classic_position<POW2>(h, kSalts64.a[j], a.num_bits, a.bit_shift);
        const uint32_t word = static_cast<uint32_t>(p >> 5);
        r[u * K + j] = (static_cast<uint64_t>(word) << 32) | (static_cast<uint32_t>(p) & 31u);
        dg[u * K + j] = word >> a.shift;
      }
    }
#pragma unroll
    for (int j = kRecs; j < kPer; ++j) {
      r[j] = 0;
      dg[j] = 0;
    }
    const uint32_t row = (t - t0) % ROWS;
    auto in = [&](int j) { return j < kRecs && ok[j / K]; };
    group_positions(l, dg, in, row, kNoClip, rank, [] {}, [] {});
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (in(j)) l.stage[l.start[dg[j]] + rank[j]] = r[j];
    __syncthreads();
    if constexpr (SPLIT)
      RecordSplit{a.lo, a.blk}.template store_step<kClassicThreads>(t, l.stage, a.local_mask);
    else
      RecordPairs{a.rec}.template store_step<kClassicThreads>(t, l.stage, 0);
    if (row == ROWS - 1 || t + 1 == t1) group_flush_rows(l, a.table, a.stride, t - row, row + 1, a.digits);
  }
}

// Apply: one workgroup per chunk, or per slice of a chunk.  Bound by LDS
// bank conflicts of the ORs and by the memory latencies of a chunk's phases
// (runs, image, records), which the second workgroup of the CU covers; two
// records per lane in flight beside two in use are what 64 VGPRs hold (four
// and four spill: 0.945 ms against 0.913).  (A grid-stride
// loop would make the compiler keep every LDS address of the image copies in
// registers across chunks.)
// Two workgroups share a CU (their chunk images and unit lists take 156 KiB
// of its LDS): 8 waves per SIMD, 64 VGPRs.
template <typename W, int S_WORDS, int K, int Z, int UNIT>
__global__ __launch_bounds__(kApplyThreads, 8) void part_apply_kernel(ApplyArgs a) {
  __shared__ __attribute__((aligned(16))) uint32_t lds_raw[kChunkBytes / 4];
  __shared__ RunLds<kApplyThreads, kApplyList> runs;
  W* lds = reinterpret_cast<W*>(lds_raw);
  u32x4* lvec = reinterpret_cast<u32x4*>(lds_raw);
  const BlockRule<W, S_WORDS, K, Z> rule;
  const uint32_t blocks_per_chunk = 1u << a.chunk_shift;
  constexpr int kU = 2;  // records per lane: this many used while as many are loaded
  const uint32_t item = xcd_item(blockIdx.x, gridDim.x);
  uint32_t c = item;
  uint32_t si = 0, ns = 1;
  PartWork w{};
  if (a.work) {
    w = a.work[item];
    c = w.bucket;
    si = w.split;
    ns = w.nsplit;
  } else if (a.split > 1) {
    c = item / a.split;
    si = item % a.split;
    ns = a.split;
  }
  // the chunk's runs: one per step of the first pass, or of its high
  // digit's part of the second
  uint32_t e0 = 0, e1 = a.steps, row = c;
  if (a.steps == 0) {
    const uint32_t d1 = c >> a.low_bits;
    row = c & ((1u << a.low_bits) - 1);
    e0 = a.slot0[a.work ? w.item0 : d1 * a.per_digit];
    e1 = a.slot0[a.work ? w.item1 : (d1 + 1) * a.per_digit];
  }
  const uint32_t* entries = a.table + row * a.stride;
  if (ns > 1) {
    const uint64_t n = e1 - e0;
    e1 = e0 + static_cast<uint32_t>(n * (si + 1) / ns);
    e0 += static_cast<uint32_t>(n * si / ns);
  }
  W* words = static_cast<W*>(a.words);
  uint64_t num_blocks = a.num_blocks, local_chunk = c;
  if (a.nfilters > 1) {
    const PartFilter& f = a.filters[a.chunk_owner[c]];
    words = static_cast<W*>(f.words);
    num_blocks = f.num_blocks;
    local_chunk = c - f.chunk_base;
  }
  const uint64_t first_block = local_chunk << a.chunk_shift;
  const uint64_t nblk = num_blocks - first_block < blocks_per_chunk ? num_blocks - first_block
                                                                    : blocks_per_chunk;
  const uint32_t nbytes = static_cast<uint32_t>(nblk * S_WORDS * sizeof(W));
  const uint32_t nvec = nbytes / 16;
  const u32x4* gsrc = reinterpret_cast<const u32x4*>(words + first_block * S_WORDS);
  // The sole owner of a chunk starts from its words (copied into the
  // swizzled LDS image); one of several slices of a chunk accumulates its
  // bits only (zeroed image) and merges them with atomic OR.
  constexpr int kPer = static_cast<int>(sizeof(W) / 4);
  const uint32_t tail = nvec * 4 + threadIdx.x;  // < nbytes / 4 for at most 3 threads
  auto load_image = [&] {
    if (ns == 1) {
      constexpr int kFly = 2;  // vectors in flight
      static_assert(kVecPerThread % kFly == 0, "whole batches");
#pragma unroll 1
      for (int w = 0; w < kVecPerThread; w += kFly) {
        u32x4 v[kFly];
#pragma unroll
        for (int u = 0; u < kFly; ++u) {
          const uint32_t i = threadIdx.x + (w + u) * kApplyThreads;
          if (i < nvec) v[u] = gsrc[i];
        }
#pragma unroll
        for (int u = 0; u < kFly; ++u) {
          const uint32_t i = threadIdx.x + (w + u) * kApplyThreads;
          if (i < nvec) {
            if constexpr (S_WORDS == 1) {
              lvec[i] = v[u];
            } else {
#pragma unroll
              for (int q = 0; q < 4; ++q) lds_raw[lds_u32<S_WORDS, kPer>(4 * i + q)] = v[u][q];
            }
          }
        }
      }
      if (tail < nbytes / 4)
        lds_raw[lds_u32<S_WORDS, kPer>(tail)] = reinterpret_cast<const uint32_t*>(gsrc)[tail];
      return;
    }
#pragma unroll
    for (int u = 0; u < kVecPerThread; ++u) {
      const uint32_t i = threadIdx.x + u * kApplyThreads;
      if (i < nvec) lvec[i] = u32x4{0u, 0u, 0u, 0u};
    }
    if (tail < nbytes / 4) lds_raw[tail] = 0u;
  };
  const bool any = for_each_record<UNIT, kU>(
      runs, a.lo, a.blk, entries + e0, e0, e1 - e0, load_image, [&](uint64_t, bool ok, const SplitRecord& r) {
        if (ok) rule.add_lds(lds, r.blk, r.lo, a.k);
      });
  if (!any) return;  // untouched: no traffic at all
  u32x4* gdst = reinterpret_cast<u32x4*>(words + first_block * S_WORDS);
  if (ns == 1) {
#pragma unroll
    for (int u = 0; u < kVecPerThread; ++u) {
      const uint32_t i = threadIdx.x + u * kApplyThreads;
      if (i < nvec) {
        if constexpr (S_WORDS == 1) {
          gdst[i] = lvec[i];
        } else {
          gdst[i] = u32x4{lds_raw[lds_u32<S_WORDS, kPer>(4 * i)], lds_raw[lds_u32<S_WORDS, kPer>(4 * i + 1)],
                          lds_raw[lds_u32<S_WORDS, kPer>(4 * i + 2)],
                          lds_raw[lds_u32<S_WORDS, kPer>(4 * i + 3)]};
        }
      }
    }
    if (tail < nbytes / 4)
      reinterpret_cast<uint32_t*>(gdst)[tail] = lds_raw[lds_u32<S_WORDS, kPer>(tail)];
  } else {  // slices of one chunk merge with atomic OR of the words they set
    uint32_t* g32 = reinterpret_cast<uint32_t*>(gdst);
    for (uint32_t i = threadIdx.x; i < nbytes / 4; i += kApplyThreads) {
      const uint32_t v = lds_raw[lds_u32<S_WORDS, kPer>(i)];
      if (v) __hip_atomic_fetch_or(g32 + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

}  // namespace bfhip
