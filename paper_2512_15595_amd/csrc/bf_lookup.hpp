// bf_lookup.hpp -- grouped lookup: bulk contains of a filter larger than an
// XCD's L2, with the keys grouped by filter chunk so that every chunk is
// read once, into LDS, and tested there.
//
// A direct lookup fetches one 128-byte line per key from beyond the L2, at
// the line rate of the memory (57 G lines/s on MI355X; the 256 lines a CU's
// L1 holds are in flight for one memory latency).  Here instead
//   group    keys -> hashed records, each step of 8,192 sorted by chunk (or
//            by high digit, and once more by chunk: regroup), and per key
//            its place in the sorted step;
//   test     per chunk: the words into LDS, every record of the chunk's runs
//            tested there, one result byte at the record's slot;
//   return   per step: the results in key order (for two digits a step of
//            the second pass first returns to the slots it was read from).
// Grouping passes and table of runs are those of bf_group.hpp.  Results are
// exactly those of the direct lookup.
//
// Repeated keys would load one chunk's workgroups with most of the records,
// so a run is clipped five standard deviations over the length that
// uniformly hashed keys give it; the keys beyond (of such keys hardly any)
// are looked up directly by the return step, spread over all workgroups.
//
// Measured on MI355X (256-bit blocks, k = 8, half of the keys present; us,
// direct -> grouped): 2^26 keys in 16 MiB 927 -> 442, 32 MiB 1120 -> 462,
// 64 MiB 1246 -> 529, 256 MiB 1336 -> 755, 1 GiB 1274 -> 960; 2^28 keys in
// 1 GiB 5070 -> 2951.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bf_group.hpp"
#include "bf_hash.hpp"
#include "bf_kernels.hpp"

namespace bfhip {

constexpr int kTestThreads = 1024;
constexpr int kReturnThreads = 512;
constexpr int kLookupDigits = 512;  // chunks up to which one digit is enough

// The chunk of words a test workgroup holds in LDS: 128 KiB (one workgroup
// per CU, longer runs) or 64 KiB (two per CU, so that one loads its words
// while the other tests).
constexpr int test_chunk_bytes(bool two) { return two ? 64 * 1024 : 128 * 1024; }

struct TestArgs {
  const void* words;
  uint64_t nbytes;
  const uint32_t* table;   // runs by chunk (one digit) or by second digit
  uint64_t stride;
  const uint32_t* lo;
  const uint16_t* blk;
  uint8_t* res;            // per record slot: 0 or 1 (slots of no visible record: not written)
  const uint32_t* slot0;   // two digits: first step of every second-pass item
  uint32_t steps;          // one digit: table entries per chunk (else 0)
  uint32_t per_digit;
  uint32_t low_bits;
  uint32_t split;          // workgroups per chunk
  uint32_t k;
};

// Results of a second-pass step to the first pass's slots.
struct ReturnSlotsArgs {
  const uint16_t* place;
  const uint8_t* res;      // by slot of the sorted steps
  uint8_t* out;            // by slot of the first pass
  const uint32_t* units;   // where a step was read from
  const uint32_t* nsteps;  // the number of steps
};

struct ReturnArgs {
  const uint16_t* place;
  const uint8_t* res;      // by slot of the sorted steps: 0, 1 or kUntested
  uint8_t* out;            // by key
  uint64_t n;
  // for the keys that were not tested
  const void* words;
  const uint64_t* keys;
  uint64_t hash_init;
  uint32_t nb_lo;
  uint32_t nb_hi_mask;
  uint32_t k;
};
constexpr uint8_t kUntested = 2;

// LDS position of 16-byte unit q of chunk-local block lb (NU units per
// block): the units of a block are permuted by the block bits above those
// that choose its place in a 256-byte row, so that the lanes of one LDS
// instruction, which read unit q of 64 random blocks, spread over all banks.
template <int NU>
__device__ __forceinline__ uint32_t test_unit(uint32_t lb, uint32_t q) {
  constexpr int kGroups = 16 / NU > 1 ? 16 / NU : 1;
  return lb * NU + (q ^ ((lb / kGroups) & (NU - 1)));
}

template <typename W, int S_WORDS, int K, bool TWO, typename SALTS>
__device__ __forceinline__ void test_chunk(const TestArgs& a) {
  constexpr uint32_t kChunk = test_chunk_bytes(TWO);
  // short runs (one digit: up to 512 chunks of a step) in units of 8 slots
  constexpr int kUnitSlots = TWO ? 16 : 8;
  constexpr int kFly = TWO ? 2 : 6;
  constexpr int kList = TWO ? 1536 : 4096;
  constexpr int kBlockBytes = S_WORDS * static_cast<int>(sizeof(W));
  constexpr int NU = kBlockBytes / 16;
  __shared__ u32x4 lds[kChunk / 16];
  __shared__ RunLds<kTestThreads, kList> runs;
  const LanePatterns<W, S_WORDS, K, 1, S_WORDS> lp(0, SALTS{});
  const uint32_t tid = threadIdx.x;
  const uint32_t item = xcd_item(blockIdx.x, gridDim.x);
  const uint32_t c = item / a.split, si = item % a.split;
  uint32_t e0 = 0, e1 = a.steps, row = c;
  if constexpr (TWO) {
    const uint32_t d1 = c >> a.low_bits;
    row = c & ((1u << a.low_bits) - 1);
    e0 = a.slot0[d1 * a.per_digit];
    e1 = a.slot0[(d1 + 1) * a.per_digit];
  }
  const uint64_t n = e1 - e0;
  e1 = e0 + static_cast<uint32_t>(n * (si + 1) / a.split);
  e0 += static_cast<uint32_t>(n * si / a.split);
  const char* src = static_cast<const char*>(a.words) + static_cast<uint64_t>(c) * kChunk;
  const uint64_t left = a.nbytes - static_cast<uint64_t>(c) * kChunk;
  const uint32_t nbytes = left < kChunk ? static_cast<uint32_t>(left) : kChunk;
  auto load_words_image = [&] {
    constexpr int kVec = kChunk / 16 / kTestThreads, kAtOnce = TWO ? 2 : 4;
#pragma unroll 1
    for (int w = 0; w < kVec; w += kAtOnce) {
      u32x4 v[kAtOnce];
#pragma unroll
      for (int u = 0; u < kAtOnce; ++u) {
        const uint32_t i = tid + (w + u) * kTestThreads;
        if (i < nbytes / 16) v[u] = reinterpret_cast<const u32x4*>(src)[i];
      }
#pragma unroll
      for (int u = 0; u < kAtOnce; ++u) {
        const uint32_t i = tid + (w + u) * kTestThreads;
        if (i < nbytes / 16) {
          if constexpr (NU > 1)
            lds[test_unit<NU>(i / NU, i % NU)] = v[u];
          else
            lds[i] = v[u];
        }
      }
    }
    if (tid < nbytes % 16 / 4)
      reinterpret_cast<uint32_t*>(lds)[nbytes / 16 * 4 + tid] =
          reinterpret_cast<const uint32_t*>(src)[nbytes / 16 * 4 + tid];
  };
  for_each_record<kUnitSlots, kFly>(
      runs, a.lo, a.blk, a.table + row * a.stride + e0, e0, e1 - e0, load_words_image,
      [&](uint64_t slot, bool ok, const SplitRecord& r) {
        W miss = 0;
        if constexpr (NU > 1) {
          constexpr int kPerUnit = 16 / static_cast<int>(sizeof(W));
#pragma unroll
          for (int q = 0; q < NU; ++q) {
            const u32x4 x = lds[test_unit<NU>(r.blk, static_cast<uint32_t>(q))];
            W v[kPerUnit];
            __builtin_memcpy(v, &x, 16);
#pragma unroll
            for (int f = 0; f < kPerUnit; ++f) miss |= lp.word(0, q * kPerUnit + f, r.lo, a.k) & ~v[f];
          }
        } else {
          W v[S_WORDS];
          load_words<W, S_WORDS>(reinterpret_cast<const W*>(lds) + r.blk * S_WORDS, v);
#pragma unroll
          for (int f = 0; f < S_WORDS; ++f) miss |= lp.word(0, f, r.lo, a.k) & ~v[f];
        }
        if (ok) a.res[slot] = miss == 0 ? 1 : 0;
      });
}

// A step's results in key order.  `out` may have any alignment: whole
// 16-byte vectors where it is aligned, bytes elsewhere.
template <typename W, int S_WORDS, int K, typename SALTS>
__device__ __forceinline__ void return_keys(const ReturnArgs& a) {
  static_assert(kStep / kReturnThreads == 16, "one 16-byte vector of results per thread");
  __shared__ __attribute__((aligned(16))) uint8_t res[kStep];
  const uint32_t tid = threadIdx.x;
  const uint64_t s = static_cast<uint64_t>(blockIdx.x) * kStep;
  const uint32_t valid = static_cast<uint32_t>(a.n - s < kStep ? a.n - s : kStep);
  reinterpret_cast<u32x4*>(res)[tid] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(a.res + s) + tid);
  const u32x4* places = reinterpret_cast<const u32x4*>(a.place + s + 16 * tid);
  const u32x4 p[2] = {__builtin_nontemporal_load(places), __builtin_nontemporal_load(places + 1)};
  __syncthreads();
  u32x4 v;
  bool untested = false;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t x = p[q / 2][2 * (q % 2)], y = p[q / 2][2 * (q % 2) + 1];
    untested = untested || (x & 0xffffu) == kNoPlace || x >> 16 == kNoPlace || (y & 0xffffu) == kNoPlace ||
               y >> 16 == kNoPlace;
    v[q] = res[x & (kStep - 1)] | static_cast<uint32_t>(res[x >> 16 & (kStep - 1)]) << 8 |
           static_cast<uint32_t>(res[y & (kStep - 1)]) << 16 | static_cast<uint32_t>(res[y >> 16 & (kStep - 1)]) << 24;
    untested = untested || (v[q] & 0x02020202u) != 0;
  }
  if (__syncthreads_or(untested ? 1 : 0)) {
    // some keys of the step: looked up directly, a key per lane
    const LanePatterns<W, S_WORDS, K, 1, S_WORDS> lp(0, SALTS{});
#pragma unroll 2
    for (uint32_t p = tid; p < valid; p += kReturnThreads) {
      const uint32_t place = a.place[s + p];
      uint32_t r = place == kNoPlace ? kUntested : res[place];
      if (r == kUntested) {
        const uint64_t h = xxh64_u64(a.keys[s + p], a.hash_init);
        r = test_block<W, S_WORDS, K, 1, S_WORDS>(static_cast<const W*>(a.words),
                                                  block_of(h, a.nb_lo, a.nb_hi_mask), static_cast<uint32_t>(h), lp,
                                                  a.k) ? 1u : 0u;
      }
      a.out[s + p] = static_cast<uint8_t>(r);
    }
    return;
  }
  uint8_t* out = a.out + s + 16 * tid;
  if (reinterpret_cast<uintptr_t>(a.out) % 16 == 0 && 16 * tid + 16 <= valid) {
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(out));
  } else {
#pragma unroll
    for (int q = 0; q < 16; ++q)
      if (16 * tid + q < valid) out[q] = static_cast<uint8_t>(v[q / 4] >> (8 * (q % 4)));
  }
}

template <typename W, int S_WORDS, int K>
__global__ __launch_bounds__(kReturnThreads) void lookup_return_kernel(ReturnArgs a) {
  return_keys<W, S_WORDS, K, PaperSalts>(a);
}

template <typename W, int S_WORDS, int K, bool TWO>
__global__ __launch_bounds__(kTestThreads, TWO ? 8 : 4) void lookup_test_kernel(TestArgs a) {
  test_chunk<W, S_WORDS, K, TWO, PaperSalts>(a);
}

}  // namespace bfhip
