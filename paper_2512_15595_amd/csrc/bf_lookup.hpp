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
// Where many keys repeat, the caches answer direct lookups faster than any
// grouping could: a sample of the keys decides before anything is grouped
// (bf_lookup.hip), and then the return step looks up all keys.  2^26 keys in
// 32 MiB, us direct / grouped / by the sample: different ones 1074 / 439 /
// 444, a tenth of them one key 975 / 658 / 658, half 578 / 700 / 605, all of
// them 200 / 858 / 169.
//
// Measured on MI355X (256-bit blocks, k = 8; us, direct -> grouped): 2^26 keys
// in 16 MiB 904 -> 427, 32 MiB 1074 -> 444, 128 MiB 1254 -> 744, 512 MiB 1256 ->
// 845, 1 GiB 1272 -> 983; 2^28 keys in 1 GiB 5116 -> 3140.
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
  const uint32_t* direct;  // as in GroupArgs
};

// Results of a second-pass step to the first pass's slots.
struct ReturnSlotsArgs {
  const uint16_t* place;
  const uint8_t* res;      // by slot of the sorted steps
  uint8_t* out;            // by slot of the first pass
  const uint32_t* units;   // where a step was read from
  const uint32_t* nsteps;  // the number of steps
  const uint32_t* direct;
};

struct ReturnArgs {
  const uint16_t* place;
  const uint8_t* res;      // by slot of the sorted steps: 0, 1 or kUntested
  uint8_t* out;            // by key
  uint64_t n;
  const uint32_t* direct;  // nonzero: every key is looked up here
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
  if (*a.direct != 0) return;
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
// 16-byte vectors where it is aligned, bytes elsewhere.  Keys without a
// result are looked up here, a key per lane, and join the others in LDS: the
// listed ones (beyond their run's clip), or with a.direct all of the step's.
template <typename W, int S_WORDS, int K, typename SALTS>
__device__ __forceinline__ void return_keys(const ReturnArgs& a) {
  static_assert(kStep / kReturnThreads == 16, "one 16-byte vector of results per thread");
  __shared__ __attribute__((aligned(16))) uint8_t res[kStep];
  __shared__ uint16_t list[kStep];
  __shared__ uint32_t listed;
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint64_t s = static_cast<uint64_t>(blockIdx.x) * kStep;
  const uint32_t valid = static_cast<uint32_t>(a.n - s < kStep ? a.n - s : kStep);
  const LanePatterns<W, S_WORDS, K, 1, S_WORDS> lp(0, SALTS{});
  // res[key_at(i)] for i < n, the next key of a lane loaded behind this one's
  // block.  (Two and four at a time: the registers cost the return of tested
  // keys more, 940 -> 980 us for 2^26 keys in 1 GiB, than they gain here.)
  auto look_up = [&](uint32_t n, auto key_at) {
    if (n == 0) return;
    uint32_t p = key_at(tid < n ? tid : n - 1);
    uint64_t key = __builtin_nontemporal_load(a.keys + s + p);
#pragma unroll 1
    for (uint32_t i = tid; i < n; i += kReturnThreads) {
      const uint32_t at = p;
      const uint64_t h = xxh64_u64(key, a.hash_init);
      W w[S_WORDS];
      load_words<W, S_WORDS>(static_cast<const W*>(a.words) +
                                 static_cast<uint64_t>(block_of(h, a.nb_lo, a.nb_hi_mask)) * S_WORDS, w);
      p = key_at(i + kReturnThreads < n ? i + kReturnThreads : n - 1);
      key = __builtin_nontemporal_load(a.keys + s + p);
      W miss = 0;
#pragma unroll
      for (int x = 0; x < S_WORDS; ++x) miss |= lp.word(0, x, static_cast<uint32_t>(h), a.k) & ~w[x];
      res[at] = miss == 0 ? 1 : 0;
    }
  };
  u32x4 v;
  if (*a.direct != 0) {
    look_up(valid, [](uint32_t i) { return i; });
    __syncthreads();
    v = reinterpret_cast<const u32x4*>(res)[tid];
  } else {
    if (tid == 0) listed = 0;
    reinterpret_cast<u32x4*>(res)[tid] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(a.res + s) + tid);
    const u32x4* places = reinterpret_cast<const u32x4*>(a.place + s + 16 * tid);
    const u32x4 p[2] = {__builtin_nontemporal_load(places), __builtin_nontemporal_load(places + 1)};
    __syncthreads();
    uint32_t untested = 0;  // of the thread's 16 keys
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[q] = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t place = p[q / 2][2 * (q % 2) + i / 2] >> (16 * (i % 2)) & 0xffffu;
        uint32_t r = res[place & (kStep - 1)];
        if (place == kNoPlace) r = kUntested;
        untested |= (r >> 1 & 1u) << (4 * q + i);
        v[q] |= r << (8 * i);
      }
    }
    if (16 * tid + 16 > valid) untested &= 16 * tid < valid ? (1u << (valid - 16 * tid)) - 1 : 0u;
    if (__syncthreads_or(untested != 0 ? 1 : 0)) {
      reinterpret_cast<u32x4*>(res)[tid] = v;
      uint32_t incl = __popc(untested);
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t x = __shfl_up(incl, off, 64);
        if (lane >= static_cast<uint32_t>(off)) incl += x;
      }
      uint32_t at = 0;
      if (lane == 63 && incl != 0) at = atomicAdd(&listed, incl);
      at = __shfl(at, 63, 64) + incl - __popc(untested);
      for (uint32_t u = untested; u != 0; u &= u - 1) list[at++] = static_cast<uint16_t>(16 * tid + __ffs(u) - 1);
      __syncthreads();
      look_up(listed, [&](uint32_t i) -> uint32_t { return list[i]; });
      __syncthreads();
      v = reinterpret_cast<const u32x4*>(res)[tid];
    }
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
