// bf_resident.hpp -- lookups in filters that fit the LDS: a workgroup copies
// the filter and tests its share of the keys there.
//
// A random read of the caches moves a line of 128 bytes per key and a CU takes
// one line per clock at best, so direct lookups fall from 300 G keys/s in
// 4 KiB (L1) to 150 in 64 KiB (L2); LDS reads are banked, and what is left is
// the vector work of the hash and the test.  Measured with 32-byte blocks,
// k = 8: 2^26 keys in 64 KiB 277 us -> 174 (386 G keys/s, 3.5 TB/s of keys and
// results); 4,096 filters of 4 KiB..16 MiB, half of 2^28 keys in filters of up
// to 160 KiB: 2.78 ms -> 2.35.  Items of 16,384 or 65,536 keys measured the
// same within 2 %: 32,768 keeps a launch's tail short and the copies rare.
#pragma once

#include "bf_batch_kernels.hpp"
#include "bf_partition.hpp"

namespace bfhip {

constexpr int kResidentThreads = 1024;
constexpr uint32_t kResidentKeys = 32768;  // of one workgroup, at most
// The largest filters of the two variants: two workgroups per CU, or one.
constexpr uint32_t kResidentBytes[2] = {80u << 10, 160u << 10};

// Layouts whose blocks fit the registers of such workgroups.
template <typename W, int S_WORDS>
constexpr bool lookup_resides() {
  return S_WORDS * sizeof(W) <= 32;
}

struct ResidentArgs {
  BatchFilter f;               // the filter, where there are no items
  const BatchFilter* filters;  // else those of the items
  const BatchTile* items;      // one per workgroup; meta is the key count
  uint64_t n;                  // without items: workgroup b tests keys [b * per, min(n, (b + 1) * per))
  uint32_t per;
  uint32_t k;
};

// The loads of a turn's keys are behind the last turn's results, as in the
// tiled batched lookup: a wait for keys covers no store of this turn.
template <typename W, int S_WORDS, int K, int BIG, typename SALTS>
__device__ __forceinline__ void resident_lookup(const ResidentArgs& a) {
  constexpr int KT = 2;
  constexpr uint32_t kTurn = KT * kResidentThreads;
  __shared__ u32x4 lds[kResidentBytes[BIG] / 16];
  const LanePatterns<W, S_WORDS, K, 1, S_WORDS> lp(0, SALTS{});
  BatchFilter f = a.f;
  uint64_t start = static_cast<uint64_t>(blockIdx.x) * a.per;
  uint32_t last = static_cast<uint32_t>(a.n - start < a.per ? a.n - start : a.per) - 1;
  if (a.items != nullptr) {
    const BatchTile t = read_constant(a.items + blockIdx.x);
    f = read_constant(a.filters + t.filter);
    start = t.key_start;
    last = t.meta - 1;
  }
  const uint64_t* keys = as_global(f.keys) + start;
  uint8_t* out = as_global(f.out) + start;
  uint64_t key[KT];
  auto load = [&](uint32_t base) {
#pragma unroll
    for (int q = 0; q < KT; ++q) {
      const uint32_t x = base + q * kResidentThreads + threadIdx.x;
      key[q] = __builtin_nontemporal_load(keys + (x < last ? x : last));
    }
  };
  load(0);
  const uint32_t nbytes = f.nb_lo * static_cast<uint32_t>(S_WORDS * sizeof(W));
  const char* words = as_global(static_cast<const char*>(f.words));
  if (nbytes % 16 == 0 && reinterpret_cast<uintptr_t>(words) % 16 == 0) {
    constexpr int kTurns = kResidentBytes[BIG] / 16 / kResidentThreads;
    u32x4 v[kTurns];
#pragma unroll
    for (int i = 0; i < kTurns; ++i) {
      const uint32_t x = i * kResidentThreads + threadIdx.x;
      if (x < nbytes / 16) v[i] = reinterpret_cast<const u32x4*>(words)[x];
    }
#pragma unroll
    for (int i = 0; i < kTurns; ++i) {
      const uint32_t x = i * kResidentThreads + threadIdx.x;
      if (x < nbytes / 16) lds[x] = v[i];
    }
  } else {
    for (uint32_t x = threadIdx.x; x < nbytes / 4; x += kResidentThreads)
      reinterpret_cast<uint32_t*>(lds)[x] = reinterpret_cast<const uint32_t*>(words)[x];
  }
  __syncthreads();
  const W* filter = reinterpret_cast<const W*>(lds);
  uint32_t res[KT] = {};
  uint32_t from = last + 1;  // of the keys that res is for
  auto store = [&] {
#pragma unroll
    for (int q = 0; q < KT; ++q) {
      const uint32_t x = from + q * kResidentThreads + threadIdx.x;
      if (x <= last) __builtin_nontemporal_store(static_cast<uint8_t>(res[q]), out + x);
    }
  };
  // opaque: the compiler would merge the first load with the loop's, at its head
#pragma unroll
  for (int q = 0; q < KT; ++q) asm("" : "+v"(key[q]));
  for (uint32_t base = 0; base <= last; base += kTurn) {
    uint32_t lo[KT];
    W v[KT][S_WORDS];
#pragma unroll
    for (int q = 0; q < KT; ++q) {
      const uint64_t h = xxh64_u64(key[q], f.hash_init);
      lo[q] = static_cast<uint32_t>(h);
      load_words<W, S_WORDS>(filter + block_of(h, f.nb_lo, 0) * S_WORDS, v[q]);
    }
    store();
    load(base + kTurn);
#pragma unroll
    for (int q = 0; q < KT; ++q) {
      W miss = 0;
#pragma unroll
      for (int w = 0; w < S_WORDS; ++w) miss |= lp.word(0, w, lo[q], a.k) & ~v[q][w];
      res[q] = miss == 0 ? 1u : 0u;
    }
    from = base;
  }
  store();
}

// Adds: the share's bits are set in an image in LDS, which is then merged
// into the filter; words that hold their bits already are only read.  The
// direct adds pay a memory-side atomic per word pair of a block (20..27 G/s),
// the partitioned construction two passes over 8-byte records.  Measured with
// 32-byte blocks, k = 8: 2^20 keys into 4 KiB 299 us -> 16, into 64 KiB 48 ->
// 26; 2^27 keys over 1,024 filters of 32 KiB 0.36 ms; 4,096 filters of
// 4 KiB..16 MiB and 2^28 keys (half of them in filters of up to 160 KiB)
// 4.23 ms -> 3.18.
template <typename W, int S_WORDS, int K, int BIG, int Z>
__device__ __forceinline__ void resident_add(const ResidentArgs& a) {
  constexpr int KT = 2;
  constexpr uint32_t kTurn = KT * kResidentThreads;
  constexpr int kPer = sizeof(W) / 4;
  __shared__ u32x4 lds[kResidentBytes[BIG] / 16];
  const BlockRule<W, S_WORDS, K, Z> rule;
  BatchFilter f = a.f;
  uint64_t start = static_cast<uint64_t>(blockIdx.x) * a.per;
  uint32_t last = static_cast<uint32_t>(a.n - start < a.per ? a.n - start : a.per) - 1;
  if (a.items != nullptr) {
    const BatchTile t = read_constant(a.items + blockIdx.x);
    f = read_constant(a.filters + t.filter);
    start = t.key_start;
    last = t.meta - 1;
  }
  const uint64_t* keys = as_global(f.keys) + start;
  uint64_t key[KT];
  auto load = [&](uint32_t base) {
#pragma unroll
    for (int q = 0; q < KT; ++q) {
      const uint32_t x = base + q * kResidentThreads + threadIdx.x;
      key[q] = __builtin_nontemporal_load(keys + (x < last ? x : last));
    }
  };
  load(0);
  const uint32_t words = f.nb_lo * (S_WORDS * kPer);  // of 32 bits
  for (uint32_t x = threadIdx.x; x < (words + 3) / 4; x += kResidentThreads) lds[x] = u32x4{0u, 0u, 0u, 0u};
  __syncthreads();
#pragma unroll
  for (int q = 0; q < KT; ++q) asm("" : "+v"(key[q]));
  for (uint32_t base = 0; base <= last; base += kTurn) {
    uint32_t lo[KT], blk[KT];
#pragma unroll
    for (int q = 0; q < KT; ++q) {
      const uint64_t h = xxh64_u64(key[q], f.hash_init);
      lo[q] = static_cast<uint32_t>(h);
      blk[q] = static_cast<uint32_t>(block_of(h, f.nb_lo, 0));
    }
    load(base + kTurn);
    // a lane past the last key sets that key's bits again
#pragma unroll
    for (int q = 0; q < KT; ++q) rule.add_lds(reinterpret_cast<W*>(lds), blk[q], lo[q], a.k);
  }
  __syncthreads();
  uint32_t* g = as_global(static_cast<uint32_t*>(f.words));
  constexpr int kFly = 8;
  for (uint32_t x0 = threadIdx.x; x0 < words; x0 += kFly * kResidentThreads) {
    uint32_t v[kFly], have[kFly];
#pragma unroll
    for (int i = 0; i < kFly; ++i) {
      const uint32_t x = x0 + i * kResidentThreads;
      have[i] = g[x < words ? x : words - 1];
    }
#pragma unroll
    for (int i = 0; i < kFly; ++i) {
      const uint32_t x = x0 + i * kResidentThreads;
      v[i] = x < words ? reinterpret_cast<const uint32_t*>(lds)[lds_u32<S_WORDS, kPer>(x)] & ~have[i] : 0u;
      if (v[i] != 0) __hip_atomic_fetch_or(g + x, v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

template <typename W, int S_WORDS, int K, int BIG>
__global__ __launch_bounds__(kResidentThreads, BIG ? 4 : 8) void bf_resident_add_kernel(ResidentArgs a) {
  resident_add<W, S_WORDS, K, BIG, 0>(a);
}

template <typename W, int S_WORDS, int K, int BIG>
__global__ __launch_bounds__(kResidentThreads, BIG ? 4 : 8) void bf_resident_kernel(ResidentArgs a) {
  resident_lookup<W, S_WORDS, K, BIG, PaperSalts>(a);
}

}  // namespace bfhip
