// bf_batch_kernels.hpp -- one persistent kernel over the tiles of many filters.
//
// Each tile is up to 256 * KT keys of one filter.  The tile list is ordered
// on the host so that slot i is only ever taken by workgroups with
// blockIdx.x = i (mod 8) (the grid is a multiple of 8 and strides over the
// slots); workgroups are dispatched to the 8 XCDs round-robin, so all tiles
// of a filter run on one XCD and the filter's lines stay in that XCD's L2.
// The execution mapping of a tile is compiled per size class of its filter
// from the autotuned table, so one launch uses several mappings.
#pragma once

#include "bf_kernels.hpp"
#include "bf_tuned.hpp"

namespace bfhip {

struct BatchFilter {  // 48 bytes: one filter (or one request on a filter)
  void* words;
  uint64_t hash_init;
  uint32_t nb_lo;
  uint32_t nb_hi_mask;
  const uint64_t* keys;  // tile key_start indexes into keys / out
  uint8_t* out;
  uint64_t reserved;
};

struct BatchTile {  // 16 bytes
  uint64_t key_start;  // offset of the tile's first key in the key / result arrays
  uint32_t filter;
  uint32_t meta;       // bits 0..15 key count, 16..17 size class, 18 packed loads allowed
};

constexpr uint32_t kTileCountMask = 0xffffu;
constexpr int kTileClassShift = 16;
constexpr uint32_t kTileVecBit = 1u << 18;

struct BatchArgs {
  const BatchFilter* filters;
  const BatchTile* tiles;
  uint64_t ntiles;
  uint32_t k;
  uint32_t pad;
};

// The mapping a size class runs with (256-thread workgroups: tiles are
// planned on the host at that size).  Runtime-k layouts use one lane per key
// and one key per lane, as the single-filter path does.
template <typename W, int S_WORDS, int K, int OP, int CLS>
constexpr MapSpec batch_map() {
  if constexpr (K == 0) {
    return MapSpec{1, static_cast<uint32_t>(S_WORDS), 1, 32, 0, kBlockThreads, true};
  } else {
    // batched launches are large: the tuned rows of large batches at k
    return tuned_map(OP, 8 * static_cast<int>(sizeof(W)), S_WORDS, CLS, K, 1);
  }
}

template <typename W, int S_WORDS, int K, int OP, int CLS, typename SALTS>
__device__ __forceinline__ void batch_tile(const BatchArgs& a, const BatchTile& t,
                                           const BatchFilter& f, const FilterView& fv) {
  constexpr MapSpec m = batch_map<W, S_WORDS, K, OP, CLS>();
  constexpr int kTheta = static_cast<int>(m.theta);
  constexpr int kPhi = static_cast<int>(m.phi);
  constexpr int kKt = static_cast<int>(m.kt);
  static_assert(kTheta * kPhi <= S_WORDS && kTheta <= 16, "tuned mapping fits the block");
  constexpr bool kAtom64 = OP == 0 && sizeof(W) == 4 && kPhi >= 2 && m.atomic_bits == 64;
  const LanePatterns<W, S_WORDS, K, kTheta, kPhi> lp((threadIdx.x & 63u) & (kTheta - 1), SALTS{});
  const uint32_t count = t.meta & kTileCountMask;
  const bool vec_ok = (t.meta & kTileVecBit) != 0;
  if constexpr (OP == 0) {
    add_tile<W, S_WORDS, K, kTheta, kPhi, kKt, kAtom64>(fv, f.keys + t.key_start, count, vec_ok,
                                                        a.k, lp);
  } else {
    contains_tile<W, S_WORDS, K, kTheta, kPhi, kKt>(fv, f.keys + t.key_start, f.out + t.key_start,
                                                    count, vec_ok, a.k, lp);
  }
}

// Whether every size class looks a key up with one lane and the same number
// of keys per lane: then the lookups' tile walk is pipelined.
template <typename W, int S_WORDS, int K>
constexpr bool batch_lookup_pipelines() {
  constexpr MapSpec m0 = batch_map<W, S_WORDS, K, 1, 0>(), m1 = batch_map<W, S_WORDS, K, 1, 1>(),
                    m2 = batch_map<W, S_WORDS, K, 1, 2>();
  return m0.theta == 1 && m1.theta == 1 && m2.theta == 1 && m0.kt == m1.kt && m0.kt == m2.kt &&
         S_WORDS * sizeof(W) <= 32;
}

// An object that nothing writes while the kernel runs (tiles, the filter
// table): read as a constant it takes scalar loads, which a kernel's stores
// would otherwise forbid.
template <typename T>
__device__ __forceinline__ T read_constant(const T* p) {
  using Word = const __attribute__((address_space(4))) uint32_t;
  Word* w = (Word*)(p);
  uint32_t raw[sizeof(T) / 4];
#pragma unroll
  for (uint32_t x = 0; x < sizeof(T) / 4; ++x) raw[x] = w[x];
  return __builtin_bit_cast(T, raw);
}

// A pointer to global memory that came from such an object: without the cast
// its accesses would be flat ones, whose waits cover the scalar loads too.
template <typename T>
__device__ __forceinline__ T* as_global(T* p) {
  return (T*)(__attribute__((address_space(1))) T*)(reinterpret_cast<uintptr_t>(p));
}

// Lookups with the next tile's loads in flight: otherwise a workgroup pays a
// tile's chain of dependent loads (tile, filter, keys, blocks) in full for
// every 512 keys.  Tiles are read three turns ahead, filters two, keys one;
// the keys are loaded behind this tile's blocks, because loads return in
// order and a wait for the blocks then leaves the keys in flight.  Measured
// on MI355X over 4,096 filters of 4 KiB..16 MiB and 2^28 keys: 3.01 -> 2.78 ms
// (4 KiB filters 221 -> 250 G keys/s, 64 KiB 123 -> 139, 1 MiB 66 -> 65:
// from 512 KiB on the blocks' fetches from beyond the L2 bound it).  Bringing
// the next filter to the L2 one turn ahead, by vector or by scalar loads,
// changed none of these.
template <typename W, int S_WORDS, int K, typename SALTS>
__device__ __forceinline__ void batch_lookup_tiles(const BatchArgs& a) {
  constexpr int KT = static_cast<int>(batch_map<W, S_WORDS, K, 1, 0>().kt);
  const LanePatterns<W, S_WORDS, K, 1, S_WORDS> lp(0, SALTS{});
  const uint64_t g = gridDim.x;
  uint64_t i = blockIdx.x;
  if (i >= a.ntiles) return;
  const uint64_t last_tile = a.ntiles - 1;
  auto tile_at = [&](uint64_t i) {
    BatchTile t = read_constant(a.tiles + (i < last_tile ? i : last_tile));
    t.meta = i <= last_tile ? t.meta : 0u;
    return t;
  };
  auto filter_of = [&](const BatchTile& t) { return read_constant(a.filters + t.filter); };
  // One key per lane and load, whatever the alignment, and every load made on
  // every path: the compiler can then count the loads that it need not wait
  // for.  Lanes past the count repeat the last key, a slot without keys (the
  // padding, the end of the walk) reads the filter table instead.
  auto load = [&](const BatchTile& t, const BatchFilter& f, uint64_t (&key)[KT]) {
    const uint32_t count = t.meta & kTileCountMask;
    const uint64_t* keys = as_global(count != 0 ? f.keys + t.key_start : reinterpret_cast<const uint64_t*>(a.filters));
    const uint32_t last = count != 0 ? count - 1 : 0;
#pragma unroll
    for (int q = 0; q < KT; ++q) {
      const uint32_t x = q * kBlockThreads + threadIdx.x;
      key[q] = __builtin_nontemporal_load(keys + (x < last ? x : last));
    }
  };
  BatchTile t = tile_at(i), t1 = tile_at(i + g), t2 = tile_at(i + 2 * g);
  BatchFilter f = filter_of(t), f1 = filter_of(t1);
  uint64_t key[KT];
  load(t, f, key);
  // Opaque here, or the compiler merges this load with the loop's and moves
  // both to the loop's head, where nothing hides them.
#pragma unroll
  for (int q = 0; q < KT; ++q) asm("" : "+v"(key[q]));
  // A tile's results are stored behind the next tile's blocks: a wait for
  // keys then never waits for a store that was just issued.
  uint32_t res[KT] = {};
  uint8_t* out = nullptr;
  uint32_t out_count = 0;
  auto store = [&] {
#pragma unroll
    for (int q = 0; q < KT; ++q) {
      const uint32_t x = q * kBlockThreads + threadIdx.x;
      if (x < out_count) __builtin_nontemporal_store(static_cast<uint8_t>(res[q]), out + x);
    }
  };
  for (; i < a.ntiles; i += g) {
    const BatchTile t3 = tile_at(i + 3 * g);
    const BatchFilter f2 = filter_of(t2);
    uint32_t lo[KT];
    W v[KT][S_WORDS];
#pragma unroll
    for (int q = 0; q < KT; ++q) {
      const uint64_t h = xxh64_u64(key[q], f.hash_init);
      lo[q] = static_cast<uint32_t>(h);
      load_words<W, S_WORDS>(as_global(static_cast<const W*>(f.words)) +
                                 static_cast<uint64_t>(block_of(h, f.nb_lo, f.nb_hi_mask)) * S_WORDS, v[q]);
    }
    store();
    load(t1, f1, key);
#pragma unroll
    for (int q = 0; q < KT; ++q) {
      W miss = 0;
#pragma unroll
      for (int w = 0; w < S_WORDS; ++w) miss |= lp.word(0, w, lo[q], a.k) & ~v[q][w];
      res[q] = miss == 0 ? 1u : 0u;
    }
    out = as_global(f.out) + t.key_start;
    out_count = t.meta & kTileCountMask;
    t = t1;
    f = f1;
    t1 = t2;
    f1 = f2;
    t2 = t3;
  }
  store();
}

// The tile walk, for the pattern multipliers SALTS (bf_hash.hpp's salts,
// or another filter format's table).
template <typename W, int S_WORDS, int K, int OP, typename SALTS>
__device__ __forceinline__ void batch_tiles(const BatchArgs& a) {
  if constexpr (OP == 1 && batch_lookup_pipelines<W, S_WORDS, K>()) {
    batch_lookup_tiles<W, S_WORDS, K, SALTS>(a);
    return;
  }
  for (uint64_t i = blockIdx.x; i < a.ntiles; i += gridDim.x) {
    const BatchTile t = a.tiles[i];
    if ((t.meta & kTileCountMask) == 0) continue;  // padding slot
    const BatchFilter f = a.filters[t.filter];
    const FilterView fv{f.words, f.hash_init, f.nb_lo, f.nb_hi_mask};
    switch ((t.meta >> kTileClassShift) & 3u) {
      case 0: batch_tile<W, S_WORDS, K, OP, 0, SALTS>(a, t, f, fv); break;
      case 1: batch_tile<W, S_WORDS, K, OP, 1, SALTS>(a, t, f, fv); break;
      default: batch_tile<W, S_WORDS, K, OP, 2, SALTS>(a, t, f, fv); break;
    }
  }
}

template <typename W, int S_WORDS, int K, int OP>
__global__ __launch_bounds__(kBlockThreads) void bf_batch_kernel(BatchArgs a) {
  batch_tiles<W, S_WORDS, K, OP, PaperSalts>(a);
}

}  // namespace bfhip
