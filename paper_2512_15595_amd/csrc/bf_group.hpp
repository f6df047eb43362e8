// bf_group.hpp -- grouping of hashed records by a digit, the first half of
// the partitioned construction and of the grouped lookup.
//
// A workgroup takes its records a step (8,192) at a time, counting-sorts a
// step in LDS by digit and writes it out whole: the records of step t fill
// slots [t * 8192, (t + 1) * 8192) of the record buffer, those of one digit
// as one run, and the table holds for every (digit, step) where the run
// starts and how many records it has.  All stores are contiguous and no
// record has to be fitted into a bucket.  A reader of digit d collects its
// runs from all steps: for_each_record below.
//
// Why whole steps: a pass that writes every digit's run to the digit's own
// bucket is bound by those short unaligned stores.  Measured on MI355X with
// 2^28 keys (6-byte records and a 4-byte word per key): 1.12 ms for 32
// digits, 1.48 for 128 and 1.93 for 512 into buckets, 0.89-0.90 for any
// number of digits as whole steps.  What is left is the streaming of 16
// bytes per key (0.83 ms at the rate of a 1 GiB copy, 5.2 TB/s) and the LDS
// sort beside it (0.6 ms without any stores); counters put the pass at the
// copy's rate.  The price is paid by the reader, in runs of 8192 / digits
// records on average.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bf_hash.hpp"
#include "bf_kernels.hpp"

namespace bfhip {

constexpr int kStep = 8192;         // records per step
constexpr int kGroupThreads = 1024;
constexpr int kGroupPer = kStep / kGroupThreads;  // records per thread and step

// A run of the table: its first record within the step and its length.
__host__ __device__ constexpr uint32_t run_entry(uint32_t start, uint32_t len) { return start | len << 16; }
__device__ __forceinline__ uint32_t run_start(uint32_t e) { return e & 0xffffu; }
__device__ __forceinline__ uint32_t run_len(uint32_t e) { return e >> 16; }

// Workgroups go to the 8 XCDs round-robin by index.  Readers of neighbouring
// digits share the lines where their runs meet (a run is rarely a whole
// number of 128-byte lines), so workgroup b takes the work item that puts 64
// consecutive ones (fewer if there are few) on one XCD, whose L2 then fetches
// such a line once (measured on MI355X: apply of 11.6 M keys into 512 chunks 72.8 -> 68.7 us;
// no difference at 16,384 chunks, whose lines the Infinity Cache serves).
__device__ __forceinline__ uint32_t xcd_item(uint32_t b, uint32_t n) {
  const uint32_t G = n >= 512 ? 64 : n / 8;
  if (G == 0 || b >= n / (8 * G) * (8 * G)) return b;
  const uint32_t x = b & 7u, j = b >> 3;
  return (j / G * 8 + x) * G + j % G;
}

// LDS scratch of a grouping workgroup: up to D digits, table rows written
// out ROWS steps at a time (ROWS * 4 contiguous bytes per digit).
template <int D, int ROWS>
struct GroupLds {
  uint64_t stage[kStep];
  uint32_t cnt[D];
  uint32_t start[D];
  uint32_t rows[D * (ROWS + 1)];  // one column of padding keeps a row's writes off one bank
};

// Sorts one step: record j of this thread (valid_of(j)) has digit dg[j].
// On return rank[j] is its number among the digit's records, so that its
// place in the sorted step is l.start[dg[j]] + rank[j], and l.rows[.. row]
// is set (a run's length there is at most `clip`: readers then see that many
// of its records); the caller writes its records to l.stage, passes a
// barrier and stores the step.  after_rank() runs before the first barrier
// and after_count() behind it: loads issued there are in flight during the
// rest of the step.
// l.cnt is zero on entry and on return.  Two barriers.
template <int D, int ROWS, int PER, typename ValidOf, typename AfterRank, typename AfterCount>
__device__ __forceinline__ void group_positions(GroupLds<D, ROWS>& l, const uint32_t (&dg)[PER], ValidOf valid_of,
                                                uint32_t row, uint32_t clip, uint32_t (&rank)[PER],
                                                AfterRank after_rank, AfterCount after_count) {
  constexpr int kDig = D / 64;
  const uint32_t tid = threadIdx.x;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    rank[j] = 0;
    if (valid_of(j)) rank[j] = atomicAdd(&l.cnt[dg[j]], 1u);
  }
  after_rank();
  __syncthreads();
  after_count();
  if (tid < 64) {  // exclusive scan of the counts by one wave
    uint32_t c[kDig], sum = 0;
#pragma unroll
    for (int i = 0; i < kDig; ++i) {
      c[i] = l.cnt[tid * kDig + i];
      sum += c[i];
    }
#pragma unroll
    for (int i = 0; i < kDig; ++i) l.cnt[tid * kDig + i] = 0;
    uint32_t incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t v = __shfl_up(incl, off, 64);
      if (tid >= static_cast<uint32_t>(off)) incl += v;
    }
    uint32_t run = incl - sum;
#pragma unroll
    for (int i = 0; i < kDig; ++i) {
      l.start[tid * kDig + i] = run;
      l.rows[(tid * kDig + i) * (ROWS + 1) + row] = run_entry(run, c[i] < clip ? c[i] : clip);
      run += c[i];
    }
  }
  __syncthreads();
}

constexpr uint32_t kNoClip = kStep;
constexpr uint32_t kNoPlace = 0xffffu;  // the place of a record beyond its run's clip

// Writes the table rows [0, nrows) of l.rows for digits below ndigits, as
// steps first .. first + nrows - 1 of a table of `stride` steps per digit.
template <int D, int ROWS>
__device__ __forceinline__ void group_flush_rows(const GroupLds<D, ROWS>& l, uint32_t* table, uint64_t stride,
                                                 uint64_t first, uint32_t nrows, uint32_t ndigits) {
  for (uint32_t i = threadIdx.x; i < ndigits * ROWS; i += blockDim.x) {
    const uint32_t d = i / ROWS, r = i % ROWS;
    if (r < nrows) table[d * stride + first + r] = l.rows[d * (ROWS + 1) + r];
  }
}

// Record formats of a stored step (l.stage holds block << 32 | lo32).
// Pairs: the two words as they are.
struct RecordPairs {
  uint64_t* rec;
  template <int THREADS>
  __device__ __forceinline__ void store_step(uint64_t step, const uint64_t* stage, uint32_t) const {
    u32x4* out = reinterpret_cast<u32x4*>(rec + step * kStep);
    const u32x4* in = reinterpret_cast<const u32x4*>(stage);
#pragma unroll
    for (int j = 0; j < kStep / 2 / THREADS; ++j) out[j * THREADS + threadIdx.x] = in[j * THREADS + threadIdx.x];
  }
};
// Split: lo32 in one array, the block within its digit (at most 2^16 blocks)
// in another: 6 bytes.
struct RecordSplit {
  uint32_t* lo;
  uint16_t* blk;
  template <int THREADS>
  __device__ __forceinline__ void store_step(uint64_t step, const uint64_t* stage, uint32_t local_mask) const {
    u32x4* out_lo = reinterpret_cast<u32x4*>(lo + step * kStep);
    u32x2* out_blk = reinterpret_cast<u32x2*>(blk + step * kStep);
    const u32x4* in = reinterpret_cast<const u32x4*>(stage);
#pragma unroll
    for (int j = 0; j < kStep / 4 / THREADS; ++j) {
      const uint32_t i = j * THREADS + threadIdx.x;
      const u32x4 a = in[2 * i], b = in[2 * i + 1];
      out_lo[i] = u32x4{a[0], a[2], b[0], b[2]};
      out_blk[i] = u32x2{(a[1] & local_mask) | (a[3] & local_mask) << 16, (b[1] & local_mask) | (b[3] & local_mask) << 16};
    }
  }
};

// A unit of a run, packed: its first slot relative to the batch of at most
// 1,024 steps it was listed in (23 bits) and its length less one (4 bits).
__device__ __forceinline__ uint32_t unit_entry(uint32_t slot, uint32_t len) { return slot << 4 | (len - 1); }

// LDS scratch of a reader, with a list of LIST unit entries.
template <int THREADS, int LIST>
struct RunLds {
  uint32_t run[THREADS];
  uint32_t pre[THREADS];  // units before each run of the batch
  uint32_t list[LIST];
  uint32_t wave_sum[THREADS / 64];
};

// The unit u of a batch of RUNS runs whose unit prefix sums are pre[]: in
// the last run r with pre[r] <= u.
template <int UNIT, int RUNS>
__device__ __forceinline__ uint32_t find_unit(const uint32_t* pre, const uint32_t* run, uint32_t u) {
  uint32_t r = 0;
#pragma unroll
  for (uint32_t b = RUNS / 2; b != 0; b >>= 1)
    if (pre[r + b] <= u) r += b;
  const uint32_t e = run[r], o = (u - pre[r]) * UNIT, left = run_len(e) - o;
  return unit_entry(r * kStep + run_start(e) + o, left < UNIT ? left : UNIT);
}

// A split record as a reader loads it.
struct SplitRecord {
  uint32_t lo;
  uint32_t blk;
};

// Visits the split records (lo[], blk[]) of `n` consecutive table entries,
// those of steps first_step, first_step + 1, ...: use(slot, ok, record) for
// UNROLL slots per lane and call; a lane without a record has ok false, its
// slot is one that may be read.  All threads of the workgroup call this.
// prepare() is called once, with a barrier between it and the first use,
// unless there are no records at all: then nothing is called.  Returns
// whether there were records (uniform).
// THREADS entries are taken at a time and their runs cut into units of UNIT
// slots, listed in LDS (as many at once as the list holds); UNIT adjacent
// lanes take a unit.  The records of a call are loaded before those of the
// call before it are used.
template <int UNIT, int UNROLL, int THREADS, int LIST, typename Prepare, typename Use>
__device__ __forceinline__ bool for_each_record(RunLds<THREADS, LIST>& l, const uint32_t* lo, const uint16_t* blk,
                                                const uint32_t* entries, uint64_t first_step, uint32_t n,
                                                Prepare prepare, Use use) {
  static_assert(UNIT <= 16 && (UNIT & (UNIT - 1)) == 0 && THREADS <= 1024, "the fields of a unit entry");
  constexpr uint32_t kList = LIST, kGroups = THREADS / UNIT;
  constexpr uint32_t kLong = 8;  // units of a run that its thread lists by itself
  constexpr uint32_t kLongBit = 1u << 31;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t g = tid / UNIT, in = tid % UNIT;
  uint32_t e_next = tid < n ? entries[tid] : 0u;
  bool any = false;
  for (uint32_t base = 0; base < n; base += THREADS) {
    const uint32_t e = e_next;
    e_next = base + THREADS + tid < n ? entries[base + THREADS + tid] : 0u;
    const uint32_t len = run_len(e), units = (len + UNIT - 1) / UNIT;
    uint32_t incl = units;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t v = __shfl_up(incl, off, 64);
      if (lane >= static_cast<uint32_t>(off)) incl += v;
    }
    const bool wave_long = __any(units > kLong);
    if (lane == 63) l.wave_sum[wave] = incl | (wave_long ? kLongBit : 0u);
    __syncthreads();
    uint32_t at = incl - units, total = 0, long_runs = 0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) {
      const uint32_t s = l.wave_sum[w];
      long_runs |= s & kLongBit;
      if (static_cast<uint32_t>(w) < wave) at += s & ~kLongBit;
      total += s & ~kLongBit;
    }
    if (long_runs) {
      l.run[tid] = e;
      l.pre[tid] = at;
    }
    if (total != 0 && !any) {
      any = true;
      prepare();
    }
    const uint32_t slot = tid * kStep + run_start(e);
    const uint64_t slot0 = (first_step + base) * kStep;
    for (uint32_t w0 = 0; w0 < total; w0 += kList) {
      const uint32_t m = total - w0 < kList ? total - w0 : kList;
      if (long_runs) {  // every unit of the window looked up
        __syncthreads();
        for (uint32_t u = tid; u < m; u += THREADS) l.list[u] = find_unit<UNIT, THREADS>(l.pre, l.run, w0 + u);
      } else {  // this thread's units [at, at + units) that fall in the window
        const uint32_t u0 = at > w0 ? at : w0, u1 = at + units < w0 + kList ? at + units : w0 + kList;
        for (uint32_t u = u0; u < u1; ++u) {
          const uint32_t o = (u - at) * UNIT;
          l.list[u - w0] = unit_entry(slot + o, len - o < UNIT ? len - o : UNIT);
        }
      }
      __syncthreads();
      const uint32_t* lo0 = lo + slot0;
      const uint16_t* blk0 = blk + slot0;
      uint32_t i[UNROLL];
      SplitRecord r[UNROLL];
      uint32_t ok = 0;
      auto fetch = [&](uint32_t u) {
        ok = 0;
#pragma unroll
        for (int q = 0; q < UNROLL; ++q) {
          const uint32_t at_u = u + q * kGroups + g;
          const uint32_t v = l.list[at_u < m ? at_u : 0];
          const bool has = at_u < m && in <= (v & 15u);
          i[q] = (v >> 4) + (has ? in : 0u);
          ok |= static_cast<uint32_t>(has) << q;
        }
#pragma unroll
        for (int q = 0; q < UNROLL; ++q) r[q] = SplitRecord{lo0[i[q]], blk0[i[q]]};
      };
      fetch(0);
      for (uint32_t u = 0; u < m; u += kGroups * UNROLL) {
        SplitRecord cur[UNROLL];
        uint32_t ci[UNROLL];
        const uint32_t cok = ok;
#pragma unroll
        for (int q = 0; q < UNROLL; ++q) {
          cur[q] = r[q];
          ci[q] = i[q];
        }
        if (u + kGroups * UNROLL < m) fetch(u + kGroups * UNROLL);
#pragma unroll
        for (int q = 0; q < UNROLL; ++q) use(slot0 + ci[q], (cok >> q & 1u) != 0, cur[q]);
      }
      __syncthreads();
    }
    if (total == 0) __syncthreads();  // wave_sum is rewritten next
  }
  return any;
}

// ---------------------------------------------------------------------------
// First pass: hash the keys and group their records by digit.
// ---------------------------------------------------------------------------

// One filter of a multi-filter partitioned add.  Its blocks occupy global
// blocks [block_base, block_base + num_blocks) and its chunks global chunks
// from chunk_base (block_base is a multiple of the blocks per chunk); its
// keys are keys[key_begin, key_end).  A `direct` filter (few keys for its
// size) takes no part: its keys are left to a direct launch, so none of its
// chunks is read or written here.
struct PartFilter {
  void* words;
  uint64_t hash_init;
  uint32_t nb_lo;
  uint32_t nb_hi_mask;
  uint64_t num_blocks;
  uint64_t block_base;
  uint64_t chunk_base;
  uint64_t key_begin;
  uint64_t key_end;
  uint32_t direct;
  uint32_t reserved;
};

// The keys [begin, end) of filter `filter`: one first-pass workgroup of a
// multi-filter plan, whose steps are first_step and on.
struct PartRange {
  uint64_t begin;
  uint64_t end;
  uint32_t filter;
  uint32_t first_step;
};

struct GroupArgs {
  const uint64_t* keys;
  uint64_t n;
  uint64_t hash_init;
  uint32_t nb_lo;
  uint32_t nb_hi_mask;
  uint32_t shift;       // digit = block >> shift
  uint32_t local_mask;  // block within its digit (split records)
  uint32_t digits;
  uint32_t steps;
  uint32_t wg_steps;    // steps per workgroup (one filter)
  uint64_t stride;      // table entries per digit (>= steps)
  uint32_t* table;
  uint64_t* rec;        // records of steps * kStep slots: pairs ...
  uint32_t* lo;         // ... or split
  uint16_t* blk;
  uint16_t* place;      // lookups: each key's place in its sorted step (kNoPlace: beyond clip)
  uint32_t clip;        // lookups: records of a run that readers see
  const uint32_t* direct;  // lookups: nonzero if the keys are looked up directly and nothing is grouped
  const PartRange* ranges;    // multi-filter plans
  const PartFilter* filters;
  uint64_t num_bits;    // classic filter
  uint32_t bit_shift;
};

// MULTI: the workgroup's keys are one range of one filter of a plan, whose
// fields are read once before the key loop.  SPLIT: 6-byte records.  PLACE:
// a.place is written (lookups).
template <int D, int ROWS, bool SPLIT, bool MULTI, bool PLACE>
__global__ __launch_bounds__(kGroupThreads) void group_keys_kernel(GroupArgs a) {
  __shared__ __attribute__((aligned(16))) GroupLds<D, ROWS> l;
  if constexpr (PLACE)
    if (*a.direct != 0) return;
  const uint32_t tid = threadIdx.x;
  for (uint32_t d = tid; d < D; d += kGroupThreads) l.cnt[d] = 0;
  uint64_t begin, end, hinit = a.hash_init;
  uint32_t t0, nb_lo = a.nb_lo, nb_hi = a.nb_hi_mask, block0 = 0;
  if constexpr (MULTI) {
    const PartRange r = a.ranges[blockIdx.x];
    const PartFilter& f = a.filters[r.filter];
    begin = r.begin;
    end = r.end;
    t0 = r.first_step;
    hinit = f.hash_init;
    nb_lo = f.nb_lo;
    nb_hi = f.nb_hi_mask;
    block0 = static_cast<uint32_t>(f.block_base);
  } else {
    t0 = blockIdx.x * a.wg_steps;
    begin = static_cast<uint64_t>(t0) * kStep;
    const uint64_t most = begin + static_cast<uint64_t>(a.wg_steps) * kStep;
    end = most < a.n ? most : a.n;
  }
  const uint32_t t1 = t0 + static_cast<uint32_t>((end - begin + kStep - 1) / kStep);
  uint64_t next[kGroupPer];
  auto load = [&](uint64_t s) {
    const uint32_t valid = static_cast<uint32_t>(end - s < kStep ? end - s : kStep);
    const char* base = reinterpret_cast<const char*>(a.keys + s);
#pragma unroll
    for (int j = 0; j < kGroupPer; ++j) {
      const uint32_t p = tid + j * kGroupThreads;
      next[j] = __builtin_nontemporal_load(reinterpret_cast<const uint64_t*>(base + 8u * (p < valid ? p : 0u)));
    }
  };
  load(begin);
  // the first keys are waited for here, so that at the top of every step the
  // outstanding operations are those of the step before
  __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));
  __syncthreads();
  uint64_t s = begin;
  for (uint32_t t = t0; t < t1; ++t, s += kStep) {
    const uint32_t valid = static_cast<uint32_t>(end - s < kStep ? end - s : kStep);
    uint32_t blk[kGroupPer], lo[kGroupPer], dg[kGroupPer], rank[kGroupPer];
#pragma unroll
    for (int j = 0; j < kGroupPer; ++j) {
      const uint64_t h = xxh64_u64(next[j], hinit);
      blk[j] = block0 + block_of(h, nb_lo, nb_hi);
      lo[j] = static_cast<uint32_t>(h);
      dg[j] = blk[j] >> a.shift;
    }
    const uint32_t row = (t - t0) % ROWS;
    auto in = [&](int j) { return tid + j * kGroupThreads < valid; };
    group_positions(l, dg, in, row, PLACE ? a.clip : kNoClip, rank, [&] { if (t + 1 < t1) load(s + kStep); }, [] {});
#pragma unroll
    for (int j = 0; j < kGroupPer; ++j) {
      const uint32_t pos = l.start[dg[j]] + rank[j];
      if (in(j)) l.stage[pos] = static_cast<uint64_t>(blk[j]) << 32 | lo[j];
      // a whole step of places may be written: the array has kStep per step
      if constexpr (PLACE)
        a.place[static_cast<uint64_t>(t) * kStep + tid + j * kGroupThreads] =
            static_cast<uint16_t>(rank[j] < a.clip ? pos : kNoPlace);
    }
    __syncthreads();
    if constexpr (SPLIT)
      RecordSplit{a.lo, a.blk}.template store_step<kGroupThreads>(t, l.stage, a.local_mask);
    else
      RecordPairs{a.rec}.template store_step<kGroupThreads>(t, l.stage, 0);
    if (row == ROWS - 1 || t + 1 == t1) group_flush_rows(l, a.table, a.stride, t - row, row + 1, a.digits);
  }
}

// ---------------------------------------------------------------------------
// Second pass: group the records of one first-pass digit by the next digit.
// ---------------------------------------------------------------------------
constexpr int kUnit = 16;                      // slots per unit of the second pass ...
constexpr int kShortUnit = 8;                  // ... where the first pass's runs are short
constexpr int kStepUnits = kStep / kUnit;      // units per step of a lookup
constexpr int kRegroupRuns = 1024;             // runs per batch

// One workgroup's work: the runs of digit d1 in steps [t0, t1).
struct PartItem {
  uint32_t d1, t0, t1, reserved;
};

struct RegroupArgs {
  const uint64_t* rec;     // the first pass's pairs and table
  const uint32_t* table1;
  uint64_t stride1;
  uint32_t steps1;
  uint32_t items;
  uint32_t per_digit;      // items per first digit (one filter) ...
  uint32_t item_steps;     // ... and first-pass steps per item
  const PartItem* list;    // or the items of a multi-filter plan, by digit
  uint32_t* item_count;    // per item: its steps
  uint32_t* slot0;         // items + 1: first step of each item's output
  uint32_t shift;          // second digit = (block >> shift) & (digits - 1)
  uint32_t digits;
  uint32_t* lo;            // output: split records and table
  uint16_t* blk;
  uint32_t* table2;
  uint64_t stride2;
  uint16_t* place;         // lookups: place of each slot's record in the sorted step (kNoPlace: beyond clip)
  uint32_t clip, clip_last;  // (its last first digit may have fewer second digits, so longer runs)
  uint32_t* units;         // lookups: the units a step was read from
  const uint32_t* direct;  // lookups: as in GroupArgs (nullptr for adds)
};

// The items of one step range and neighbouring digits are neighbours here.
__device__ __forceinline__ uint32_t regroup_item_of(const RegroupArgs& a, uint32_t b) {
  if (a.list != nullptr) return b;
  const uint32_t digits1 = a.items / a.per_digit;
  const uint32_t i = xcd_item(b, a.items);
  return i % digits1 * a.per_digit + i / digits1;
}

__device__ __forceinline__ PartItem regroup_item(const RegroupArgs& a, uint32_t item) {
  if (a.list != nullptr) return a.list[item];
  const uint32_t d1 = item / a.per_digit, g = item % a.per_digit;
  const uint32_t t0 = g * a.item_steps, t1 = t0 + a.item_steps;
  return PartItem{d1, t0 < a.steps1 ? t0 : a.steps1, t1 < a.steps1 ? t1 : a.steps1, 0};
}

constexpr int kPlanThreads = 256;   // counting every item's output steps
constexpr int kScanThreads = 1024;  // ... and their prefix sums (one workgroup)

template <int D, int ROWS, int UNIT>
struct RegroupLds {
  GroupLds<D, ROWS> g;
  uint32_t run[kRegroupRuns];
  uint32_t pre[kRegroupRuns];          // units before each run of the batch
  uint32_t list[2][kStep / UNIT];      // the step's units, of even and odd steps
  uint32_t wave_sum[kGroupThreads / 64];
};

template <int D, int ROWS, bool PLACE, int UNIT>
__global__ __launch_bounds__(kGroupThreads) void regroup_kernel(RegroupArgs a) {
  static_assert(kRegroupRuns == kGroupThreads, "a thread per run of a batch");
  static_assert(!PLACE || UNIT == kUnit, "the return of a lookup's results reads units of kUnit slots");
  constexpr int kUnits = kStep / UNIT;
  __shared__ __attribute__((aligned(16))) RegroupLds<D, ROWS, UNIT> l;
  if constexpr (PLACE)
    if (*a.direct != 0) return;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  for (uint32_t d = tid; d < D; d += kGroupThreads) l.g.cnt[d] = 0;
  const uint32_t item = regroup_item_of(a, blockIdx.x);
  const PartItem it = regroup_item(a, item);
  const uint32_t first = a.slot0[item];
  uint32_t row = 0;  // steps written
  uint32_t clip = kNoClip;
  if constexpr (PLACE) clip = it.d1 + 1 == a.items / a.per_digit ? a.clip_last : a.clip;
  const uint32_t mask = a.digits - 1, local_mask = (1u << a.shift) - 1;
  const uint32_t* entries = a.table1 + it.d1 * a.stride1;
  for (uint32_t base = it.t0; base < it.t1; base += kRegroupRuns) {
    const uint32_t e = base + tid < it.t1 ? entries[base + tid] : 0u;
    const uint32_t units = (run_len(e) + UNIT - 1) / UNIT;
    uint32_t incl = units;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t v = __shfl_up(incl, off, 64);
      if (lane >= static_cast<uint32_t>(off)) incl += v;
    }
    if (lane == 63) l.wave_sum[wave] = incl;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kGroupThreads / 64; ++w) {
      const uint32_t s = l.wave_sum[w];
      if (static_cast<uint32_t>(w) < wave) before += s;
      total += s;
    }
    l.run[tid] = e;
    l.pre[tid] = before + incl - units;
    __syncthreads();
    if (total == 0) continue;
    // unit u of the batch is in the last run r with pre[r] <= u
    auto find = [&](uint32_t w) {
      if (tid < kUnits) {
        const uint32_t u = w * kUnits + tid;
        uint32_t v = 0xffffffffu;
        if (u < total) v = find_unit<UNIT, kRegroupRuns>(l.pre, l.run, u);
        l.list[w & 1u][tid] = v;
      }
    };
    uint64_t next[kGroupPer];
    uint32_t next_ok = 0;
    const uint64_t* src = a.rec + static_cast<uint64_t>(base) * kStep;
    auto load = [&](uint32_t w) {
      next_ok = 0;
#pragma unroll
      for (int j = 0; j < kGroupPer; ++j) {
        const uint32_t v = l.list[w & 1u][(tid + j * kGroupThreads) / UNIT];
        const bool ok = v != 0xffffffffu && tid % UNIT <= (v & 15u);
        next[j] = src[ok ? (v >> 4) + tid % UNIT : 0u];
        next_ok |= static_cast<uint32_t>(ok) << j;
      }
    };
    const uint32_t windows = (total + kUnits - 1) / kUnits;
    find(0);
    __syncthreads();
    load(0);
    for (uint32_t w = 0; w < windows; ++w, ++row) {
      uint64_t r[kGroupPer];
      uint32_t dg[kGroupPer], rank[kGroupPer];
      const uint32_t ok = next_ok;
#pragma unroll
      for (int j = 0; j < kGroupPer; ++j) {
        r[j] = next[j];
        dg[j] = static_cast<uint32_t>(r[j] >> 32) >> a.shift & mask;
      }
      auto in = [&](int j) { return (ok >> j & 1u) != 0; };
      group_positions(l.g, dg, in, row % ROWS, clip, rank, [&] { if (w + 1 < windows) find(w + 1); },
                      [&] { if (w + 1 < windows) load(w + 1); });
      const uint64_t step = first + row;
#pragma unroll
      for (int j = 0; j < kGroupPer; ++j) {
        const uint32_t pos = l.g.start[dg[j]] + rank[j];
        if (in(j)) l.g.stage[pos] = r[j];
        if constexpr (PLACE)
          a.place[step * kStep + tid + j * kGroupThreads] = static_cast<uint16_t>(rank[j] < clip ? pos : kNoPlace);
      }
      if constexpr (PLACE) {
        if (tid < kUnits) {
          const uint32_t v = l.list[w & 1u][tid];
          a.units[step * kUnits + tid] = v == 0xffffffffu ? v : v + (base * kStep << 4);
        }
      }
      __syncthreads();
      RecordSplit{a.lo, a.blk}.template store_step<kGroupThreads>(step, l.g.stage, local_mask);
      if (row % ROWS == ROWS - 1) group_flush_rows(l.g, a.table2, a.stride2, step - (ROWS - 1), ROWS, a.digits);
    }
    __syncthreads();  // the next batch replaces run and pre
  }
  if (row % ROWS != 0) group_flush_rows(l.g, a.table2, a.stride2, first + row - row % ROWS, row % ROWS, a.digits);
}

// The grouping kernels (bf_group.hip) for a number of digits: the first pass
// (nullptr for an unsupported number), the second pass and its
// two planning kernels.
const void* group_keys_fn(uint32_t digits, bool split, bool multi, bool place);
const void* regroup_fn(uint32_t digits, bool place, bool short_units);
const void* regroup_plan_fn(bool short_units);
const void* regroup_scan_fn();

}  // namespace bfhip
