// bf_batch.hip -- batched plans (C ABI in include/bf_batch.h): tile list
// construction, XCD-aware ordering, HIP graph of one persistent launch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <functional>
#include <new>
#include <mutex>
#include <numeric>
#include <utility>
#include <vector>

#include "../../include/bf_batch.h"
#include "bf_batch_kernels.hpp"
#include "bf_resident.hpp"
#include "bf_internal.hpp"
#include "bf_partition.hpp"
#include "bf_registry.hpp"
#include "bf_tuned.hpp"

using namespace bfhip;

namespace {

constexpr int kXcds = 8;          // MI355X: 8 XCDs, workgroups dispatched round-robin
constexpr int kWgPerCu = 8;       // persistent grid: 8 workgroups (32 waves) per CU

}  // namespace

struct bf_batch {
  int op;
  uint32_t nfilters;
  uint64_t nkeys;
  std::vector<bf_filter*> filters;
  std::vector<uint64_t> offsets;
  const uint64_t* d_keys;
  uint8_t* d_out;
  BatchFilter* d_filters;
  BatchTile* d_tiles;
  uint64_t ntiles;      // slots of the persistent launch
  // lookups in the filters that fit the LDS, one launch per variant: their
  // items lie behind the slots
  struct Resident {
    const void* fn;
    uint64_t nitems;
    ResidentArgs args;
  } resident[2];
  uint32_t grid;
  uint32_t tiles_per_class[kNumSizeClasses];
  bf_mapping_t mapping[kNumSizeClasses];
  const void* fn;
  BatchArgs args;
  hipGraph_t graph;
  hipGraphExec_t exec;
  // partitioned construction over the dense filters of the plan (add only);
  // part_direct[i] marks the filters left to the tiled direct launch
  bool partitioned;
  std::vector<uint8_t> part_direct;
  PartArgs part;
  PartKernels part_k;
  void* part_scratch;
  // device memory from lib_alloc (pooled: released in stream order)
  int device;
  bool pooled_filters, pooled_tiles, pooled_scratch;
  // one event per stream the plan was launched on, recorded after its last
  // launch there: bf_batch_destroy waits for these and nothing else
  std::mutex mark_mu;
  std::vector<std::pair<hipStream_t, hipEvent_t>> marks;
  bool unmarked;  // a launch whose event could not be recorded: destroy waits for the device
};

namespace {

// The mapping the batched kernel compiles in for a size class (bf_batch_kernels.hpp:
// batch_map): the tuned rows of large batches at the filters' k.
MapSpec class_map(int op, const bf_filter* f, int cls) {
  if (k_index(f->k) == 0) return MapSpec{1, f->s, 1, 32, 0, kBlockThreads, true};
  return tuned_map(op, static_cast<int>(f->word_bits), static_cast<int>(f->s), cls,
                   static_cast<int>(f->k), 1);
}

uint64_t items_of(const bf_batch* b) { return b->resident[0].nitems + b->resident[1].nitems; }

void free_plan(bf_batch* b) {
  if (b->exec) (void)hipGraphExecDestroy(b->exec);
  if (b->graph) (void)hipGraphDestroy(b->graph);
  lib_free(b->device, b->d_filters, b->pooled_filters);
  lib_free(b->device, b->d_tiles, b->pooled_tiles);
  lib_free(b->device, b->part_scratch, b->pooled_scratch);
  for (auto& m : b->marks) (void)hipEventDestroy(m.second);
  delete b;
}

// The mark of a launch of the plan on `stream`: the stream's event (none for
// a stream being captured: such a launch runs when the caller's graph does,
// which the caller orders against the plan's destruction).  mark_mu is held.
CallMark begin_launch(bf_batch* b, hipStream_t stream) {
  CallMark mark;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &cap) == hipSuccess && cap != hipStreamCaptureStatusNone) return mark;
  for (auto& m : b->marks)
    if (m.first == stream) mark.event = m.second;
  if (mark.event == nullptr) {
    if (hipEventCreateWithFlags(&mark.event, hipEventDisableTiming) == hipSuccess) {
      b->marks.emplace_back(stream, mark.event);
    } else {
      (void)hipGetLastError();
      mark.event = nullptr;
      mark.lost = true;
      b->unmarked = true;  // destroy waits for the device
    }
  }
  return mark;
}

// Records the mark where no kernel of the launch signals it.
bf_status end_launch(bf_batch* b, hipStream_t stream, const CallMark& mark) {
  if (mark.signalled) return BF_OK;
  if (mark.event == nullptr) return mark.lost ? BF_EDEVICE : BF_OK;
  if (hipEventRecord(mark.event, stream) != hipSuccess) {
    (void)hipGetLastError();
    b->unmarked = true;  // the work is enqueued: destroy must still wait for it
    return BF_EDEVICE;
  }
  return BF_OK;
}

// Whether a filter of the plan with n keys runs in LDS (bf_resident.hpp).
// It is copied or merged once per item; below one key per 32 bytes that would
// move more than the keys' blocks.  Lookups, with 131,072 keys per filter of
// 32-byte blocks, in G keys/s: 4 KiB 250 from the caches, 370 from LDS;
// 64 KiB 135, 371; 128 KiB (one workgroup per CU) 120, 278.
bool resides(const bf_batch* b, const bf_filter* f, uint64_t n) {
  const int big = f->nbytes > kResidentBytes[0];
  return b->resident[big].fn != nullptr && f->nbytes <= kResidentBytes[big] &&
         n * (b->op == BF_OP_ADD ? 8 : 32) >= f->nbytes;
}

uint64_t resident_keys_of(const bf_batch* b, bf_filter* const* filters, uint32_t nfilters, const uint64_t* h_offsets) {
  uint64_t keys = 0;
  for (uint32_t i = 0; i < nfilters; ++i) {
    const uint64_t n = h_offsets[i + 1] - h_offsets[i];
    if (resides(b, filters[i], n)) keys += n;
  }
  return keys;
}

// Whether the plan is faster with its small filters in LDS.  A lookup plan's
// tiles of one filter stay on one XCD, so its time is that of the fullest XCD:
// 12 keys per ns in filters beyond 160 KiB, in smaller ones 18, 15 with blocks
// of 32 bytes and more, 9 with a k that is not compiled in (k = 16: 9.6 and 15.8).  The launches in
// LDS cost 17 us and test 240 keys per ns over all CUs with k = 8, fewer with
// more bits per key.  So plans whose largest filter does not fit the LDS and
// bounds them gain nothing, nor do plans of few keys.  Measured, us from the
// caches / in LDS: 1,024 filters of 32 KiB and 8,192 keys 71 / 44 (4 x 64 bits,
// k = 16: 63 / 51; k = 9: 101 / 70), 300 of 16 KiB and 30,000 keys 67 / 52,
// 512 of 128 KiB and 8,192 keys 47 / 46 (1 x 32 bits: 40 / 44; 4 x 64: 42 / 50),
// 64 of Zipf counts, 2^24 keys 288 / 212 (4 x 64: 251 / 270), 1,024 of Zipf counts, 2^22 keys 57 / 58 (1 x 32: 49 / 55), 2^23 109 / 97.
// Add plans gain from 1.5 M such keys on (1,024 filters of Zipf counts: 2^21
// keys 133 us without, 141 with; 2^22 keys 296, 202).
bool resides_pays(const bf_batch* b, bf_filter* const* filters, uint32_t nfilters, const uint64_t* h_offsets) {
  const uint64_t keys = resident_keys_of(b, filters, nfilters, h_offsets);
  if (b->op == BF_OP_ADD) return keys >= 3u << 19;
  if (keys == 0) return false;
  const bf_filter* f0 = filters[0];
  const bool generic = k_index(f0->k) == 0;
  const double small = generic ? 9.0 : f0->k >= 16 ? 15.8 : f0->s * f0->word_bits >= 256 ? 15.0 : 18.0;
  const double large = generic ? 9.0 : f0->k >= 16 ? 9.6 : 12.0;
  const double lds = 240.0 / (generic ? 2.3 : 0.75 + f0->k / 32.0);
  std::vector<std::pair<double, bool>> costs(nfilters);  // ns on one XCD, and whether in LDS
  for (uint32_t i = 0; i < nfilters; ++i) {
    const uint64_t n = h_offsets[i + 1] - h_offsets[i];
    const bool in_lds = resides(b, filters[i], n);
    costs[i] = {static_cast<double>(n) / (in_lds ? small : large), in_lds};
  }
  std::sort(costs.begin(), costs.end(), [](const auto& x, const auto& y) { return x.first > y.first; });
  double all[kXcds] = {}, rest[kXcds] = {};
  for (const auto& [ns, in_lds] : costs) {
    *std::min_element(all, all + kXcds) += ns;
    if (!in_lds) *std::min_element(rest, rest + kXcds) += ns;
  }
  const double caches = *std::max_element(all, all + kXcds);
  return *std::max_element(rest, rest + kXcds) + static_cast<double>(keys) / lds + 20000.0 < caches;
}

// A chunk of a partitioned construction is read, updated in LDS and written
// back by the workgroups of its plan entry, so no two entries may own the
// same words: where entries' words overlap (a filter named twice, two views
// of one buffer) one of them stays and the others' keys are left to the
// direct launch, which runs behind the construction and merges by atomic OR.
void leave_overlaps_direct(bf_filter* const* filters, std::vector<PartFilter>& pf) {
  std::vector<uint32_t> order;
  for (uint32_t i = 0; i < pf.size(); ++i)
    if (!pf[i].direct && pf[i].key_end > pf[i].key_begin) order.push_back(i);
  auto begin = [&](uint32_t i) { return reinterpret_cast<uintptr_t>(pf[i].words); };
  std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) { return begin(x) < begin(y); });
  uintptr_t end = 0;  // of the words that are owned
  for (uint32_t i : order) {
    if (begin(i) < end)
      pf[i].direct = 1;
    else
      end = begin(i) + filters[i]->nbytes;
  }
}

// ps per key of a plan's adds into f in tiles; the rows are measured with a k
// that is compiled in (1,024 filters of Zipf counts, 2^21 keys: k = 8 140 us,
// k = 9 787).
double tile_add_ps(const CrossoverRow* r, const bf_filter* f) {
  return (r != nullptr ? r->d_ps[size_class_of(f->nbytes)] : 37.0) * (k_index(f->k) == 0 ? 5.6 : 1.0);
}

// Whether a dense filter's n keys are worth a step of a plan's construction.
// A step holds one filter's keys and is stored whole, 42 ns over all CUs and
// 64 KiB of workspace however few they are, where the direct launch takes
// d - c ps more per key (the layout's measured costs).  Plans of 20,000 filters,
// us and MB of the plan, partitioned against direct: 4 KiB and 110 keys each 851
// and 1,344 against 97 and 2, 32 KiB and 600 keys 1,072 and 1,434 against 546
// and 2, 1,500 keys 1,176 and 1,550 against 1,137 and 2.
bool fills_step(const CrossoverRow* r, const bf_filter* f, uint64_t n) {
  const double gain = tile_add_ps(r, f) - (r != nullptr ? r->c_ps : 10.8);
  return n >= static_cast<uint64_t>(kStep) || static_cast<double>(n) * gain > 42000.0;
}

// The costs of a plan's dense filters, in us: those that fit the LDS there and
// the others (not `direct`) in tiles, whose atomics the device takes at d ps
// per key and one XCD, which has all tiles of a filter, at 76; or all of them
// in one construction.  Measured, us: 2,048 filters of 64 KiB with 2^24 keys and
// one of 16 MiB with 2^22 430 against 364 together, 512 of 128 KiB with 2^23 and
// four of 4 MiB with 2^22 274 against 194; apart 186 with one of 1 MiB and 2^20,
// and with 100 of 256 KiB and 2 M (together about 200).
double lds_and_tiles_us(const CrossoverRow* r, bf_filter* const* filters, const std::vector<PartFilter>& pf,
                        uint64_t in_lds) {
  std::vector<uint64_t> counts;
  double device = 0.0;
  for (size_t i = 0; i < pf.size(); ++i) {
    if (pf[i].direct) continue;
    counts.push_back(pf[i].key_end - pf[i].key_begin);
    device += static_cast<double>(counts.back()) * tile_add_ps(r, filters[i]);
  }
  std::sort(counts.begin(), counts.end(), std::greater<uint64_t>());
  uint64_t load[kXcds] = {};
  for (uint64_t c : counts) *std::min_element(load, load + kXcds) += c;
  const double xcd = static_cast<double>(*std::max_element(load, load + kXcds)) * 76.0;
  return 25.0 + 5e-6 * static_cast<double>(in_lds) + std::max(device, xcd) * 1e-6;
}

double construction_us(const CrossoverRow* r, uint64_t n, uint64_t chunks) {
  const double mib = static_cast<double>(chunks) / 16.0;
  return r != nullptr ? r->a_us + r->b_us_per_mib * mib + r->c_ps * 1e-6 * static_cast<double>(n)
                      : 40.0 + 0.43 * mib + 10.8e-6 * static_cast<double>(n);
}

// Partitioned construction for an add plan: the filters' blocks are laid
// end to end in one global block space (each filter starting on a chunk
// boundary), so one radix partition groups every key of every filter by
// global chunk.  With the automatic strategy a filter whose keys are too
// few for its size is left to the direct launch (b->part_direct): by the
// layout's measured costs (the crossover rows of bf_tuned.hpp, without the
// fixed cost, which the plan shares), streaming its chunks would cost more
// than its keys' atomics, and its chunks then get neither records nor
// traffic.  Returns BF_OK and sets b->partitioned when taken, and takes the
// small filters out of the LDS launches where they join it.
bf_status plan_partitioned(bf_batch* b, bf_filter* const* filters, uint32_t nfilters,
                           const uint64_t* d_keys, const uint64_t* h_offsets) {
  const bf_filter* f0 = filters[0];
  const uint32_t strategy = f0->mapping[BF_OP_ADD].strategy;
  if (strategy == BF_STRATEGY_DIRECT) return BF_OK;
  const bool forced = strategy == BF_STRATEGY_PARTITIONED;
  const uint32_t shift = part_chunk_shift(f0->s, f0->word_bits);
  const uint64_t bpc = 1ull << shift;
  std::vector<PartFilter> pf(nfilters);
  const CrossoverRow* xr = crossover_of(f0);
  uint64_t chunks = 0;
  for (uint32_t i = 0; i < nfilters; ++i) {
    const bf_filter* f = filters[i];
    pf[i].words = f->d_words;
    pf[i].hash_init = xxh64_u64_init(f->seed);
    pf[i].nb_lo = static_cast<uint32_t>(f->num_blocks);
    pf[i].nb_hi_mask = (f->num_blocks >> 32) ? 0xffffffffu : 0u;
    pf[i].num_blocks = f->num_blocks;
    pf[i].chunk_base = chunks;
    pf[i].block_base = chunks * bpc;
    pf[i].key_begin = h_offsets[i] - h_offsets[0];
    pf[i].key_end = h_offsets[i + 1] - h_offsets[0];
    chunks += (f->num_blocks + bpc - 1) / bpc;
  }
  const uint64_t n = h_offsets[nfilters] - h_offsets[0];
  if (n == 0 || chunks * bpc > (1ull << 32)) return BF_OK;  // global blocks must fit 32 bits
  uint64_t n_dense = 0, dense_chunks = 0;
  auto choose = [&] {  // the filters that take part
    n_dense = dense_chunks = 0;
    for (uint32_t i = 0; i < nfilters; ++i) {
      const bf_filter* f = filters[i];
      const uint64_t ni = pf[i].key_end - pf[i].key_begin;
      const bool left = !dense_enough(xr, f->nbytes, ni, true) || !fills_step(xr, f, ni) || resides(b, f, ni);
      pf[i].direct = !forced && left ? 1u : 0u;
    }
    leave_overlaps_direct(filters, pf);
    for (uint32_t i = 0; i < nfilters; ++i) {
      if (pf[i].direct) continue;
      n_dense += pf[i].key_end - pf[i].key_begin;
      dense_chunks += (pf[i].num_blocks + bpc - 1) / bpc;
    }
    return forced || (dense_chunks >= 512 && n_dense >= (1ull << 21));
  };
  if (!choose()) {
    // Too little for a construction is left beside the filters in LDS: it
    // would go to tiles.  Together they may be enough, and cheaper.
    const uint64_t in_lds = resident_keys_of(b, filters, nfilters, h_offsets);
    if (in_lds == 0) return BF_OK;
    const double apart = lds_and_tiles_us(xr, filters, pf, in_lds);
    b->resident[0].fn = b->resident[1].fn = nullptr;
    if (!choose() || construction_us(xr, n_dense, dense_chunks) >= apart) return BF_OK;
  }
  PartArgs a{};
  PartLayout L{};
  if (!part_digits(chunks, shift, kMaxDigits2, a)) return BF_OK;
  const uint64_t f2 = a.r.digits, f1 = a.g.digits;
  // First-pass ranges: at most range1 keys of one dense filter each (the
  // keys of direct filters are not read), whose steps are numbered in filter
  // order; filter i's are first_step[i] .. first_step[i + 1].
  const uint64_t range1 = std::max<uint64_t>((n / 1024 + kStep) / kStep, 1) * kStep;
  std::vector<PartRange> ranges;
  std::vector<uint64_t> first_step(nfilters + 1, 0);
  uint64_t steps = 0, runs = 0;
  for (uint32_t i = 0; i < nfilters; ++i) {
    first_step[i] = steps;
    const uint64_t ni = pf[i].key_end - pf[i].key_begin;
    if (pf[i].direct || ni == 0) continue;
    for (uint64_t s = 0; s < ni; s += range1)
      ranges.push_back(PartRange{pf[i].key_begin + s, pf[i].key_begin + std::min(s + range1, ni), i,
                                 static_cast<uint32_t>(steps + s / kStep)});
    const uint64_t si = (ni + kStep - 1) / kStep;
    const uint64_t nc = (pf[i].num_blocks + bpc - 1) / bpc;
    const uint64_t digits = (pf[i].chunk_base + nc - 1) / f2 - pf[i].chunk_base / f2 + 1;
    steps += si;
    runs += si * digits;
  }
  first_step[nfilters] = steps;
  if (ranges.empty() || ranges.size() > 0x7fffffffull || steps * kStep > 0xffffffffull * 16) return BF_OK;
  // longest first: workgroups are dispatched in index order as CUs free up,
  // so the short ranges fill the gaps at the end
  std::stable_sort(ranges.begin(), ranges.end(), [](const PartRange& x, const PartRange& y) {
    return x.end - x.begin > y.end - y.begin;
  });
  // Second-pass items, by digit: the steps of the digit's filters cut so that
  // an item expects about 64 Ki records, or fewer (two steps at least) where
  // that would leave under a thousand items for 256 CUs.  Apply work: one item per chunk of a
  // dense filter with keys; heavily loaded chunks are split over several
  // workgroups (~128 Ki records each, each of which then merges its whole
  // chunk image with atomics).
  const double target = static_cast<double>(std::clamp<uint64_t>(n_dense / 1024, 2 * kStep, 65536));
  std::vector<PartItem> items;
  std::vector<PartWork> work;
  uint64_t batches = 0;
  uint32_t fi = 0;  // first filter with chunks in the digit
  for (uint64_t d = 0; d < f1; ++d) {
    const uint64_t c0 = d * f2, c1 = std::min<uint64_t>(chunks, c0 + f2);
    auto chunk_end = [&](uint32_t i) { return i + 1 < nfilters ? pf[i + 1].chunk_base : chunks; };
    while (fi < nfilters && chunk_end(fi) <= c0) ++fi;
    double acc = 0.0;
    uint64_t t0 = 0, t1 = 0;  // the open item
    auto close = [&] {
      if (t1 > t0) {
        items.push_back(PartItem{static_cast<uint32_t>(d), static_cast<uint32_t>(t0), static_cast<uint32_t>(t1), 0});
        batches += (t1 - t0 + kRegroupRuns - 1) / kRegroupRuns;
      }
      t0 = t1;
      acc = 0.0;
    };
    for (uint32_t i = fi; i < nfilters && pf[i].chunk_base < c1; ++i) {
      const uint64_t ni = pf[i].key_end - pf[i].key_begin;
      const uint64_t si = first_step[i + 1] - first_step[i];
      if (si == 0) continue;
      // the filter's keys spread uniformly over its blocks
      const uint64_t fc0 = std::max(c0, pf[i].chunk_base), fc1 = std::min(c1, chunk_end(i));
      const double per_block = static_cast<double>(ni) / static_cast<double>(pf[i].num_blocks);
      auto blocks_to = [&](uint64_t c) { return std::min((c - pf[i].chunk_base) * bpc, pf[i].num_blocks); };
      const double per_step = per_block * static_cast<double>(blocks_to(fc1) - blocks_to(fc0)) / static_cast<double>(si);
      if (t1 != first_step[i] || t1 == t0) {
        close();
        t0 = t1 = first_step[i];
      }
      const uint32_t i0 = static_cast<uint32_t>(items.size());
      while (t1 < first_step[i + 1]) {
        const uint64_t fit = static_cast<uint64_t>(std::max(1.0, (target - acc) / std::max(per_step, 1e-3)));
        const uint64_t take = std::min(fit, first_step[i + 1] - t1);
        t1 += take;
        acc += per_step * static_cast<double>(take);
        if (acc >= target - 0.5 * per_step) close();
      }
      const uint32_t i1 = static_cast<uint32_t>(items.size()) + (t1 > t0 ? 1 : 0);
      for (uint64_t c = fc0; c < fc1; ++c) {
        const double load = per_block * static_cast<double>(blocks_to(c + 1) - blocks_to(c));
        const uint64_t ns = std::clamp<uint64_t>(static_cast<uint64_t>(load / 131072.0) + 1, 1, 65535);
        for (uint64_t j = 0; j < ns; ++j)
          work.push_back(PartWork{static_cast<uint32_t>(c), static_cast<uint16_t>(j), static_cast<uint16_t>(ns), i0, i1});
      }
    }
    close();
  }
  if (items.empty() || items.size() > 0x7fffffffull || work.size() > 0xffffffffull) return BF_OK;
  part_layout_two(a, L, steps, items.size(), batches, runs, n_dense);
  // tables after the buffers: filters, chunk owners, ranges, items, apply work
  std::vector<uint32_t> owner(chunks);
  for (uint32_t i = 0; i < nfilters; ++i) {
    const uint64_t c_end = i + 1 < nfilters ? pf[i + 1].chunk_base : chunks;
    std::fill(owner.begin() + static_cast<std::ptrdiff_t>(pf[i].chunk_base),
              owner.begin() + static_cast<std::ptrdiff_t>(c_end), i);
  }
  struct Table {
    const void* src;
    uint64_t bytes;
    uint64_t at;
  } tables[] = {{pf.data(), pf.size() * sizeof(PartFilter), 0},   {owner.data(), owner.size() * 4, 0},
                {ranges.data(), ranges.size() * sizeof(PartRange), 0}, {items.data(), items.size() * sizeof(PartItem), 0},
                {work.data(), work.size() * sizeof(PartWork), 0}};
  uint64_t total = L.total;
  for (Table& t : tables) {
    t.at = total;
    total = (total + t.bytes + 255) & ~255ull;
  }
  a.g.ranges = reinterpret_cast<const PartRange*>(1);  // a plan: the multi-filter first pass
  const PartKernels k = part_kernels(f0, a);
  if (!part_runs(a, k)) return BF_OK;
  b->part_scratch = lib_alloc(b->device, total, &b->pooled_scratch);
  if (b->part_scratch == nullptr) return forced ? BF_ENOMEM : BF_OK;  // no memory for it: tiles need little
  uint8_t* base = static_cast<uint8_t*>(b->part_scratch);
  for (const Table& t : tables)
    if (hipMemcpy(base + t.at, t.src, t.bytes, hipMemcpyHostToDevice) != hipSuccess) return BF_EDEVICE;
  part_bind(a, L, b->part_scratch);
  a.p.filters = reinterpret_cast<const PartFilter*>(base + tables[0].at);
  a.g.filters = a.p.filters;
  a.p.chunk_owner = reinterpret_cast<const uint32_t*>(base + tables[1].at);
  a.g.ranges = reinterpret_cast<const PartRange*>(base + tables[2].at);
  a.nranges = static_cast<uint32_t>(ranges.size());
  a.r.list = reinterpret_cast<const PartItem*>(base + tables[3].at);
  a.p.work = reinterpret_cast<const PartWork*>(base + tables[4].at);
  a.nwork = static_cast<uint32_t>(work.size());
  a.p.words = pf[0].words;  // the single-filter fields mirror filter 0
  a.p.num_blocks = pf[0].num_blocks;
  a.p.nfilters = nfilters;
  a.p.k = f0->k;
  a.g.keys = d_keys + h_offsets[0];
  a.g.n = n;
  b->part = a;
  b->part_k = k;
  b->partitioned = true;
  b->part_direct.resize(nfilters);
  for (uint32_t i = 0; i < nfilters; ++i) b->part_direct[i] = static_cast<uint8_t>(pf[i].direct);
  return BF_OK;
}

// The plan's graph: the partitioned construction's five kernels (when taken)
// or the lookups in LDS (where filters take them), then the persistent tiled
// launch (when it has tiles, or when there is nothing else).  The nodes run
// one after another: the tiled launch beside the construction took 4.35 ms
// where the chain takes 4.23 (4,096 filters, 2^28 keys).
bf_status build_graph(bf_batch* b) {
  hipGraphNode_t prev = nullptr, node = nullptr;
  if (hipGraphCreate(&b->graph, 0) != hipSuccess) return BF_EDEVICE;
  auto add_node = [&](const void* fn, dim3 grid, dim3 block, void** args) {
    hipKernelNodeParams p{};
    p.func = const_cast<void*>(fn);
    p.gridDim = grid;
    p.blockDim = block;
    p.sharedMemBytes = 0;
    p.kernelParams = args;
    p.extra = nullptr;
    if (hipGraphAddKernelNode(&node, b->graph, prev ? &prev : nullptr, prev ? 1 : 0, &p) != hipSuccess)
      return false;
    prev = node;
    return true;
  };
  if (b->partitioned) {
    void* gargs[] = {&b->part.g};
    void* rargs[] = {&b->part.r};
    void* pargs[] = {&b->part.p};
    if (!add_node(b->part_k.group, part_grid_group(b->part), dim3(b->part_k.threads1), gargs) ||
        !add_node(b->part_k.plan, dim3(b->part.r.items), dim3(kPlanThreads), rargs) ||
        !add_node(b->part_k.scan, dim3(1), dim3(kScanThreads), rargs) ||
        !add_node(b->part_k.regroup, dim3(b->part.r.items), dim3(kGroupThreads), rargs) ||
        !add_node(b->part_k.apply, part_grid_apply(b->part), dim3(kApplyThreads), pargs))
      return BF_EDEVICE;
  }
  for (bf_batch::Resident& r : b->resident) {
    void* kargs[] = {&r.args};
    if (r.nitems > 0 && !add_node(r.fn, dim3(static_cast<uint32_t>(r.nitems)), dim3(kResidentThreads), kargs))
      return BF_EDEVICE;
  }
  if (b->ntiles > 0 || (!b->partitioned && items_of(b) == 0)) {
    void* kargs[] = {&b->args};
    if (!add_node(b->fn, dim3(b->grid), dim3(kBlockThreads), kargs)) return BF_EDEVICE;
  }
  return hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0) == hipSuccess ? BF_OK
                                                                                     : BF_EDEVICE;
}

// The tiled direct plan: every key of the selected filters (all when
// `only` is null) in tiles of one persistent launch.  Filters go to the 8
// XCD queues by longest-processing-time on their key counts.
bf_status build_tiles(bf_batch* b, bf_filter* const* filters, uint32_t nfilters, const uint64_t* d_keys,
                      const uint64_t* h_offsets, uint8_t* d_out, const std::vector<uint8_t>* only) {
  const int op = b->op;
  const bf_filter* f0 = filters[0];
  // Mapping per size class (identical for all filters of a class).
  for (int c = 0; c < kNumSizeClasses; ++c) {
    const MapSpec m = class_map(op, f0, c);
    bf_mapping_t bm{};
    bm.lanes_per_key = m.theta;
    bm.words_per_lane = m.phi;
    bm.keys_per_lane = m.kt;
    bm.atomic_bits = op == BF_OP_ADD ? m.atomic_bits : 0;
    bm.workgroup_threads = kBlockThreads;  // tiles are planned at this size
    b->mapping[c] = bm;
  }

  std::vector<uint32_t> order(nfilters);
  std::iota(order.begin(), order.end(), 0u);
  std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) {
    return h_offsets[x + 1] - h_offsets[x] > h_offsets[y + 1] - h_offsets[y];
  });
  std::vector<std::vector<BatchTile>> queue(kXcds);
  std::vector<uint64_t> load(kXcds, 0);
  std::vector<BatchTile> items[2];
  // Each item copies a filter or merges an image into it, so items are as long
  // as keeps the launch's tail short: adds of 2^22 keys in 1,024 filters take
  // 0.26 ms with 65,536 keys per item and 0.20 with 8,192; of 2^28 keys in
  // 4,096 filters 3.30 with 32,768, 3.26 with 65,536, 3.28 with 131,072.
  const uint64_t resident_keys = resident_keys_of(b, filters, nfilters, h_offsets);
  const uint64_t item_keys = op == BF_OP_ADD ? std::clamp<uint64_t>(resident_keys / 2048, 8192, 65536)
                                             : std::clamp<uint64_t>(resident_keys / 2048, 4096, kResidentKeys);
  for (uint32_t i : order) {
    const uint64_t n = h_offsets[i + 1] - h_offsets[i];
    if (n == 0 || (only != nullptr && !(*only)[i])) continue;
    const bf_filter* f = filters[i];
    const int cls = size_class_of(f->nbytes);
    if (resides(b, f, n)) {
      const int big = f->nbytes > kResidentBytes[0];
      const uint64_t parts = (n + item_keys - 1) / item_keys;
      for (uint64_t p = 0; p < parts; ++p) {
        const uint64_t from = n * p / parts;
        items[big].push_back({h_offsets[i] + from, i, static_cast<uint32_t>(n * (p + 1) / parts - from)});
        b->tiles_per_class[cls] += 1;
      }
      continue;
    }
    const uint32_t kt = b->mapping[cls].keys_per_lane;
    const uint64_t tile = static_cast<uint64_t>(kBlockThreads) * kt;
    const int x = static_cast<int>(std::min_element(load.begin(), load.end()) - load.begin());
    load[x] += n;
    for (uint64_t s = 0; s < n; s += tile) {
      const uint64_t start = h_offsets[i] + s;
      const uint32_t count = static_cast<uint32_t>(std::min<uint64_t>(tile, n - s));
      const bool vec = count == tile && (start % kt) == 0 &&
                       (reinterpret_cast<uintptr_t>(d_keys) % (8u * kt)) == 0 &&
                       (d_out == nullptr || reinterpret_cast<uintptr_t>(d_out) % kt == 0);
      BatchTile t{};
      t.key_start = start;
      t.filter = i;
      t.meta = count | (static_cast<uint32_t>(cls) << kTileClassShift) | (vec ? kTileVecBit : 0u);
      queue[x].push_back(t);
      b->tiles_per_class[cls] += 1;
    }
  }
  // Interleave: slot 8*j + x holds the j-th tile of queue x (empty if none).
  size_t longest = 0;
  for (const auto& q : queue) longest = std::max(longest, q.size());
  std::vector<BatchTile> tiles(longest * kXcds, BatchTile{0, 0, 0});
  for (int x = 0; x < kXcds; ++x)
    for (size_t j = 0; j < queue[x].size(); ++j) tiles[j * kXcds + x] = queue[x][j];
  b->ntiles = tiles.size();
  for (int big = 0; big < 2; ++big) {
    b->resident[big].nitems = items[big].size();
    tiles.insert(tiles.end(), items[big].begin(), items[big].end());
  }

  int cus = 256;
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, f0->device) == hipSuccess && prop.multiProcessorCount > 0)
    cus = prop.multiProcessorCount;
  uint64_t grid = static_cast<uint64_t>(cus) * kWgPerCu;
  grid = std::min<uint64_t>(grid, std::max<uint64_t>(b->ntiles, kXcds));
  grid = (grid + kXcds - 1) / kXcds * kXcds;  // a multiple of 8 keeps slots on their XCD
  b->grid = static_cast<uint32_t>(grid);

  std::vector<BatchFilter> descs(nfilters);
  for (uint32_t i = 0; i < nfilters; ++i) {
    const bf_filter* f = filters[i];
    descs[i].words = f->d_words;
    descs[i].hash_init = xxh64_u64_init(f->seed);
    descs[i].nb_lo = static_cast<uint32_t>(f->num_blocks);
    descs[i].nb_hi_mask = (f->num_blocks >> 32) ? 0xffffffffu : 0u;
    descs[i].keys = d_keys;
    descs[i].out = d_out;
    descs[i].reserved = 0;
  }
  const size_t tiles_bytes = std::max<size_t>(1, tiles.size()) * sizeof(BatchTile);
  b->d_filters = static_cast<BatchFilter*>(
      lib_alloc(b->device, descs.size() * sizeof(BatchFilter), &b->pooled_filters));
  if (b->d_filters == nullptr) return BF_ENOMEM;
  b->d_tiles = static_cast<BatchTile*>(lib_alloc(b->device, tiles_bytes, &b->pooled_tiles));
  if (b->d_tiles == nullptr) return BF_ENOMEM;
  if (hipMemcpy(b->d_filters, descs.data(), descs.size() * sizeof(BatchFilter),
                hipMemcpyHostToDevice) != hipSuccess ||
      (!tiles.empty() && hipMemcpy(b->d_tiles, tiles.data(), tiles.size() * sizeof(BatchTile),
                                   hipMemcpyHostToDevice) != hipSuccess)) {
    return BF_EDEVICE;
  }

  b->args.filters = b->d_filters;
  b->args.tiles = b->d_tiles;
  b->args.ntiles = b->ntiles;
  b->args.k = f0->k;
  for (int big = 0; big < 2; ++big) {
    b->resident[big].args.filters = b->d_filters;
    b->resident[big].args.items = b->d_tiles + b->ntiles + (big ? b->resident[0].nitems : 0);
    b->resident[big].args.k = f0->k;
  }

  return BF_OK;
}

}  // namespace

extern "C" {

bf_status bf_batch_plan(int op, bf_filter* const* filters, uint32_t nfilters,
                        const uint64_t* d_keys, const uint64_t* h_offsets, uint8_t* d_out,
                        bf_batch** out) {
  if (out == nullptr || filters == nullptr || h_offsets == nullptr || nfilters == 0)
    return BF_EINVAL;
  if (op != BF_OP_ADD && op != BF_OP_CONTAINS) return BF_EINVAL;
  const bf_filter* f0 = filters[0];
  if (f0 == nullptr) return BF_EINVAL;
  for (uint32_t i = 0; i < nfilters; ++i) {
    const bf_filter* f = filters[i];
    if (f != nullptr && f->layout != BF_LAYOUT_SECTORIZED) return BF_EUNSUPPORTED;
    if (f == nullptr || f->s != f0->s || f->word_bits != f0->word_bits || f->k != f0->k ||
        f->device != f0->device || f->salts != f0->salts)
      return BF_EINVAL;
    if (h_offsets[i + 1] < h_offsets[i]) return BF_EINVAL;
  }
  const uint64_t nkeys = h_offsets[nfilters] - h_offsets[0];
  if (nkeys > 0 && (d_keys == nullptr || reinterpret_cast<uintptr_t>(d_keys) % 8 != 0))
    return BF_EINVAL;
  if (op == BF_OP_CONTAINS && nkeys > 0 && d_out == nullptr) return BF_EINVAL;

  const void* fn = kernel_table(f0->salts == kSaltsParquet).batch_fn[batch_index(op, static_cast<int>(f0->word_bits),
                                                   static_cast<int>(f0->s), k_index(f0->k))];
  if (fn == nullptr) return BF_EUNSUPPORTED;

  bf_batch* b = new (std::nothrow) bf_batch{};
  if (b == nullptr) return BF_ENOMEM;
  b->op = op;
  b->nfilters = nfilters;
  b->nkeys = nkeys;
  b->filters.assign(filters, filters + nfilters);
  b->offsets.assign(h_offsets, h_offsets + nfilters + 1);
  b->d_keys = d_keys;
  b->d_out = d_out;
  b->fn = fn;
  // (the caller's strategy of an add plan stands)
  if (op == BF_OP_CONTAINS || f0->mapping[BF_OP_ADD].strategy == BF_STRATEGY_AUTO)
    for (int big = 0; big < 2; ++big)
      b->resident[big].fn = kernel_table(f0->salts == kSaltsParquet)
                                .resident_fn[big][batch_index(op, static_cast<int>(f0->word_bits),
                                                              static_cast<int>(f0->s), k_index(f0->k))];
  if (!resides_pays(b, filters, nfilters, h_offsets)) b->resident[0].fn = b->resident[1].fn = nullptr;
  b->device = f0->device;

  if (op == BF_OP_ADD) {
    const void* fns[2] = {b->resident[0].fn, b->resident[1].fn};
    bf_status pst = plan_partitioned(b, filters, nfilters, d_keys, h_offsets);
    if (pst != BF_OK) {
      free_plan(b);
      return pst;
    }
    // (small filters that would have joined a construction run in LDS)
    for (int big = 0; big < 2 && !b->partitioned; ++big) b->resident[big].fn = fns[big];
  }
  // The tiled direct launch: every filter, or (partitioned plan) the filters
  // left to it that have keys.
  bool tiled = !b->partitioned;
  if (b->partitioned)
    for (uint32_t i = 0; i < nfilters; ++i)
      tiled = tiled || (b->part_direct[i] && h_offsets[i + 1] > h_offsets[i]);
  if (tiled) {
    const bf_status st =
        build_tiles(b, filters, nfilters, d_keys, h_offsets, d_out, b->partitioned ? &b->part_direct : nullptr);
    if (st != BF_OK) {
      (void)hipGetLastError();
      free_plan(b);
      return st;
    }
  } else {
    b->ntiles = 0;
    b->grid = part_grid_group(b->part).x;
  }
  if (build_graph(b) != BF_OK) {
    (void)hipGetLastError();
    free_plan(b);
    return BF_EDEVICE;
  }
  *out = b;
  return BF_OK;
}

bf_status bf_batch_launch(bf_batch* b, void* stream) {
  if (b == nullptr) return BF_EINVAL;
  if (b->ntiles + items_of(b) == 0 && !b->partitioned) return BF_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  std::lock_guard<std::mutex> lk(b->mark_mu);
  const CallMark mark = begin_launch(b, s);
  if (hipGraphLaunch(b->exec, s) != hipSuccess) return BF_EDEVICE;
  return end_launch(b, s, mark);
}

bf_status bf_batch_launch_direct(bf_batch* b, void* stream) {
  if (b == nullptr) return BF_EINVAL;
  if (b->ntiles + items_of(b) == 0 && !b->partitioned) return BF_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  std::lock_guard<std::mutex> lk(b->mark_mu);
  CallMark mark = begin_launch(b, s);
  if (b->partitioned) {
    const bf_status st = part_launch(b->part, b->part_k, s);
    if (st != BF_OK) return st;
  }
  for (bf_batch::Resident& r : b->resident) {
    if (r.nitems == 0) continue;
    void* kargs[] = {&r.args};
    if (hipLaunchKernel(r.fn, dim3(static_cast<uint32_t>(r.nitems)), dim3(kResidentThreads), kargs, 0, s) !=
        hipSuccess)
      return BF_EDEVICE;
  }
  if (b->ntiles > 0) {
    void* kargs[] = {&b->args};
    if (launch_marked(b->fn, dim3(b->grid), dim3(kBlockThreads), kargs, s, &mark) != hipSuccess) return BF_EDEVICE;
  }
  return end_launch(b, s, mark);
}

bf_status bf_batch_launch_per_filter(bf_batch* b, void* stream) {
  if (b == nullptr) return BF_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  for (uint32_t i = 0; i < b->nfilters; ++i) {
    const uint64_t n = b->offsets[i + 1] - b->offsets[i];
    if (n == 0) continue;
    const uint64_t off = b->offsets[i];
    bf_status st = b->op == BF_OP_ADD
                       ? launch_routed(b->filters[i], BF_OP_ADD, b->d_keys + off, n, nullptr, s)
                       : launch_routed(b->filters[i], BF_OP_CONTAINS, b->d_keys + off, n, b->d_out + off, s);
    if (st != BF_OK) return st;
  }
  return BF_OK;
}

bf_status bf_batch_info(const bf_batch* b, bf_batch_info_t* out) {
  if (b == nullptr || out == nullptr) return BF_EINVAL;
  bf_batch_info_t i{};
  i.op = static_cast<uint32_t>(b->op);
  i.nfilters = b->nfilters;
  i.nkeys = b->nkeys;
  i.ntiles = b->ntiles + items_of(b);
  i.grid = b->grid;
  i.strategy = b->partitioned ? BF_STRATEGY_PARTITIONED : BF_STRATEGY_DIRECT;
  for (int c = 0; c < kNumSizeClasses; ++c) {
    i.tiles_per_class[c] = b->tiles_per_class[c];
    i.mapping[c] = b->mapping[c];
  }
  *out = i;
  return BF_OK;
}

bf_status bf_batch_destroy(bf_batch* b) {
  if (b == nullptr) return BF_OK;
  // the host waits for the plan's own launches only (its graph is destroyed
  // next); its memory then returns to the pool in the library stream's order
  bf_status st = BF_OK;
  if (b->unmarked) {
    if (hipDeviceSynchronize() != hipSuccess) st = BF_EDEVICE;
  } else {
    for (auto& m : b->marks)
      if (hipEventSynchronize(m.second) != hipSuccess) st = BF_EDEVICE;
  }
  free_plan(b);
  return st;
}

}  // extern "C"
