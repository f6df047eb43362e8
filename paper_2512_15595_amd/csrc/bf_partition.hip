// bf_partition.hip -- host side of partitioned construction: geometry,
// workspace and the launch sequence (kernels in bf_group.hpp and
// bf_partition.hpp), for one filter and for a table of filters.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <map>
#include <mutex>

#include "bf_internal.hpp"
#include "bf_variant_registry.hpp"
#include "bf_partition.hpp"
#include "bf_registry.hpp"

namespace bfhip {

namespace {

uint64_t align256(uint64_t v) { return (v + 255) & ~255ull; }
uint64_t ceil_div(uint64_t a, uint64_t b) { return (a + b - 1) / b; }

uint32_t ceil_pow2(uint64_t v) {
  uint32_t p = 1;
  while (p < v) p <<= 1;
  return p;
}

// Keys of one first-pass step: kStep, or for the classic filter the whole
// keys whose k records fit it.
uint64_t step_keys(uint64_t records_per_key) {
  if (records_per_key <= 1) return kStep;
  return static_cast<uint64_t>(kClassicThreads) * (kStep / kClassicThreads / records_per_key);
}

}  // namespace

uint32_t part_chunk_shift(uint32_t words_per_block, uint32_t word_bits) {
  const uint64_t bpc = kChunkBytes / (static_cast<uint64_t>(words_per_block) * word_bits / 8);
  uint32_t shift = 0;
  while ((1ull << shift) < bpc) ++shift;
  return shift;
}

// Digits balanced between the passes: f2 ~ sqrt(chunks).  Both passes write
// whole steps, so their cost hardly depends on the digits; what does is the
// length of the runs that the next pass reads.
bool part_digits(uint64_t chunks, uint32_t chunk_shift, uint32_t most_digits2, PartArgs& a) {
  const uint64_t root = static_cast<uint64_t>(std::ceil(std::sqrt(static_cast<double>(chunks))));
  const uint32_t f2 = std::min<uint32_t>(ceil_pow2(std::max<uint64_t>(root, 1)), most_digits2);
  const uint64_t f1 = ceil_div(chunks, f2);
  if (chunks == 0 || f1 > static_cast<uint64_t>(kMaxDigits)) return false;
  a.p.chunk_shift = chunk_shift;
  a.chunks = chunks;
  a.p.low_bits = 0;
  while ((1u << a.p.low_bits) < f2) ++a.p.low_bits;
  a.g.shift = chunk_shift + a.p.low_bits;
  a.g.digits = static_cast<uint32_t>(f1);
  a.r.shift = chunk_shift;
  a.r.digits = f2;
  return true;
}

// The two-pass buffers for `steps` first-pass steps, `items` second-pass
// items of `batches` batches in all, at most `runs` non-empty runs of the
// first table and `records` records.  A run of c records is ceil(c / unit)
// units and only a batch's last output step is partial, which bounds the
// second pass's steps whatever the keys are.
void part_layout_two(PartArgs& a, PartLayout& L, uint64_t steps, uint64_t items, uint64_t batches, uint64_t runs,
                     uint64_t records) {
  a.one_pass = false;
  a.g.steps = static_cast<uint32_t>(steps);
  a.g.stride = ceil_div(steps, 16) * 16;
  a.r.stride1 = a.g.stride;
  a.r.steps1 = a.g.steps;
  a.r.items = static_cast<uint32_t>(items);
  const uint64_t unit = a.short_units ? kShortUnit : kUnit;
  const uint64_t units = records / unit + std::min(runs, records);
  const uint64_t steps2 = units / (kStep / unit) + batches;
  a.r.stride2 = ceil_div(steps2, 16) * 16;
  uint64_t off = 0;
  auto take = [&off](uint64_t bytes) {
    const uint64_t at = off;
    off = align256(off + bytes);
    return at;
  };
  L.rec = take(8 * steps * kStep);
  L.table1 = take(4 * a.g.digits * a.g.stride);
  L.lo = take(4 * steps2 * kStep);
  L.blk = take(2 * steps2 * kStep);
  L.table2 = take(4 * a.r.digits * a.r.stride2);
  L.item_count = take(4 * items);
  L.slot0 = take(4 * (items + 1));
  L.total = off;
}

namespace {

// One pass for a filter of at most kChunkDigits chunks: the first pass's
// digit is the chunk, and the apply step reads its runs.
void one_pass_geometry(uint64_t chunks, uint32_t chunk_shift, uint64_t steps, PartArgs& a, PartLayout& L) {
  a.one_pass = true;
  a.p.chunk_shift = chunk_shift;
  a.p.low_bits = 0;
  a.p.steps = static_cast<uint32_t>(steps);
  a.chunks = chunks;
  a.g.shift = chunk_shift;
  a.g.digits = static_cast<uint32_t>(chunks);
  a.g.steps = static_cast<uint32_t>(steps);
  a.g.stride = ceil_div(steps, 16) * 16;
  uint64_t off = 0;
  auto take = [&off](uint64_t bytes) {
    const uint64_t at = off;
    off = align256(off + bytes);
    return at;
  };
  L.lo = take(4 * steps * kStep);
  L.blk = take(2 * steps * kStep);
  L.table1 = take(4 * chunks * a.g.stride);
  L.total = off;
}

}  // namespace

void part_bind(PartArgs& a, const PartLayout& L, void* base_ptr) {
  uint8_t* base = static_cast<uint8_t*>(base_ptr);
  a.g.table = reinterpret_cast<uint32_t*>(base + L.table1);
  uint32_t* lo = reinterpret_cast<uint32_t*>(base + L.lo);
  uint16_t* blk = reinterpret_cast<uint16_t*>(base + L.blk);
  a.g.local_mask = (1u << a.p.chunk_shift) - 1;
  a.p.lo = lo;
  a.p.blk = blk;
  if (a.one_pass) {
    a.g.lo = lo;
    a.g.blk = blk;
    a.p.table = a.g.table;
    a.p.stride = a.g.stride;
    return;
  }
  a.g.rec = reinterpret_cast<uint64_t*>(base + L.rec);
  a.r.rec = a.g.rec;
  a.r.table1 = a.g.table;
  a.r.item_count = reinterpret_cast<uint32_t*>(base + L.item_count);
  a.r.slot0 = reinterpret_cast<uint32_t*>(base + L.slot0);
  a.r.lo = lo;
  a.r.blk = blk;
  a.r.table2 = reinterpret_cast<uint32_t*>(base + L.table2);
  a.p.table = a.r.table2;
  a.p.stride = a.r.stride2;
  a.p.slot0 = a.r.slot0;
  a.p.per_digit = a.r.per_digit;
}

// The kernels of a partitioned add of f with geometry a.
PartKernels part_kernels(const bf_filter* f, const PartArgs& a) {
  // Units of 8 slots where the runs are short (32 records of a step or
  // fewer), of 16 where they are longer.
  const int unit8 = a.one_pass && a.chunks >= 256 ? 1 : 0;
  PartKernels k{};
  k.threads1 = kGroupThreads;
  if (f->layout == BF_LAYOUT_CLASSIC) {
    ensure_variant_registry();
    const VariantRegistry& r = variant_registry();
    const int pow2 = (f->num_bits & (f->num_bits - 1)) == 0 ? 1 : 0;
    k.threads1 = kClassicThreads;
    k.group = r.classic_group[classic_group_index(k_index(f->k), pow2, a.g.digits, a.one_pass)];
    k.apply = r.classic_apply[unit8];
  } else if (f->layout == BF_LAYOUT_CACHE_SECTORIZED) {
    ensure_variant_registry();
    const int idx = csbf_part_index(static_cast<int>(f->word_bits), static_cast<int>(f->s),
                                    static_cast<int>(f->groups), k_index(f->k));
    k.apply = variant_registry().csbf_apply[unit8][idx];
  } else {
    const int idx = batch_index(0, static_cast<int>(f->word_bits), static_cast<int>(f->s), k_index(f->k));
    k.apply = kernel_table(f->salts == kSaltsParquet).apply_fn[unit8][idx];
  }
  if (f->layout != BF_LAYOUT_CLASSIC) k.group = group_keys_fn(a.g.digits, a.one_pass, a.g.ranges != nullptr, false);
  if (!a.one_pass) {
    k.plan = regroup_plan_fn(a.short_units);
    k.scan = regroup_scan_fn();
    k.regroup = regroup_fn(a.r.digits, false, a.short_units);
  }
  return k;
}

bool part_runs(const PartArgs& a, const PartKernels& k) {
  return k.group != nullptr && k.apply != nullptr && (a.one_pass || (k.plan != nullptr && k.regroup != nullptr));
}

bf_status part_launch(const PartArgs& a, const PartKernels& k, hipStream_t stream) {
  if (!part_runs(a, k)) return BF_EUNSUPPORTED;
  PartArgs copy = a;
  void* gargs[] = {&copy.g};
  void* rargs[] = {&copy.r};
  void* pargs[] = {&copy.p};
  hipError_t e = hipLaunchKernel(k.group, part_grid_group(a), dim3(k.threads1), gargs, 0, stream);
  if (e == hipSuccess && !a.one_pass) {
    e = hipLaunchKernel(k.plan, dim3(a.r.items), dim3(kPlanThreads), rargs, 0, stream);
    if (e == hipSuccess) e = hipLaunchKernel(k.scan, dim3(1), dim3(kScanThreads), rargs, 0, stream);
    if (e == hipSuccess) e = hipLaunchKernel(k.regroup, dim3(a.r.items), dim3(kGroupThreads), rargs, 0, stream);
  }
  if (e == hipSuccess) e = hipLaunchKernel(k.apply, part_grid_apply(a), dim3(kApplyThreads), pargs, 0, stream);
  return e == hipSuccess && hipGetLastError() == hipSuccess ? BF_OK : BF_EDEVICE;
}

dim3 part_grid_group(const PartArgs& a) {
  if (a.g.ranges) return dim3(a.nranges);
  return dim3(static_cast<uint32_t>(ceil_div(a.g.steps, a.g.wg_steps)));
}
dim3 part_grid_apply(const PartArgs& a) {
  const uint64_t items = a.p.work ? a.nwork : a.chunks * std::max<uint32_t>(a.p.split, 1);
  return dim3(static_cast<uint32_t>(std::max<uint64_t>(1, items)));
}

namespace {

// Chunks of a filter and log2 of the blocks in each; the classic filter is
// partitioned as blocks of one 32-bit word, with k records per key.
uint64_t filter_chunks(const bf_filter* f, uint32_t* shift) {
  const bool classic = f->layout == BF_LAYOUT_CLASSIC;
  *shift = classic ? part_chunk_shift(1, 32) : part_chunk_shift(f->s, f->word_bits);
  const uint64_t blocks = classic ? f->num_bits / 32 : f->num_blocks;
  return (blocks + (1ull << *shift) - 1) >> *shift;
}

uint64_t records_per_key(const bf_filter* f) { return f->layout == BF_LAYOUT_CLASSIC ? f->k : 1; }

bool single_geometry(const bf_filter* f, uint64_t n, PartArgs& a, PartLayout& L) {
  uint32_t shift;
  const uint64_t chunks = filter_chunks(f, &shift);
  const uint64_t records = n * records_per_key(f);
  const uint64_t steps = ceil_div(n, step_keys(records_per_key(f)));
  a.g.n = n;
  a.g.wg_steps = static_cast<uint32_t>(std::max<uint64_t>(ceil_div(steps, 1024), 1));
  // A filter of few chunks (L2 or Infinity-Cache sized) leaves too few to
  // fill 256 CUs: every chunk's records are split over several apply
  // workgroups (at least 8 Ki records each), about two thousand in all.
  // Split slices merge with atomic OR.
  const uint64_t split_fill = ceil_div(2048, chunks);
  a.p.split =
      static_cast<uint32_t>(std::clamp<uint64_t>(std::min<uint64_t>(split_fill, records / chunks / 8192), 1, 1024));
  if (chunks <= static_cast<uint64_t>(kChunkDigits)) {
    one_pass_geometry(chunks, shift, steps, a, L);
    return true;
  }
  if (chunks > static_cast<uint64_t>(kMaxChunks) || !part_digits(chunks, shift, kWideDigits2, a)) return false;
  // The fewer records a first-pass run has (32 of a step of 256 digits), the
  // more of its last unit is empty, and the second pass's buffers must hold
  // that for any keys: units of 8 slots and 1,024 second digits instead of 512
  // keep the workspace of 2^28 keys into 32 GiB at 5.3 GiB, not 8.4, and into
  // 4 GiB at 4.3, not 4.7.
  a.short_units = a.g.digits >= 256;
  // Second-pass items of about 64 Ki records (8 steps), and at least about
  // 512 of them where every item still has a full step.
  const uint64_t per_bucket = ceil_div(records, a.g.digits);
  const uint64_t fill = ceil_div(512, a.g.digits);
  a.r.per_digit = static_cast<uint32_t>(
      std::max<uint64_t>(std::max(ceil_div(per_bucket, 65536), std::min<uint64_t>(fill, per_bucket / kStep)), 1));
  a.r.item_steps = static_cast<uint32_t>(ceil_div(steps, a.r.per_digit));
  const uint64_t items = static_cast<uint64_t>(a.g.digits) * a.r.per_digit;
  part_layout_two(a, L, steps, items, items * ceil_div(a.r.item_steps, kRegroupRuns), steps * a.g.digits, records);
  return true;
}

// The size at which bf_add_noalloc accounts an add of n keys: 14-22 bytes per
// key, about 6 into a filter that takes one pass.  It is the size of buckets
// for the expected load of uniformly hashed keys plus six standard
// deviations, not what a pass takes: it only sets the number of keys that
// call accepts, which callers rely on, whatever the geometry.
uint64_t capacity(double mean, uint64_t margin, uint64_t align) {
  const double c = mean + 6.0 * std::sqrt(mean) + static_cast<double>(margin);
  return (static_cast<uint64_t>(std::ceil(c)) + align - 1) / align * align;
}

uint64_t noalloc_bytes(const bf_filter* f, uint64_t n) {
  uint32_t shift;
  const uint64_t chunks = filter_chunks(f, &shift);
  const uint64_t per_key = records_per_key(f), records = n * per_key;
  const bool two = chunks > static_cast<uint64_t>(kChunkDigits) || f->layout == BF_LAYOUT_CLASSIC;
  constexpr uint64_t kSpare = 64;
  const uint64_t slots2 = chunks * capacity(static_cast<double>(records) / static_cast<double>(chunks), 64, 16);
  uint64_t off = 0, fills = chunks;
  if (two) {
    PartArgs a{};
    if (!part_digits(chunks, shift, kMaxDigits2, a)) return 0;
    const uint64_t keys = step_keys(per_key);
    const uint64_t range = std::max(ceil_div(ceil_div(n, 1024), keys) * keys, keys);
    const uint64_t g1 = std::max<uint64_t>(ceil_div(n, range), 1);
    const uint64_t slice = capacity(static_cast<double>(range * per_key) / a.g.digits, 16, 16);
    off = align256(8 * (a.g.digits * g1 * slice + kSpare));
    fills += a.g.digits * g1;
  }
  off = align256(off + 4 * (slots2 + kSpare));
  off = align256(off + 2 * (slots2 + kSpare));
  return align256(off + 8 * fills);
}

}  // namespace

bool partition_applicable(const bf_filter* f, uint64_t n) {
  if (f->layout == BF_LAYOUT_SECTORIZED_CHAINED) return false;
  // classic records address 32-bit words by a 32-bit index (m <= 2^37) and
  // need a compiled k (at most 16 positions per key)
  if (f->layout == BF_LAYOUT_CLASSIC && (f->num_bits > (1ull << 37) || k_index(f->k) == 0))
    return false;
  PartArgs a{};
  PartLayout L{};
  return n > 0 && n < (1ull << 40) && single_geometry(f, 1, a, L);
}

// The workspace of partitioned adds and grouped lookups comes from one
// stream-ordered memory pool per device: taken at the start of a call and
// returned at its end on the same stream, so a call never synchronizes the
// device and no filter keeps a workspace.  The pool keeps its memory for later
// calls (returned at every synchronization instead, 2^28 lookups in 1 GiB with
// a wait after each took 3.5 ms, not 3.1, and adds up to 124, not 2.5) until a
// filter or plan needs it or the caller asks for it (bf_release_workspace).
namespace {
std::mutex g_pool_mu;
std::map<int, hipMemPool_t> g_pools;
}  // namespace

hipMemPool_t workspace_pool(int device) {
  std::lock_guard<std::mutex> lk(g_pool_mu);
  auto it = g_pools.find(device);
  if (it != g_pools.end()) return it->second;
  hipMemPoolProps props{};
  props.allocType = hipMemAllocationTypePinned;
  props.location.type = hipMemLocationTypeDevice;
  props.location.id = device;
  hipMemPool_t pool = nullptr;
  if (hipMemPoolCreate(&pool, &props) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  uint64_t keep = UINT64_MAX;
  (void)hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep);
  g_pools[device] = pool;
  return pool;
}

void* workspace_alloc(int device, uint64_t bytes, hipStream_t stream) {
  hipMemPool_t pool = workspace_pool(device);
  void* p = nullptr;
  if (pool != nullptr && hipMallocFromPoolAsync(&p, bytes, pool, stream) == hipSuccess) return p;
  (void)hipGetLastError();
  return nullptr;
}

bool release_workspace(int device) {
  std::lock_guard<std::mutex> lk(g_pool_mu);
  auto it = g_pools.find(device);
  if (it == g_pools.end()) return true;
  // no call that returned its workspace in stream order is still using it
  if (hipDeviceSynchronize() == hipSuccess && hipMemPoolTrimTo(it->second, 0) == hipSuccess) return true;
  (void)hipGetLastError();
  return false;
}

namespace {


// One pass of a partitioned add over the workspace `ws` (at least L.total
// bytes of the geometry single_geometry gives for n): sets the arguments and
// enqueues the kernels.
bf_status partitioned_pass_in(bf_filter* f, const uint64_t* keys, hipStream_t stream, PartArgs& a,
                              const PartLayout& L, void* ws) {
  part_bind(a, L, ws);
  a.p.words = f->d_words;
  a.p.num_blocks = f->layout == BF_LAYOUT_CLASSIC ? f->num_bits / 32 : f->num_blocks;
  a.g.num_bits = f->num_bits;
  if ((f->num_bits & (f->num_bits - 1)) == 0) {
    uint32_t lg = 0;
    while ((1ull << lg) < f->num_bits) ++lg;
    a.g.bit_shift = 64 - lg;
  }
  a.g.hash_init = xxh64_u64_init(f->seed);
  a.g.nb_lo = static_cast<uint32_t>(f->num_blocks);
  a.g.nb_hi_mask = (f->num_blocks >> 32) ? 0xffffffffu : 0u;
  a.g.keys = keys;
  a.p.nfilters = 1;
  // the cache-sectorized rule takes the bits per selected word
  a.p.k = f->layout == BF_LAYOUT_CACHE_SECTORIZED ? f->k / f->groups : f->k;
  return part_launch(a, part_kernels(f, a), stream);
}

// One pass with its workspace taken from the device pool and returned at
// its end, both in stream order.
bf_status partitioned_pass(bf_filter* f, const uint64_t* keys, uint64_t n, hipStream_t stream) {
  PartArgs a{};
  PartLayout L{};
  if (!single_geometry(f, n, a, L) || !part_runs(a, part_kernels(f, a))) return BF_EUNSUPPORTED;
  if (workspace_pool(f->device) == nullptr) return BF_EDEVICE;
  void* ws = workspace_alloc(f->device, L.total, stream);
  if (ws == nullptr) return BF_ENOMEM;
  bf_status st = partitioned_pass_in(f, keys, stream, a, L, ws);
  if (hipFreeAsync(ws, stream) != hipSuccess && st == BF_OK) st = BF_EDEVICE;
  return st;
}

uint64_t max_pass_keys(const bf_filter* f) { return std::max<uint64_t>((1ull << 28) / records_per_key(f), 1); }

}  // namespace

uint64_t partition_pass_bytes(const bf_filter* f, uint64_t n) {
  PartArgs a{};
  PartLayout L{};
  return n > 0 && single_geometry(f, n, a, L) ? L.total : 0;
}

// noalloc_bytes decides what is taken; an add whose real workspace is larger
// than ws_bytes (few keys into a large filter, or a table of many digits)
// runs in several passes over it, which give the same words: of n keys,
// halved until the workspace of a pass fits, and that of the shorter last
// pass too (a geometry of fewer keys can need more: fewer second-pass items
// hold more batches).
uint64_t noalloc_pass_keys(const bf_filter* f, uint64_t n, uint64_t ws_bytes) {
  if (!partition_applicable(f, n) || n > max_pass_keys(f) || noalloc_bytes(f, n) > ws_bytes) return 0;
  for (uint64_t pass = n; pass > 0; pass = pass > 1 ? (pass + 1) / 2 : 0)
    if (std::max(partition_pass_bytes(f, pass), partition_pass_bytes(f, n % pass)) <= ws_bytes) return pass;
  return 0;
}

bf_status partitioned_add_in(bf_filter* f, const uint64_t* keys, uint64_t n, hipStream_t stream,
                             void* ws, uint64_t ws_bytes) {
  if (n == 0 || n > max_pass_keys(f)) return BF_EINVAL;
  const uint64_t pass = noalloc_pass_keys(f, n, ws_bytes);
  if (pass == 0) return BF_ESCRATCH;
  for (uint64_t off = 0; off < n; off += pass) {
    PartArgs a{};
    PartLayout L{};
    if (!single_geometry(f, std::min(pass, n - off), a, L) || !part_runs(a, part_kernels(f, a))) return BF_EUNSUPPORTED;
    const bf_status st = partitioned_pass_in(f, keys + off, stream, a, L, ws);
    if (st != BF_OK) return st;
  }
  return BF_OK;
}

// Passes of at most 2^28 records bound the workspace (4.1 GiB into 1 GiB, 4.3
// into 4 GiB, 5.3 into 32 GiB; 5.1, 5.3 and, at 16 GiB, 6.5 for the classic
// filter: the shorter the first pass's runs, the emptier their last units);
// each pass after the first reads and writes the touched chunks once more.
bf_status partitioned_add(bf_filter* f, const uint64_t* keys, uint64_t n, hipStream_t stream) {
  const uint64_t max_keys = max_pass_keys(f);
  for (uint64_t off = 0; off < n; off += max_keys) {
    const bf_status st = partitioned_pass(f, keys + off, std::min(max_keys, n - off), stream);
    if (st != BF_OK) return st;
  }
  return BF_OK;
}

uint64_t partition_workspace_bytes(const bf_filter* f, uint64_t n) {
  if (!partition_applicable(f, n)) return 0;
  const uint64_t most = max_pass_keys(f), rest = n % most;
  // the passes' workspaces follow one another
  return std::max(partition_pass_bytes(f, std::min(n, most)), n > most ? partition_pass_bytes(f, rest) : 0);
}

}  // namespace bfhip
