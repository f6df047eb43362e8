// bf_lookup.hip -- host side of the grouped lookup (bf_lookup.hpp): when it
// is taken, its workspace and launches, and its return kernels, which depend
// on no layout.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "bf_internal.hpp"
#include "bf_lookup.hpp"
#include "bf_partition.hpp"
#include "bf_registry.hpp"
#include "bf_resident.hpp"

namespace bfhip {

namespace {

// Whether the keys of a pass repeat so often that looking them up directly is
// faster, because the repeated ones' lines stay in the caches: *direct is set
// where at least `limit` of kSampleKeys sampled keys were seen before in the
// sample.  The sample's size is of the order of the lines that an XCD's L2
// holds, so that a key seen twice in it is about one whose line the L2 keeps;
// it is taken in kSampleKeys / 64 stretches of 64 keys, which shows repeats
// that are neighbours too (5 us with the launch).  A bit of kSampleBits stands
// for a key that was seen: of different keys 127 look like repeats.
constexpr int kSampleThreads = 1024;
constexpr int kSampleKeys = 8192;
constexpr uint32_t kSampleBits = 1u << 18;
constexpr uint32_t kSampleChance = 127;

__global__ __launch_bounds__(kSampleThreads) void sample_kernel(const uint64_t* keys, uint64_t n, uint64_t hash_init,
                                                                uint32_t limit, uint32_t* direct) {
  __shared__ __attribute__((aligned(16))) uint32_t bits[kSampleBits / 32];
  __shared__ uint32_t count;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  if (n < kSampleKeys || limit == 0) {
    if (tid == 0) *direct = 1;
    return;
  }
  constexpr int kPer = kSampleKeys / kSampleThreads;
  constexpr uint64_t kStretches = kSampleKeys / 64;
  uint64_t key[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    key[j] = keys[(n - 64) * (j * (kSampleThreads / 64) + wave) / (kStretches - 1) + lane];
  for (uint32_t i = tid; i < kSampleBits / 128; i += kSampleThreads) reinterpret_cast<u32x4*>(bits)[i] = u32x4{0u, 0u, 0u, 0u};
  if (tid == 0) count = 0;
  __syncthreads();
  uint32_t seen = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint32_t i = static_cast<uint32_t>(xxh64_u64(key[j], hash_init)) & (kSampleBits - 1);
    const uint32_t bit = 1u << (i & 31u);
    uint32_t old = bits[i >> 5];
    if ((old & bit) == 0) old = atomicOr(&bits[i >> 5], bit);
    seen += (old & bit) != 0 ? 1u : 0u;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) seen += __shfl_down(seen, off, 64);
  if (lane == 0) atomicAdd(&count, seen);
  __syncthreads();
  if (tid == 0) *direct = count >= limit ? 1u : 0u;
}

// A second-pass step's results at the slots of the first pass that its
// records were read from.
__global__ __launch_bounds__(kReturnThreads) void return_slots_kernel(ReturnSlotsArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t res[kStep];
  __shared__ uint32_t units[kStepUnits];
  static_assert(kStepUnits == kReturnThreads && kStep / 16 == kReturnThreads, "a unit and a vector per thread");
  if (*a.direct != 0 || blockIdx.x >= *a.nsteps) return;
  const uint32_t tid = threadIdx.x;
  const uint64_t s = static_cast<uint64_t>(blockIdx.x) * kStep;
  reinterpret_cast<u32x4*>(res)[tid] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(a.res + s) + tid);
  units[tid] = a.units[static_cast<uint64_t>(blockIdx.x) * kStepUnits + tid];
  uint16_t place[kStep / kReturnThreads];
#pragma unroll
  for (int j = 0; j < kStep / kReturnThreads; ++j) place[j] = __builtin_nontemporal_load(a.place + s + tid + j * kReturnThreads);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kStep / kReturnThreads; ++j) {
    const uint32_t p = tid + j * kReturnThreads;
    const uint32_t u = units[p / kUnit];
    if (u != 0xffffffffu && p % kUnit <= (u & 15u)) 
      a.out[(u >> 4) + p % kUnit] = place[j] == kNoPlace ? kUntested : res[place[j]];
  }
}

uint64_t align256(uint64_t v) { return (v + 255) & ~255ull; }
uint64_t ceil_div(uint64_t a, uint64_t b) { return (a + b - 1) / b; }

struct Lookup {
  GroupArgs g;
  RegroupArgs r;
  TestArgs t;
  ReturnSlotsArgs slots;
  ReturnArgs keys;
  uint32_t* direct;
  bool two;
  uint64_t chunks;
  uint64_t steps2;  // second-pass steps at most
  uint64_t total;   // workspace bytes
};

// Blocks per test chunk, as a shift.
uint32_t chunk_shift(const bf_filter* f, bool two) {
  const uint64_t block = static_cast<uint64_t>(f->s) * f->word_bits / 8;
  uint32_t shift = 0;
  while ((block << (shift + 1)) <= static_cast<uint64_t>(test_chunk_bytes(two)) && shift < 16) ++shift;
  return shift;
}

// Records of a run that its reader sees: five standard deviations over the
// mean of uniformly hashed keys, of which a digit of `blocks` blocks among
// `of` gets its share of a step.
uint32_t run_clip(uint64_t blocks, uint64_t of) {
  const double mean = static_cast<double>(kStep) * static_cast<double>(blocks) / static_cast<double>(of);
  return static_cast<uint32_t>(mean + 5.0 * std::sqrt(mean) + 8.0);
}

// Geometry and workspace of one pass of n keys (n <= kMaxPass): sets the
// sizes of `x` and, given a base, the addresses.
void layout(const bf_filter* f, uint64_t n, uint8_t* base, Lookup& x) {
  const uint64_t steps = ceil_div(n, kStep);
  const uint32_t shift = chunk_shift(f, x.two);
  x.chunks = ceil_div(f->num_blocks, 1ull << shift);
  uint32_t low = 0;
  if (x.two)
    while ((1ull << (2 * low)) < x.chunks) ++low;
  x.g.n = n;
  x.g.steps = static_cast<uint32_t>(steps);
  x.g.wg_steps = static_cast<uint32_t>(std::max<uint64_t>(ceil_div(steps, 1024), 1));
  x.g.shift = shift + low;
  x.g.local_mask = (1u << shift) - 1;
  x.g.digits = static_cast<uint32_t>(ceil_div(x.chunks, 1ull << low));
  x.g.stride = ceil_div(steps, 16) * 16;
  const uint64_t digit = 1ull << x.g.shift;  // blocks of a first digit (the last one has the rest)
  x.g.clip = run_clip(std::min(digit, f->num_blocks), f->num_blocks);
  uint64_t off = 0;
  auto take = [&off, base](uint64_t bytes) {
    uint8_t* p = base + off;
    off = align256(off + bytes);
    return p;
  };
  uint32_t* direct = reinterpret_cast<uint32_t*>(take(4));
  x.g.direct = x.r.direct = x.t.direct = x.slots.direct = x.keys.direct = x.direct = direct;
  x.g.place = reinterpret_cast<uint16_t*>(take(2 * steps * kStep));
  x.g.table = reinterpret_cast<uint32_t*>(take(4 * x.g.digits * x.g.stride));
  x.keys.place = x.g.place;
  x.keys.n = n;
  uint64_t slots = steps * kStep;
  if (x.two) {
    x.r.shift = shift;
    x.r.digits = 1u << low;
    const uint64_t last = f->num_blocks - (x.g.digits - 1) * digit;
    x.r.clip = run_clip(1, x.r.digits);
    x.r.clip_last = run_clip(std::min<uint64_t>(1ull << shift, last), last);
    const uint64_t per_bucket = ceil_div(n, x.g.digits);
    x.r.per_digit = static_cast<uint32_t>(std::max<uint64_t>(
        std::max(ceil_div(per_bucket, 65536), std::min<uint64_t>(ceil_div(512, x.g.digits), per_bucket / kStep)), 1));
    x.r.item_steps = static_cast<uint32_t>(ceil_div(steps, x.r.per_digit));
    x.r.steps1 = x.g.steps;
    x.r.stride1 = x.g.stride;
    x.r.items = x.g.digits * x.r.per_digit;
    // as for a partitioned add: a run of c records takes ceil(c / kUnit) units
    const uint64_t units = n / kUnit + std::min(steps * x.g.digits, n);
    x.steps2 = units / kStepUnits + static_cast<uint64_t>(x.r.items) * ceil_div(x.r.item_steps, kRegroupRuns);
    x.r.stride2 = ceil_div(x.steps2, 16) * 16;
    const uint64_t slots2 = x.steps2 * kStep;
    // the pairs are dead once regrouped: the results of both passes take their place
    x.g.rec = reinterpret_cast<uint64_t*>(take(std::max(8 * slots, align256(slots2) + slots)));
    uint8_t* res2 = reinterpret_cast<uint8_t*>(x.g.rec);
    uint8_t* res1 = res2 + align256(slots2);
    x.r.rec = x.g.rec;
    x.r.table1 = x.g.table;
    x.r.table2 = reinterpret_cast<uint32_t*>(take(4 * x.r.digits * x.r.stride2));
    x.r.item_count = reinterpret_cast<uint32_t*>(take(4 * x.r.items));
    x.r.slot0 = reinterpret_cast<uint32_t*>(take(4 * (x.r.items + 1)));
    x.r.place = reinterpret_cast<uint16_t*>(take(2 * slots2));
    x.r.units = reinterpret_cast<uint32_t*>(take(4 * x.steps2 * kStepUnits));
    x.r.lo = reinterpret_cast<uint32_t*>(take(4 * slots2));
    x.r.blk = reinterpret_cast<uint16_t*>(take(2 * slots2));
    x.t.table = x.r.table2;
    x.t.stride = x.r.stride2;
    x.t.lo = x.r.lo;
    x.t.blk = x.r.blk;
    x.t.slot0 = x.r.slot0;
    x.t.per_digit = x.r.per_digit;
    x.t.low_bits = low;
    x.t.res = res2;
    x.slots.place = x.r.place;
    x.slots.res = res2;
    x.slots.out = res1;
    x.slots.units = x.r.units;
    x.slots.nsteps = x.r.slot0 + x.r.items;
    x.keys.res = res1;
  } else {
    x.g.lo = reinterpret_cast<uint32_t*>(take(4 * slots));
    x.g.blk = reinterpret_cast<uint16_t*>(take(2 * slots));
    x.t.table = x.g.table;
    x.t.stride = x.g.stride;
    x.t.lo = x.g.lo;
    x.t.blk = x.g.blk;
    x.t.steps = x.g.steps;
    x.t.res = take(slots);
    x.keys.res = x.t.res;
  }
  // few chunks: each over several workgroups (at least 8 Ki records each)
  const uint64_t fill = x.two ? 512 : 256;
  x.t.split = static_cast<uint32_t>(
      std::clamp<uint64_t>(std::min(ceil_div(fill, x.chunks), n / x.chunks / 8192), 1, 256));
  x.total = off;
}

constexpr uint64_t kMaxPass = 1ull << 28;

}  // namespace

namespace {

// Costs of a lookup: grouped fixed_us + n * grouped_ps, direct n * direct_ps
// where no key repeats; repeats add kRepeatPs to the grouped form (keys beyond
// their runs' clip; 2^26 keys, 10 to 50 % of them one key: 2.2..2.4 at 16 MiB,
// 3.2..3.7 at 32 MiB, 1.8..2 from 128 MiB on) and take the direct one down to
// kCachedPs for theirs.
//
// Fitted to both forms of 21 layouts (s, S, k) at 14 sizes of 8 MiB..2,000 MiB
// and 2^22.5..2^27 keys on MI355X.  The test costs by the bits per key, the
// block and a k that is not compiled in; with one digit it runs in rounds of
// 256 workgroups, the last of which may be short.  Measured slopes, ps per key:
// 16 MiB 8 x 32 bits k = 8 5.8 and k = 9 8.8, 4 x 64 k = 16 7.0, 16 x 64 8.0;
// 24 MiB (384 workgroups) 6.7, 10.8, 8.2, 9.6; 160 MiB 10.0, 12.9, 10.8, 11.6.
// Direct: 10.2 at 8 MiB, 14.2 at 16, 16.4 at 32, 18.2 at 64, 19 up to 1 GiB, 21
// at 2; 21.5 with 20 bits in blocks of 128 bytes.
struct LookupCost {
  double fixed_us, grouped_ps, direct_ps;
};
LookupCost lookup_cost(const bf_filter* f) {
  const double mib = static_cast<double>(f->nbytes) / (1 << 20);
  const double block = static_cast<double>(f->s) * f->word_bits / 8;
  const bool generic = k_index(f->k) == 0;
  if (f->nbytes > (64ull << 20)) {
    const double beyond = std::max(mib / 1024.0 - 1.0, 0.0);  // GiB
    LookupCost c{65.0 + 0.23 * mib, 9.5 + 0.04 * f->k + 0.012 * block + 0.7 * beyond,
                 18.2 + std::min(0.8, (mib - 64.0) / 200.0) + 2.3 * beyond};
    if (generic) {
      c.fixed_us += 0.08 * mib;
      c.grouped_ps += 2.3;
      if (mib > 768.0 && block >= 32.0) c.direct_ps += 1.7;
    } else if (block > 64.0) {
      c.fixed_us += 0.14 * mib;
    }
    return c;
  }
  const double l = std::log2(mib);  // 3 .. 6
  const double test = 5.0 + 0.07 * f->k + 0.013 * block + (generic ? 2.1 : 0.0);
  const uint64_t chunks = ceil_div(f->num_blocks, 1ull << chunk_shift(f, false));
  const uint64_t groups = chunks * ceil_div(256, chunks);
  const double rounds = static_cast<double>(ceil_div(groups, 256)) * 256.0 / static_cast<double>(groups);
  LookupCost c{43.0, test + (test - 3.8) * (rounds - 1.0) + std::max(0.0, mib - 32.0) / 32.0,
               l < 4.0 ? 10.2 + 4.0 * (l - 3.0) : l < 5.0 ? 14.2 + 2.2 * (l - 4.0) : 16.4 + 1.8 * (l - 5.0)};
  if (generic) c.direct_ps = std::max(c.direct_ps, block > 64.0 ? 21.5 : block > 32.0 ? 13.3 : 10.9);
  return c;
}
constexpr double kRepeatPs[2] = {3.5, 2.5};  // one digit, two
constexpr double kCachedPs = 2.6;
// The share of the keys that the caches serve is that of the sample's repeats
// where one key repeats, and more where the keys are skewed, for most of them
// are seen once in the sample.  Break-even shares of repeats, one key / skewed:
// 16 MiB 2^26 keys 0.40 / 0.26, 32 MiB 0.41 / 0.25, 64 MiB 0.51 / 0.28, 128 MiB
// 0.40 / 0.20, 512 MiB 0.36 / 0.18.  With 0.75 (limits 0.26..0.38 and 0.16..0.22)
// no lookup of 130 measured ones is grouped that takes 15 % more than directly
// before the sample came; those that go directly take 3..10 % more with 2^26 keys
// and, for the sample and the launches, up to 23 % with 2^24 (128 MiB 131 -> 161 us).
constexpr double kSeen = 0.75;

}  // namespace

// Whether a lookup of n keys is grouped: where it pays for keys that do not
// repeat by more than the sample and the launches without work cost keys that
// do.  One digit (up to 64 MiB), us direct / grouped: 8 MiB 2^24 keys 167 /
// 135; 16 MiB 2^22 63 / 60, 2^23 120 / 92; 32 MiB 2^22 73 / 62, 2^22.5 101 /
// 75; 64 MiB 2^22.5 112 / 86 (at 4 MiB most lines come from the L2: never).
// Two digits: 128 MiB 2^24 319 / 262, 256 MiB 2^24 327 / 299; 1 GiB 2^25 634 /
// 632 and 2^26 1275 / 982.  Keys that all repeat take 12..18 us more than
// directly: 16 MiB 2^23 30 / 43, 2^25 102 / 99.
bool lookup_groups(const bf_filter* f, uint64_t n) {
  if (f->layout != BF_LAYOUT_SECTORIZED || f->nbytes < (8ull << 20) || f->nbytes > (2ull << 30)) return false;
  const uint64_t least = f->nbytes < (16ull << 20)    ? 1ull << 24
                         : f->nbytes < (32ull << 20)  ? 3ull << 21
                         : f->nbytes <= (64ull << 20) ? 5ull << 20
                                                      : (1ull << 23) + f->nbytes / 36;
  if (n < least) return false;
  // ... and where the costs of the layout give the grouped form 3 %, the
  // error of the fit
  const LookupCost c = lookup_cost(f);
  const double keys = static_cast<double>(n) * 1e-6;
  return c.direct_ps * keys > 1.03 * (c.fixed_us + c.grouped_ps * keys);
}

namespace {

// The repeats in a sample from which on the direct lookup of a pass of n keys
// is the faster: 0, always, for a last pass that would not be grouped alone.
uint32_t sample_limit(const bf_filter* f, uint64_t n) {
  if (!lookup_groups(f, n)) return 0;
  const LookupCost c = lookup_cost(f);
  const double keys = static_cast<double>(n) * 1e-6;
  const double grouped = c.fixed_us + (c.grouped_ps + kRepeatPs[f->nbytes > (64ull << 20)]) * keys;
  const double share = (c.direct_ps * keys - grouped) / ((c.direct_ps - kCachedPs) * keys);
  return kSampleChance + static_cast<uint32_t>(std::max(kSeen * share, 0.02) * kSampleKeys);
}

}  // namespace

// The line for lookups in LDS, each side measured on MI355X with 32-byte
// blocks and k = 8 (us, direct against LDS): 2^20 keys 7.4 against 7.0..7.6 at
// every size; 2^21 keys 8.2 against 7.8 in 4 KiB, 9.4 against 9.0 in 16 KiB,
// 10.7 against 9.7 in 64 KiB, 11.5 against 9.7 in 128 KiB; 2^22 keys 14.8
// against 13.9, 15.4 against 15.2, 18.3 against 15.2, 19.7 against 16.0; 2^26
// keys 243 against 207, 222 against 178, 277 against 174, 293 against 205.
// 4-byte blocks lose 0.3 us at 2^21 keys in 16 KiB, hence the two lines.
// A k that is not compiled in loses 0.9 us of 18 at 2^21 keys in 160 KiB.
bool lookup_fits_lds(const bf_filter* f, uint64_t n) {
  const bool small = f->nbytes <= (16u << 10) || (f->nbytes > kResidentBytes[0] && k_index(f->k) == 0);
  return f->layout == BF_LAYOUT_SECTORIZED && f->nbytes <= kResidentBytes[1] && n >= (small ? 1ull << 22 : 1ull << 21);
}

// Adds in LDS: a workgroup merges its image into the filter, which pays from
// 8 keys per byte on.  us against the direct adds, 32-byte blocks, k = 8:
// 4 KiB 2^15 keys 17.7 against 11.7, 2^20 299 against 16; 16 KiB 2^17 18.4
// against 12.4; 64 KiB 2^18 18.7 against 17.6, 2^19 28.5 against 20.6; 128 KiB
// 2^19 28.8 against 28.8, 2^20 48 against 34, 2^22 90 against 78; 2^24 keys,
// which were partitioned, 161..193 against 58..125.  8-byte words and k = 16
// lose at 4 keys per byte (64 KiB 2^18 19.8 against 23.8), not at 8.
bool add_fits_lds(const bf_filter* f, uint64_t n) {
  return f->layout == BF_LAYOUT_SECTORIZED && f->nbytes <= kResidentBytes[1] && n >= 8 * f->nbytes;
}

bool resident_runs(const bf_filter* f, int op) {
  const int idx = batch_index(op, static_cast<int>(f->word_bits), static_cast<int>(f->s), k_index(f->k));
  return kernel_table(f->salts == kSaltsParquet).resident_fn[f->nbytes > kResidentBytes[0]][idx] != nullptr;
}

bf_status resident_call(const bf_filter* f, int op, const uint64_t* keys, uint64_t n, uint8_t* out,
                        hipStream_t stream, CallMark* mark, bool* taken) {
  *taken = false;
  const int big = f->nbytes > kResidentBytes[0];
  const int idx = batch_index(op, static_cast<int>(f->word_bits), static_cast<int>(f->s), k_index(f->k));
  const void* fn = kernel_table(f->salts == kSaltsParquet).resident_fn[big][idx];
  if (fn == nullptr) return BF_OK;
  ResidentArgs a{};
  a.f.words = f->d_words;
  a.f.hash_init = xxh64_u64_init(f->seed);
  a.f.nb_lo = static_cast<uint32_t>(f->num_blocks);
  a.f.keys = keys;
  a.f.out = out;
  a.n = n;
  a.k = f->k;
  // whole turns of the workgroups that 256 CUs hold
  const uint64_t slots = big ? 256 : 512;
  const uint64_t turns = ceil_div(n, slots * kResidentKeys);
  a.per = static_cast<uint32_t>(ceil_div(ceil_div(n, slots * turns), 2048ull) * 2048);  // of whole loop turns
  // an add's workgroup has a key for every 8 bytes that it merges, at least
  if (op == kOpAdd) a.per = std::max(a.per, static_cast<uint32_t>(ceil_div(f->nbytes / 8, 2048ull) * 2048));
  const uint64_t grid = ceil_div(n, static_cast<uint64_t>(a.per));
  if (grid > 0x7fffffffu) return BF_OK;
  void* kargs[] = {&a};
  *taken = true;
  return launch_marked(fn, dim3(static_cast<uint32_t>(grid)), dim3(kResidentThreads), kargs, stream, mark) == hipSuccess
             ? BF_OK
             : BF_EDEVICE;
}

namespace {

struct LookupKernels {
  const void *group, *regroup, *test, *ret;
};

// The geometry of a pass of n keys and its kernels; false if there are none.
bool plan_lookup(const bf_filter* f, uint64_t n, Lookup& x, LookupKernels& k) {
  const int idx = batch_index(kOpContains, static_cast<int>(f->word_bits), static_cast<int>(f->s), k_index(f->k));
  x.two = ceil_div(f->num_blocks, 1ull << chunk_shift(f, false)) > static_cast<uint64_t>(kLookupDigits);
  layout(f, n, nullptr, x);
  const Registry& r = kernel_table(f->salts == kSaltsParquet);
  k = {group_keys_fn(x.g.digits, !x.two, false, true), x.two ? regroup_fn(x.r.digits, true, false) : nullptr,
       r.lookup_fn[x.two ? 1 : 0][idx], r.return_fn[idx]};
  return k.group != nullptr && k.test != nullptr && k.ret != nullptr && (!x.two || k.regroup != nullptr);
}

}  // namespace

uint64_t lookup_workspace_bytes(const bf_filter* f, uint64_t n) {
  Lookup x{};
  LookupKernels k;
  return plan_lookup(f, std::min(n, kMaxPass), x, k) ? x.total : 0;
}

bf_status grouped_lookup(const bf_filter* f, const uint64_t* keys, uint64_t n, uint8_t* out, hipStream_t stream,
                         bool* taken) {
  *taken = false;
  Lookup x{};
  LookupKernels k;
  const uint64_t pass = std::min(n, kMaxPass);
  if (!plan_lookup(f, pass, x, k)) return BF_OK;
  void* ws = workspace_alloc(f->device, x.total, stream);
  if (ws == nullptr) return BF_OK;  // the direct lookup needs none
  *taken = true;
  hipError_t e = hipSuccess;
  for (uint64_t at = 0; at < n && e == hipSuccess; at += pass) {
    layout(f, std::min(pass, n - at), static_cast<uint8_t*>(ws), x);
    x.g.keys = keys + at;
    x.g.hash_init = xxh64_u64_init(f->seed);
    x.g.nb_lo = static_cast<uint32_t>(f->num_blocks);
    x.g.nb_hi_mask = (f->num_blocks >> 32) ? 0xffffffffu : 0u;
    x.t.words = f->d_words;
    x.t.nbytes = f->nbytes;
    x.t.k = f->k;
    x.keys.out = out + at;
    x.keys.words = f->d_words;
    x.keys.keys = x.g.keys;
    x.keys.hash_init = x.g.hash_init;
    x.keys.nb_lo = x.g.nb_lo;
    x.keys.nb_hi_mask = x.g.nb_hi_mask;
    x.keys.k = f->k;
    auto run = [&](const void* fn, uint64_t grid, int threads, void* arg) {
      void* args[] = {arg};
      if (e == hipSuccess) e = hipLaunchKernel(fn, dim3(static_cast<uint32_t>(grid)), dim3(threads), args, 0, stream);
    };
    uint64_t count = x.g.n;
    uint32_t limit = sample_limit(f, count);
    void* sargs[] = {&x.g.keys, &count, &x.g.hash_init, &limit, &x.direct};
    e = hipLaunchKernel(reinterpret_cast<const void*>(&sample_kernel), dim3(1), dim3(kSampleThreads), sargs, 0, stream);
    run(k.group, ceil_div(x.g.steps, x.g.wg_steps), kGroupThreads, &x.g);
    if (x.two) {
      run(regroup_plan_fn(false), x.r.items, kPlanThreads, &x.r);
      run(regroup_scan_fn(), 1, kScanThreads, &x.r);
      run(k.regroup, x.r.items, kGroupThreads, &x.r);
    }
    run(k.test, x.chunks * x.t.split, kTestThreads, &x.t);
    if (x.two) run(reinterpret_cast<const void*>(&return_slots_kernel), x.steps2, kReturnThreads, &x.slots);
    run(k.ret, x.g.steps, kReturnThreads, &x.keys);
  }
  if (hipFreeAsync(ws, stream) != hipSuccess && e == hipSuccess) e = hipErrorUnknown;
  return e == hipSuccess ? BF_OK : BF_EDEVICE;
}

}  // namespace bfhip
