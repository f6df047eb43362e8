// bf_group.hip -- the grouping kernels of the partitioned construction and
// the grouped lookup (bf_group.hpp); they depend on no layout.
#include <hip/hip_runtime.h>

#include "bf_group.hpp"

namespace bfhip {

namespace {

// The number of output steps of every item: its units, kStep / UNIT to a step,
// a batch of kRegroupRuns runs at a time.
template <int UNIT>
__global__ __launch_bounds__(kPlanThreads) void regroup_plan_kernel(RegroupArgs a) {
  __shared__ uint32_t wave_sum[kPlanThreads / 64];
  if (a.direct != nullptr && *a.direct != 0) return;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const PartItem it = regroup_item(a, blockIdx.x);
  const uint32_t* entries = a.table1 + it.d1 * a.stride1;
  uint32_t steps = 0;
  for (uint32_t base = it.t0; base < it.t1; base += kRegroupRuns) {
    uint32_t sum = 0;
    for (uint32_t i = tid; i < kRegroupRuns && base + i < it.t1; i += kPlanThreads)
      sum += (run_len(entries[base + i]) + UNIT - 1) / UNIT;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, 64);
    if (lane == 0) wave_sum[wave] = sum;
    __syncthreads();
    uint32_t total = 0;
#pragma unroll
    for (int w = 0; w < kPlanThreads / 64; ++w) total += wave_sum[w];
    steps += (total + kStep / UNIT - 1) / (kStep / UNIT);
    __syncthreads();
  }
  if (tid == 0) a.item_count[blockIdx.x] = steps;
}

// First output step of every item: prefix sums of the items' step counts.
__global__ __launch_bounds__(kScanThreads) void regroup_scan_kernel(RegroupArgs a) {
  __shared__ uint32_t wave_sum[kScanThreads / 64];
  if (a.direct != nullptr && *a.direct != 0) return;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  uint32_t before = 0;
  for (uint32_t base = 0; base < a.items; base += kScanThreads) {
    const uint32_t i = base + tid;
    const uint32_t c = i < a.items ? a.item_count[i] : 0u;
    uint32_t incl = c;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t v = __shfl_up(incl, off, 64);
      if (lane >= static_cast<uint32_t>(off)) incl += v;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    uint32_t mine = before;
#pragma unroll
    for (int w = 0; w < kScanThreads / 64; ++w) {
      const uint32_t s = wave_sum[w];
      if (static_cast<uint32_t>(w) < wave) mine += s;
      before += s;
    }
    if (i < a.items) a.slot0[i] = mine + incl - c;
    __syncthreads();
  }
  if (tid == 0) a.slot0[a.items] = before;
}

template <int D, int ROWS>
const void* keys_fn(bool split, bool multi) {
  if (multi) return split ? nullptr : reinterpret_cast<const void*>(&group_keys_kernel<D, ROWS, false, true, false>);
  return split ? reinterpret_cast<const void*>(&group_keys_kernel<D, ROWS, true, false, false>)
               : reinterpret_cast<const void*>(&group_keys_kernel<D, ROWS, false, false, false>);
}

// Lookups: split records of up to 512 digits (one pass), pairs of up to 128.
const void* place_fn(uint32_t digits, bool split) {
  if (!split)
    return digits <= 128 ? reinterpret_cast<const void*>(&group_keys_kernel<128, 16, false, false, true>) : nullptr;
  return digits <= 128   ? reinterpret_cast<const void*>(&group_keys_kernel<128, 16, true, false, true>)
         : digits <= 256 ? reinterpret_cast<const void*>(&group_keys_kernel<256, 16, true, false, true>)
         : digits <= 512 ? reinterpret_cast<const void*>(&group_keys_kernel<512, 16, true, false, true>)
                         : nullptr;
}

}  // namespace

const void* group_keys_fn(uint32_t digits, bool split, bool multi, bool place) {
  if (place) return place_fn(digits, split);
  if (digits <= 128) return keys_fn<128, 16>(split, multi);
  if (digits <= 256) return keys_fn<256, 16>(split, multi);
  if (digits <= 512) return keys_fn<512, 16>(split, multi);
  if (digits <= 1024) return keys_fn<1024, 8>(split, multi);
  return nullptr;
}

// Short units: a filter of 256 first digits or more (then 128 second digits
// or more).  Places: a lookup's second digits are at most 256.
const void* regroup_fn(uint32_t digits, bool place, bool short_units) {
  if (place)
    return digits <= 128   ? reinterpret_cast<const void*>(&regroup_kernel<128, 16, true, kUnit>)
           : digits <= 256 ? reinterpret_cast<const void*>(&regroup_kernel<256, 16, true, kUnit>)
                           : nullptr;
  if (short_units)
    return digits <= 256    ? reinterpret_cast<const void*>(&regroup_kernel<256, 16, false, kShortUnit>)
           : digits <= 512  ? reinterpret_cast<const void*>(&regroup_kernel<512, 8, false, kShortUnit>)
           : digits <= 1024 ? reinterpret_cast<const void*>(&regroup_kernel<1024, 8, false, kShortUnit>)
                            : nullptr;
  return digits <= 128   ? reinterpret_cast<const void*>(&regroup_kernel<128, 16, false, kUnit>)
         : digits <= 256 ? reinterpret_cast<const void*>(&regroup_kernel<256, 16, false, kUnit>)
         : digits <= 512 ? reinterpret_cast<const void*>(&regroup_kernel<512, 8, false, kUnit>)
                         : nullptr;
}

const void* regroup_plan_fn(bool short_units) {
  return short_units ? reinterpret_cast<const void*>(&regroup_plan_kernel<kShortUnit>)
                     : reinterpret_cast<const void*>(&regroup_plan_kernel<kUnit>);
}
const void* regroup_scan_fn() { return reinterpret_cast<const void*>(&regroup_scan_kernel); }

}  // namespace bfhip
