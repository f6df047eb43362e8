// Kernel variants of the Parquet split-block filter (bf_parquet.h): every
// mapping of the sectorized 8 x 32-bit, k = 8 layout, in the same registry
// slots, the persistent batched kernels, and the apply
// kernels of the partitioned construction.
#include <utility>

#include "bf_parquet.hpp"
#include "bf_registry.hpp"

namespace bfhip {
namespace {

constexpr int kIdxK = k_index(kParquetK);

template <int THETA, int PHI, int KT>
void register_one(Registry& r) {
  if constexpr (THETA * PHI <= kParquetWords) {
    r.fn[registry_index(kOpContains, 32, kParquetWords, kIdxK, THETA, PHI, KT, 0)] =
        reinterpret_cast<const void*>(&parquet_contains_kernel<THETA, PHI, KT>);
    r.fn[registry_index(kOpAdd, 32, kParquetWords, kIdxK, THETA, PHI, KT, 0)] =
        reinterpret_cast<const void*>(&parquet_add_kernel<THETA, PHI, KT, false>);
    if constexpr (PHI >= 2)
      r.fn[registry_index(kOpAdd, 32, kParquetWords, kIdxK, THETA, PHI, KT, 1)] =
          reinterpret_cast<const void*>(&parquet_add_kernel<THETA, PHI, KT, true>);
  }
}

template <int THETA, int PHI>
void register_kt(Registry& r) {
  register_one<THETA, PHI, 1>(r);
  register_one<THETA, PHI, 2>(r);
  register_one<THETA, PHI, 4>(r);
}

template <int THETA>
void register_phi(Registry& r) {
  register_kt<THETA, 1>(r);
  register_kt<THETA, 2>(r);
  register_kt<THETA, 4>(r);
  register_kt<THETA, 8>(r);
}

}  // namespace

void register_parquet(Registry& r) {
  register_phi<1>(r);
  register_phi<2>(r);
  register_phi<4>(r);
  register_phi<8>(r);
  r.batch_fn[batch_index(kOpAdd, 32, kParquetWords, kIdxK)] =
      reinterpret_cast<const void*>(&parquet_batch_kernel<kOpAdd>);
  r.batch_fn[batch_index(kOpContains, 32, kParquetWords, kIdxK)] =
      reinterpret_cast<const void*>(&parquet_batch_kernel<kOpContains>);
  const int slot = batch_index(kOpAdd, 32, kParquetWords, kIdxK);
  r.apply_fn[0][slot] =
      reinterpret_cast<const void*>(&part_apply_kernel<uint32_t, kParquetWords, kParquetK, kZParquet, 16>);
  r.apply_fn[1][slot] =
      reinterpret_cast<const void*>(&part_apply_kernel<uint32_t, kParquetWords, kParquetK, kZParquet, 8>);
  const int look = batch_index(kOpContains, 32, kParquetWords, kIdxK);
  r.resident_fn[0][slot] = reinterpret_cast<const void*>(&parquet_resident_add_kernel<0>);
  r.resident_fn[1][slot] = reinterpret_cast<const void*>(&parquet_resident_add_kernel<1>);
  r.resident_fn[0][look] = reinterpret_cast<const void*>(&parquet_resident_kernel<0>);
  r.resident_fn[1][look] = reinterpret_cast<const void*>(&parquet_resident_kernel<1>);
  r.lookup_fn[0][look] = reinterpret_cast<const void*>(&parquet_lookup_test_kernel<false>);
  r.lookup_fn[1][look] = reinterpret_cast<const void*>(&parquet_lookup_test_kernel<true>);
  r.return_fn[look] = reinterpret_cast<const void*>(&parquet_lookup_return_kernel);
}

}  // namespace bfhip
