// Radix sort of key / value pairs for the device set-up stages.
#pragma once

#include <hip/hip_runtime.h>
#include <rocprim/rocprim.hpp>

#include <cstdint>

namespace vbcsr {

// The library's default sorts fewer than 2^20 pairs by merging: a launch and a
// pass over the data per doubling, whatever the number of key bits.  From 2^18
// pairs on one pass per 8 key bits is faster (the three sorts of 775,000 block
// product pairs with 3 and 20 bits: 5.04 ms -> 4.83 ms of the whole product;
// 519,000 pairs 2.61 -> 2.47; 134,000 pairs 1.58 -> 1.63 and left to merging).
// Stable; keys of bits 0 .. end_bit - 1.
template <typename K, typename V>
hipError_t sort_pairs(void *tmp, size_t &bytes, const K *key, K *key_sorted, const V *val,
                      V *val_sorted, int64_t count, unsigned int end_bit, hipStream_t s) {
  using Config = rocprim::radix_sort_config<rocprim::default_config, rocprim::default_config,
                                            rocprim::default_config, 1 << 18>;
  return rocprim::radix_sort_pairs<Config>(tmp, bytes, key, key_sorted, val, val_sorted,
                                           (size_t)count, 0u, end_bit, s);
}

}  // namespace vbcsr
