// skim_sort.h -- which of rocPRIM's sorts the radix sorts by a few key bits take.
//
// By default rocPRIM merges up to 2^20 keys: a block sort, then two launches
// per doubling.  Keys that differ in 10 to 24 bits are sorted in two or three
// radix passes instead, from kRadixKeys keys on.  317 thousand in-edges by
// head (15 bits): 18 kernels of 110 us in all against 4 of 55 us, and a build
// of 20,000 nodes 1.59 to 1.51 ms; of 1000 nodes (its records) 0.58 to 0.53.
#pragma once

#include <rocprim/device/device_radix_sort.hpp>

namespace skim {

constexpr size_t kRadixKeys = 1u << 15;
using FewBits = rocprim::radix_sort_config<rocprim::default_config, rocprim::default_config,
                                           rocprim::default_config, kRadixKeys>;

}  // namespace skim
