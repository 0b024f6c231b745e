#pragma once

#include <algorithm>
#include <cstdint>

namespace fdc {

// HIP counts the threads of a dimension in 32 bits: of a larger launch it runs the rest of the
// division by 2^32, without an error (of 2^32 itself it reports one).
constexpr bool launch_counts(std::uint32_t grid, std::uint32_t block) {
  return (std::uint64_t)grid * block < (1ull << 32);
}

// `total` workgroups of `threads` threads in launches that HIP can count; launch(workgroups,
// index of the first one).  `total` is below 2^32.
template <class Err, class F>
Err in_launches(long long total, int threads, Err none, F &&launch) {
  const long long most = ((1LL << 32) - 1) / threads;
  Err err = none;
  for (long long i = 0; i < total && err == none; i += most)
    err = launch((std::uint32_t)std::min(most, total - i), (std::uint32_t)i);
  return err;
}

}  // namespace fdc
