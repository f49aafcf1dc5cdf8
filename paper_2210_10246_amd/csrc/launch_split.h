// Host arithmetic of launches that have to be split (no HIP in here).
#pragma once

#include <stdint.h>

namespace tempo {

// Most workgroups of `threads` lanes in one launch: HIP refuses 2^32 lanes and more.
constexpr int64_t most_groups(int64_t wanted, int threads) {
  const int64_t fits = static_cast<int64_t>(UINT32_MAX) / threads;
  return wanted < fits ? wanted : fits;
}

// Covers `total` workgroups by launches of at most `cap`: launch(first, count) -> whether it was taken.
// Ends at the first that was not: one taken later must not hide that workgroups are missing.
template <typename F>
bool split_launch(int64_t total, int64_t cap, F&& launch) {
  for (int64_t first = 0; first < total; first += cap) {
    const int64_t left = total - first;
    if (!launch(static_cast<uint32_t>(first), static_cast<uint32_t>(left < cap ? left : cap))) return false;
  }
  return true;
}

}  // namespace tempo
