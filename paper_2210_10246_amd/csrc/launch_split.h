// Host arithmetic of launches that have to be split (no HIP in here).
#pragma once

#include <stdint.h>

namespace tempo {

// Most workgroups of `threads` lanes in one launch: HIP refuses 2^32 lanes and more.
constexpr int64_t most_groups(int64_t wanted, int threads) {
  const int64_t fits = static_cast<int64_t>(UINT32_MAX) / threads;
  return wanted < fits ? wanted : fits;
}

}  // namespace tempo
