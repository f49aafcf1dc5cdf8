// With "split TOTAL CAP FAIL_AT": prints the launches (first, count) of split_launch, of which the one
// that starts at or behind FAIL_AT is refused, and what it returned.  Else: prints most_groups(wanted,
// threads) for pairs of arguments.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "../paper_2210_10246_amd/csrc/launch_split.h"

int main(int argc, char** argv) {
  if (argc == 5 && std::strcmp(argv[1], "split") == 0) {
    const long long fail_at = std::atoll(argv[4]);
    const bool ok = tempo::split_launch(std::atoll(argv[2]), std::atoll(argv[3]), [&](uint32_t first, uint32_t n) {
      std::printf("%u %u\n", first, n);
      return static_cast<long long>(first) < fail_at;
    });
    std::printf("%d\n", ok ? 1 : 0);
    return 0;
  }
  for (int i = 1; i + 1 < argc; i += 2)
    std::printf("%lld\n", static_cast<long long>(tempo::most_groups(std::atoll(argv[i]), std::atoi(argv[i + 1]))));
}
