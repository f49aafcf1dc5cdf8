// Prints most_groups(wanted, threads) for pairs of arguments.
#include <cstdio>
#include <cstdlib>

#include "../paper_2210_10246_amd/csrc/launch_split.h"

int main(int argc, char** argv) {
  for (int i = 1; i + 1 < argc; i += 2)
    std::printf("%lld\n", static_cast<long long>(tempo::most_groups(std::atoll(argv[i]), std::atoi(argv[i + 1]))));
}
