// Prints what the dispatch rules of csrc/routes.h choose, one answer per line of standard input.
#include <cstdio>
#include <iostream>
#include <string>

#include "routes.h"

int main() {
  std::string rule;
  unsigned long long n, d, x;
  while (std::cin >> rule >> n >> d >> x) {
    if (rule == "xor128") {
      const prng::Cut c = prng::xor128_cut(n, d, x != 0);
      printf("%llu %llu\n", (unsigned long long)c.S, (unsigned long long)c.K);
    } else if (rule == "lux" || rule == "lux_f64" || rule == "lux_shared") {
      const prng::Cut c = prng::lux_cut(n, d, (uint32_t)x, rule == "lux_f64", rule == "lux_shared");
      printf("%llu %llu\n", (unsigned long long)c.S, (unsigned long long)c.K);
    } else if (rule == "mt19937") {
      printf("%d\n", (int)prng::mt_row_per_wave(n, d));
    } else if (rule == "ranmar") {
      printf("%d\n", (int)prng::ranmar_row_per_lane(n, d));
    } else if (rule == "ranmar_packed") {
      printf("%d\n", (int)prng::ranmar_packed_per_lane(n, d));
    } else if (rule == "ranmar_consumer") {
      printf("%d\n", (int)prng::ranmar_consumer_per_lane(n, d));
    } else if (rule == "leap_packed") {
      printf("%d\n", (int)prng::leap_packed_per_lane(x != 0, n, d));
    } else if (rule == "consumer") {  // x: the kind
      const double us[] = {0, prng::kGglDrawUs, prng::kXor128DrawUs, prng::kRanecuDrawUs, 0, 0, 0, prng::kDrand48DrawUs,
                           prng::kRannyuDrawUs};
      printf("%d\n", prng::consumer_width(us[x], x == 2, n, d));
    } else if (rule == "ranges") {
      prng::for_stream_ranges(n, d, [](uint64_t s0, uint64_t m) {
        printf("%llu %llu ", (unsigned long long)s0, (unsigned long long)m);
        return 0;
      });
      printf("\n");
    } else {
      return 1;
    }
  }
}
