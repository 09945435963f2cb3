// Exercises the host rules of csrc/launch_rules.h over their whole range; exits non-zero with a message at
// the first value that breaks a bound.
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "../../paper_2010_09410_amd/csrc/launch_rules.h"

static void check(bool ok, const char* what, unsigned long long a, unsigned long long b) {
  if (ok) return;
  std::printf("%s (%llu, %llu)\n", what, a, b);
  std::exit(1);
}

int main() {
  // every address width of a ROM (0 .. 32) and a RAM (1 .. 16): at least one read at a time, never more than
  // asked for, the selectors within 2^14 unless one read alone has more
  for (uint32_t v = 0; v <= 32; v++)
    for (uint64_t R : {1ull, 2ull, 3ull, 511ull, 512ull, 513ull, 16383ull, 16384ull, 16385ull, 1ull << 22}) {
      const uint64_t n = vsp::read_chunk(R, v);
      check(n >= 1 && n <= R, "reads outside [1, R]", R, v);
      check(n * v <= 1ull << 14 || n == 1, "selectors above 2^14", R, v);
      check(n == R || (n + 1) * (v ? v : 1) > 1ull << 14, "fewer reads than fit", R, v);
    }
  return 0;
}
