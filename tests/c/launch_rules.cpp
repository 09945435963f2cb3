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
  // every count of key copies (92.9 MB each), at free memories around each count's line: taken when 61.9 MB for every
  // copy and 1 GiB are free; then at least one, no more than asked for or held, within what is left when up to
  // 1 GiB of scratch has been taken, and all of them where they fit
  const uint64_t asked = 61931520, key = 92897280, GiB = 1ull << 30;
  check(vsp::key_copies_accepted(1, GiB) && !vsp::key_copies_accepted(1, GiB - 1), "one copy", 1, GiB);
  for (uint64_t held : {256ull, 2048ull})
    for (uint64_t copies = 2; copies <= 65536; copies++)
      for (int64_t off : {-1, 0, 1}) {
        const uint64_t line = copies * asked + GiB, free_b = line + off;
        check(vsp::key_copies_accepted(copies, free_b) == (off >= 0), "accepted", copies, free_b);
        if (off < 0) continue;
        for (uint64_t left : {free_b, free_b - GiB, (uint64_t)288 << 30}) {
          const uint64_t n = vsp::key_copies_made(copies, held, left, key);
          check(n >= 1 && n <= copies && n <= held, "copies outside [1, min(copies, held)]", copies, left);
          check(n * key <= left, "copies beyond the memory left", copies, left);
          if ((copies < held ? copies : held) * key + (64ull << 20) <= left)
            check(n == (copies < held ? copies : held), "fewer copies than fit", copies, left);
        }
      }
  return 0;
}
