// Host check of the automatic plans' launch rules (compiled with g++ by the test suite): one pass at
// N = 2^13 exactly where it measured faster, and the splits and row tiles on both sides of their lines.
#include <cstdio>

#include "launch_rules.hpp"

static int failures = 0;
static void check(bool ok, const char* what, unsigned long long n, bool fast) {
  if (!ok) {
    ++failures;
    std::printf("FAIL %s: %llu vectors, fast %d\n", what, n, (int)fast);
  }
}

int main() {
  struct Row { uint64_t n; bool below_60, above_60; };
  const Row one_pass[] = {{1, false, false},  {128, false, false}, {191, false, false}, {192, true, true},
                          {256, true, true},  {257, false, false}, {288, false, false}, {335, false, false},
                          {336, true, false}, {399, true, false},  {400, true, true},   {512, true, true},
                          {520, false, false}, {576, false, false}, {592, true, false}, {656, true, true},
                          {768, true, true},  {769, false, false}, {1024, true, true},  {1025, true, false},
                          {1300, true, false}, {2048, true, true}, {2100, true, false}, {1 << 20, true, true}};
  for (const Row& r : one_pass)
    for (bool fast : {true, false}) {
      const bool want = fast ? r.below_60 : r.above_60;
      check(nttr::one_pass_8192(r.n, fast) == want, "one pass at 2^13", r.n, fast);
      check(nttr::split(13, 5, r.n, fast) == (want ? 0u : 5u), "split at 2^13", r.n, fast);
      check(nttr::split(12, 0, r.n, fast) == 0 && nttr::split(14, 6, r.n, fast) == 6 && nttr::split(17, 8, r.n, fast) == 8,
            "sizes without a rule", r.n, fast);
    }
  for (bool fast : {true, false}) {
    check(nttr::split(15, 6, 64, fast) == 7 && nttr::split(15, 6, 65, fast) == 6, "2^15 at 2^21 residues", 64, fast);
    check(nttr::split(16, 6, 32, fast) == 7 && nttr::split(16, 6, 33, fast) == 6, "2^16 at 2^21 residues", 32, fast);
  }
  // row tiles: small launches of split sizes only
  check(nttr::small_rows(13, 5, 256) && !nttr::small_rows(13, 5, 257), "row tile at 2^21 residues", 256, true);
  check(nttr::small_rows(16, 4, 1) && !nttr::small_rows(17, 4, 1), "row tile of 2^12 and 2^13 points", 1, true);
  check(!nttr::small_rows(12, 0, 1) && !nttr::small_rows(13, 0, 1), "row tile of one pass", 1, true);
  std::printf("%d failures\n", failures);
  return failures != 0;
}
