"""The tags of the resident sub-cycle's exchange (csrc/lbmd_tag.h), on the
host: a value that a pass leaves in a slot is taken by no stage of another
pass or cycle."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <cstdio>
#include <set>
#include "lbmd_tag.h"
using namespace lbmd;
int main() {
  std::set<uint64_t> seen;
  long n = 0;
  const uint64_t cycles[] = {1, 2, 3, 1000, 1001, 0x7fffffffull, 0x80000000ull};
  for (uint64_t cycle : cycles)
    for (uint32_t pass = 0; pass < 2; ++pass)
      for (uint32_t s = 0; s < 300; ++s, ++n) {
        // what a reader of stage s takes: a word pair (x, x ^ tag)
        const uint64_t x = 0x3ff123456789abcdull, word[2] = {x, x ^ res_tag(cycle, pass, s)};
        for (uint64_t c2 : cycles)
          for (uint32_t p2 = 0; p2 < 2; ++p2)
            for (uint32_t s2 = s & 1; s2 < 300; s2 += 2)
              if (((word[0] ^ word[1]) == res_tag(c2, p2, s2)) != (c2 == cycle && p2 == pass && s2 == s)) {
                std::printf("cycle %llu pass %u stage %u taken for %llu %u %u\n", (unsigned long long)cycle, pass, s,
                            (unsigned long long)c2, p2, s2);
                return 1;
              }
        seen.insert(res_tag(cycle, pass, s));
      }
  std::printf("%ld tags\n", n);
  return (long)seen.size() == n ? 0 : 2;
}
"""


def test_no_stage_of_any_pass_takes_anothers_value(tmp_path):
    src, exe = tmp_path / "tags.cpp", tmp_path / "tags"
    src.write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-I" + os.path.join(ROOT, "paper_0711_2665_amd", "csrc"), "-o",
                           str(exe), str(src)])
    subprocess.check_call([str(exe)])
