"""Which attention launches load their keys and values as read once: the rule of the launch code, taken from the source and compiled for the host."""
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_15618_amd", "csrc")

MAIN = r"""
#include <cstdio>
struct Set { const void* Kc; int capb; };
%s
int main() {
  char a, b, c;
  auto blocks = [](int keys) { return (keys + 31) / 32; };
  // eight sequences of d = 1024: a memory of 128 rows and a cache of 4500 positions, then the other way round
  const Set small_memory[] = {{&a, blocks(128)}}, long_cache[] = {{&a, blocks(4500)}}, large_memory[] = {{&a, blocks(4096)}}, short_cache[] = {{&a, blocks(120)}};
  printf("%%d %%d %%d %%d\n", attn_once(small_memory, 1, 8, 16, 64), attn_once(long_cache, 1, 8, 16, 64), attn_once(large_memory, 1, 8, 16, 64), attn_once(short_cache, 1, 8, 16, 64));
  // one sequence: two sets over one cache of 3.1 MB, three caches of 3.1 MB
  const Set one[] = {{&a, blocks(768)}, {&a, blocks(768)}}, three[] = {{&a, blocks(768)}, {&b, blocks(768)}, {&c, blocks(768)}};
  printf("%%d %%d\n", attn_once(one, 2, 1, 16, 64), attn_once(three, 3, 1, 16, 64));
}
"""


def test_a_launch_is_judged_by_its_own_caches(tmp_path):
    src = open(os.path.join(CSRC, "fm_kernels_decode.h")).read()
    rule = re.search(r"^template <class SET>\nbool attn_once\(.*?^}\n", src, re.S | re.M)
    assert rule, "the rule does not look at the launch's sets"
    assert "attn_once(" not in open(os.path.join(CSRC, "flashmesh.hip")).read()
    main, exe = tmp_path / "once.cc", tmp_path / "once"
    main.write_text(MAIN % rule.group(0))
    subprocess.run(["g++", "-std=c++17", "-O1", str(main), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split() == ["0", "1", "1", "0", "0", "1"]
