"""Stage profile of the single-launch verify kernel: a stage ends when its last wave is done, not when the first one is."""
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_15618_amd", "csrc")

# One workgroup of the kernel's stamps, its threads one after another: wave w is done at time 100 + 10 * (order of w).
DRIVER = r"""
#include <algorithm>
#include <cstdio>
typedef unsigned long long u64;
struct Dim { unsigned x; } threadIdx;
struct Args { u64* prof; int prof_stage; } a;
u64 now;
u64 wall_clock64() { return now; }
void atomicMax(u64* p, u64 v) { *p = std::max(*p, v); }
MACROS
int main() {
  for (int last = 0; last < 4; last++) {
    u64 prof[1024] = {};
    a = {prof, 7};
    for (unsigned t = 0; t < 256; t++) {
      threadIdx.x = t;
      now = 100 + 10 * (((t >> 6) + 3 - last) & 3);      // wave `last` comes last
      bool worked = true;
      unsigned rr = 0;
      int stage = 7;
      PK_MARK(3);
      PK_NEXT(5);
      if (worked || stage != 8 || rr != 5) return printf("state of thread %u\n", t), 1;
      PK_NEXT(5);                                         // a stage without a unit for this workgroup
    }
    if (prof[603] != 130 || prof[8] != 130 || prof[9] != 0)
      return printf("wave %d last: phase %llu, stage %llu, stage without work %llu\n", last, prof[603], prof[8], prof[9]), 1;
  }
  return 0;
}
"""


def test_a_stage_ends_with_its_last_wave(tmp_path):
    src = open(os.path.join(CSRC, "fm_kernels_persist.h")).read()
    macros = [m.group(0) for m in re.finditer(r"^#define PK_(?:STAMP|MARK|NEXT)\b(?:.*\\\n)*.*$", src, flags=re.M)]
    assert len(macros) >= 2
    cc, exe = tmp_path / "driver.cc", tmp_path / "driver"
    cc.write_text(DRIVER.replace("MACROS", "\n".join(macros)))
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", str(cc), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout
