"""The progress words of fm_generate (commits on the device -> host loop), over more commits than their count has values."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
#include "fm_progress.h"
int main() {
  const unsigned calls[] = {1, 2, 4094, 4095};
  unsigned long long w = 0;                          // the word as it was before the first call
  for (unsigned call : calls) {
    unsigned n = progress_start(call);               // on the device
    long done = 0, commits = 0;                      // host; truth
    if (progress_call(w) == call) return printf("a word of an earlier call passes for one of call %u\n", call), 1;
    const long total = (5l << 19) + 3;               // two and a half times round
    unsigned lcg = call;
    while (commits < total) {
      const int steps = 1 + (lcg = lcg * 1664525u + 1013904223u) % 7;      // enqueued, and finished, since the host looked
      for (int i = 0; i < steps; i++) { n = progress_next(n); commits++; w = progress_word(n, 2u + (unsigned)commits); }
      if (progress_call(w) != call) return printf("call %u reads as %u after %ld commits\n", call, progress_call(w), commits), 1;
      done += progress_ahead(w, done);
      if (done != commits) return printf("call %u: %ld commits read as %ld\n", call, commits, done), 1;
      if (progress_ahead(w, done) != 0 || progress_state(w) != 2u + (unsigned)commits) return printf("state\n"), 1;
    }
  }
  return 0;
}
"""


def test_counts_past_the_width_of_the_word(tmp_path):
    src, exe = tmp_path / "driver.cc", tmp_path / "driver"
    src.write_text(DRIVER)
    inc = os.path.join(ROOT, "paper_2511_15618_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", inc, str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout
