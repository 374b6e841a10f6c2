"""What the single-launch verify kernel publishes into buffers that it uses again: a level transition proves that every tile of the stack below was waited
for, and no element of a partial tile is published that nobody waits for."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_15618_amd", "csrc")

# A wave goes on when all its lanes have what they wait for.  Who reads the published row needs all its columns, each from some
# wave; the tiles of 16 columns that the publishing waves have waited for must therefore be all of them, and every column published once.
DRIVER = r"""
#include <cstdio>
#include <vector>
#include "fm_transition.h"
template <class WAIT, class PUT>
int check(const char* what) {
  for (int d = 128; d <= 1024; d += 128) {
    std::vector<int> put(d), waited(d / 16);
    for (int wave = 0; wave < 4; wave++) {
      bool publishes = false;
      for (int t = wave * 64; t < wave * 64 + 64; t++)
        for (int k = 0; k < FM_TR_COLS; k++)
          if (PUT::col(t, k) < d) { put[PUT::col(t, k)]++; publishes = true; }
      for (int t = wave * 64; t < wave * 64 + 64; t++) {
        const int n = WAIT::count(d, t);
        if (n < 0 || n > FM_TR_COLS) return printf("%s, d = %d: thread %d has %d columns\n", what, d, t, n), 1;
        for (int k = 0; k < FM_TR_COLS; k++)
          if ((k < n) != (WAIT::col(t, k) < d)) return printf("%s, d = %d: column %d of thread %d\n", what, d, k, t), 1;
        for (int k = 0; publishes && k < n; k++) waited[WAIT::col(t, k) / 16] = 1;
      }
    }
    for (int c = 0; c < d; c++) if (put[c] != 1) return printf("%s, d = %d: column %d published %d times\n", what, d, c, put[c]), 1;
    for (int n = 0; n < d / 16; n++) if (!waited[n]) return printf("%s, d = %d: nobody who publishes waits for tile %d\n", what, d, n), 1;
  }
  return 0;
}
int main() { return check<WAIT_POOL, PoolCols>("shorten") | check<WAIT_SKIP, SkipCols>("upsample"); }
"""


def _run(tmp_path, wait_pool, wait_skip):
    src, exe = tmp_path / "driver.cc", tmp_path / "driver"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, f"-DWAIT_POOL={wait_pool}", f"-DWAIT_SKIP={wait_skip}",
                    str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)


def test_a_transition_waits_for_every_tile(tmp_path):
    """With the columns that the kernel's two units wait for and publish, as its source has them."""
    src = open(os.path.join(CSRC, "fm_kernels_persist.h")).read()
    units = re.findall(r"pk_wait_stack<FWT, (\w+)>\(a, a\.hT\[st\].*?const int i = (\w+)::col\(threadIdx\.x, k\)", src, flags=re.S)
    assert [put for _, put in units] == ["PoolCols", "SkipCols"]
    res = _run(tmp_path, units[0][0], units[1][0])
    assert res.returncode == 0, res.stdout


def test_columns_that_are_not_published_are_told_from_it(tmp_path):
    """A unit that pools pairs and waits for every 256th column leaves tiles out in narrow models."""
    res = _run(tmp_path, "SkipCols", "SkipCols")
    assert res.returncode != 0 and "shorten, d = 128: nobody who publishes waits for tile" in res.stdout


# The partial tiles of the FFN down projection are the same memory in every layer, and a later layer (behind an upsampling) may have more rows.  A store into
# them is known to have landed only if quarter 0 waited for its element before it published what the next layers read.
PARTIALS = r"""
#include <cstdio>
int main() {
  int waited = 0;
  for (int Rl = 1; Rl <= 16; Rl++)
    for (int tid = 0; tid < 256; tid++) {
      const int er = ((tid & 63) >> 4) * 4 + (tid >> 6);      // row of a thread in a tile
      const bool on = er < Rl;
      waited += WAIT;
      if (on && !(PUT)) return printf("row %d of %d is not published\n", er, Rl), 1;
      if ((PUT) && !(WAIT)) return printf("row %d of %d is published and not waited for\n", er, Rl), 1;
    }
  return waited != 16 * (16 * 17 / 2);
}
"""


def _run_partials(tmp_path, put, wait):
    src, exe = tmp_path / "partials.cc", tmp_path / "partials"
    src.write_text(PARTIALS)
    subprocess.run(["g++", "-std=c++17", "-O1", f"-DPUT={put}", f"-DWAIT={wait}", str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)


def test_no_partial_is_published_that_nobody_waits_for(tmp_path):
    """With the conditions that stand in front of the kernel's store and in its wait."""
    src = open(os.path.join(CSRC, "fm_kernels_persist.h")).read()
    assert "er = ((tid & 63) >> 4) * 4 + (tid >> 6)" in src and "const bool on = er < Rl;" in src
    put = re.findall(r"(if \(([^()]*)\) )?pk_stf\(w2p \+ ", src)
    wait = re.findall(r"pk_fetch<3>\(pr, 3, (\w+), tag, \[&\]\(int i\) \{ return w2p \+ i \* 256 \+ tid; \}", src)
    assert len(put) == 1 and len(wait) == 1
    res = _run_partials(tmp_path, put[0][1] or "true", wait[0])
    assert res.returncode == 0, res.stdout


def test_a_partial_of_a_row_that_does_not_exist_is_told(tmp_path):
    res = _run_partials(tmp_path, "true", "on")
    assert res.returncode != 0 and "row 4 of 1 is published and not waited for" in res.stdout
