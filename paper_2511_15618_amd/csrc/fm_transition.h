// Which columns of a row (of at most 1024) thread t of 256 has in a level transition of the single-launch verify kernel, ascending:
// those it publishes, and those of the stack below that it waits for first.
#pragma once

#define FM_TR_COLS 4      // columns of a thread at most

struct PoolCols {         // shorten: pairs, published as two halves in one element
  static constexpr int col(int t, int i) { return (i >> 1) * 512 + 2 * t + (i & 1); }
  static constexpr int count(int d, int t) { return 2 * ((d - 2 * t + 511) / 512); }      // below d (even)
};
struct SkipCols {         // upsample: 16 lanes have 16 columns side by side
  static constexpr int col(int t, int i) { return i * 256 + t; }
  static constexpr int count(int d, int t) { return (d - t + 255) / 256; }
};
