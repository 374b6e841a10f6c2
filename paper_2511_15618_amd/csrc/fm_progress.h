// What fm_generate and the commits on the device tell each other: one 64-bit word per sequence, so that count and state travel
// together and nothing has to be ordered.
//   upper half: number of the fm_generate call (12 bits), commits since its start modulo 2^20
//   lower half: 0 = the single-launch verify kernel gave up, 1 = sequence finished, else committed length + 2
// The host is at most a few steps behind, so it needs the count only modulo 2^20; a mesh may take more commits than that, and the
// count must then not carry into the number of the call.
#pragma once

#define FM_COMMIT_MASK 0xFFFFFu

constexpr unsigned progress_start(unsigned call) { return call << 20; }
constexpr unsigned progress_next(unsigned n) { return (n & ~FM_COMMIT_MASK) | ((n + 1) & FM_COMMIT_MASK); }
constexpr unsigned long long progress_word(unsigned n, unsigned state) { return (unsigned long long)n << 32 | state; }
constexpr unsigned progress_call(unsigned long long w) { return (unsigned)(w >> 52); }
constexpr unsigned progress_state(unsigned long long w) { return (unsigned)w; }
// commits of a word of this call beyond `done` of them
constexpr unsigned progress_ahead(unsigned long long w, long done) { return ((unsigned)(w >> 32) - (unsigned)done) & FM_COMMIT_MASK; }
