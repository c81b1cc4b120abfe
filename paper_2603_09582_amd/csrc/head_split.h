// Single launch with 4-wave workgroups, two row blocks per head: which heads one workgroup takes whole, and which two
// workgroups take, one per row block (each after the whole prologue), so that the last round takes half of its block loops.
// Plain arithmetic, the same in the library and in a host program that checks it.
#pragma once

#if defined(__HIPCC__)
#define BINATTN_HD_SPLIT __host__ __device__ __attribute__((always_inline)) inline
#else
#define BINATTN_HD_SPLIT inline
#endif

namespace binattn {

// Workgroup v runs on chiplet v % 8, which holds 64 (96) workgroups at once where two (three) share a compute unit.  Whole
// heads and row blocks are both dealt out to the chiplets in equal shares, rounded up: a rule that counts workgroups over
// the whole chip gives a chiplet one too many where the number of heads is no multiple of 8, and a round more.
constexpr int SPLIT_XCDS = 8;

// Heads left for a last round of `slots` workgroups, 128 at most: as many row blocks as fit one compute unit each.  us per call,
// whole heads / split, rounds of 512, bf16 bias: N = 197, d = 64 520 heads 36.9 / 32.3, 640 36.3 / 31.9, 1152 54.6 / 51.0;
// N = 256, d = 72 640 heads 41.5 / 37.7; N = 200, d = 32 640 heads 24.6 / 20.2; fp32 bias, N = 256, d = 96 640 heads 65.7 / 61.1; no bias, d = 64
// 640 heads 29.8 / 28.2, 1152 44.6 / 42.8.  Above 128 the halves share compute units: 704 heads 37.1 / 36.3, without a bias
// 30.5 / 31.7, d = 32 25.0 / 25.9; 1280 heads 55.9 / 57.4.
constexpr int split_last(int heads, int slots) {
    const int left = heads % slots;
    return heads > slots && left > 0 && left <= 128 ? heads - left : heads;
}
// As many row blocks as fill the last round of 768.  With r rounds a chiplet holds 96 r workgroups: from / 8 whole heads and
// 2 (heads - from) / 8 row blocks, both rounded up.
constexpr int split_fill(int heads) {
    const int eighth = (heads + SPLIT_XCDS - 1) / SPLIT_XCDS, rounds = (eighth + 95) / 96;
    const int from = SPLIT_XCDS * (2 * eighth - 96 * rounds);
    return from < heads ? from : heads;
}
// Where three workgroups share a compute unit.  Rounds of 512 count there too: the heads above them go to units that are two thirds
// full.  us per call relative to the best of all four (mean over N = 129, 160, 197, 224, 225, 256, d = 16, 32, 40, 64, no bias and bf16; whole heads / split
// above 512 n / above 768 n / to fill the round):
//   513 heads 1.16 / 1.00 / - / 1.02    520 .. 640 1.13-1.15 / 1.00-1.01 / - / 1.00 (520 to 545, d = 64, no bias 0.95-0.98 of the first)    641 .. 767 1.00-1.01 / - / - / 1.00
//   769 .. 896 1.10-1.13 / - / 1.00-1.01 / -    900 .. 1024 1.00-1.02 / - / 1.01-1.04 / -    1025 .. 1152 1.07-1.10 / 1.00 / - / 1.06-1.08
//   1160 .. 1300 1.00 / - / - / 1.01-1.03   1310 .. 1380 1.06-1.08 / - / - / 1.00    1420 .. 1500 1.00-1.01 / - / - / 1.00   1540 .. 1660 1.05-1.08 / 1.00 / 1.00 / -
//   1670 .. 2048 1.00 / - / 1.01 / 1.01-1.03    2050 .. 2170 1.04-1.07 / 1.00 / - / 1.00-1.01   2180 .. 2290 1.00-1.01 / - / - / 1.00
// (Up to 48 channels without a bias four workgroups fit a unit.  Rounds of 1024 in place of 768 leave 776 to 1000 heads where they are, to
// 1 %, gain 5 % at 1800 and lose 5-6 % at 1345, 1530 and 1600.)
constexpr int split_of_768(int heads) {
    if (heads >= 520 && heads < 768) return split_fill(heads);
    if (split_last(heads, 512) < heads) return split_last(heads, 512);
    if (split_last(heads, 768) < heads) return split_last(heads, 768);
    return heads % 768 >= 544 ? split_fill(heads) : heads;
}

// Workgroups of a call that splits its heads from `from` on: eight row blocks of a head each, then those heads' other row blocks,
// and so on, both on one chiplet.
constexpr int split_grid(int from, int heads) { return from + (heads - from + 7) / 8 * 16; }
// Head (no head if >= heads) and row block of workgroup v
BINATTN_HD_SPLIT int split_head(int v, int from, int heads) {
    const int per_tail = (heads - from + 7) >> 3;
    return v < from ? (v & 7) * (from >> 3) + (v >> 3) : from + (v & 7) * per_tail + ((v - from) >> 4);
}
BINATTN_HD_SPLIT int split_row_block(int v, int from) { return v < from ? 0 : ((v - from) >> 3) & 1; }

}  // namespace binattn
