// Which elements of a dense bias the LDS copies of the fused kernel read, and where they land.  Index arithmetic
// only, the same on the device and in a host program, so that the bounds can be checked without a GPU.
//
// A wave stages the 32 rows [row0, row0 + 32) x 128 keys of one (batch, head) in segments of 128 bytes per row.  One
// copy instruction moves 8 rows (group rg) of one segment: lane L fetches the 16-byte chunk c = bias_copy_chunk of
// row bias_copy_row and the hardware puts it at 16 L.  Chunk c of row r of the group so lands at
// 128 (r ^ (rg & 1)) + 16 (c ^ r): the later 16-byte reads of 16 consecutive rows (two groups) at one chunk index hit
// 16 different 16-byte bank groups of the 256-byte LDS row.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define BINATTN_HD __host__ __device__ __attribute__((always_inline)) inline
#else
#define BINATTN_HD inline
#endif

namespace binattn {

BINATTN_HD int bias_min(int a, int b) { return a < b ? a : b; }

// elements from the first to the last one of a bias with element strides sb, sh, sn
BINATTN_HD int64_t bias_extent(int B, int H, int N, int64_t sb, int64_t sh, int64_t sn) {
    return (int64_t)(B - 1) * sb + (int64_t)(H - 1) * sh + (int64_t)(N - 1) * sn + N;
}

// first row of group rg, clamped into the tensor; the row and chunk a lane fetches
BINATTN_HD int bias_group_row(int row0, int rg, int N) { return bias_min(row0 + 8 * rg, N - 1); }
BINATTN_HD int bias_copy_row(int group_row, int rg, int lane, int N) {
    return bias_min(group_row + ((lane >> 3) ^ (rg & 1)), N - 1);
}
BINATTN_HD int bias_copy_chunk(int rg, int lane) { return (lane & 7) ^ (lane >> 3) ^ (rg & 1); }

// LDS offset of chunk c of segment seg of row m (0 <= m < 32) inside a wave's region of `segs` segments per row
BINATTN_HD unsigned bias_lds_chunk(int m, int seg, int c, int segs) {
    return ((m >> 3) * segs + seg) * 1024 + 128 * ((m & 7) ^ ((m >> 3) & 1)) + 16 * (c ^ (m & 7));
}

// Keys from which on a wave leaves chunks of ec elements out.  The last chunk of a row that straddles N reads on
// into whatever follows the row, which is still inside the tensor except behind its very last row: a wave
// whose rows include one that would read past `extent` stops at the last whole chunk (limit N - ec + 1 instead of N)
// and fetches the rest element by element.  off: element offset of the wave's (batch, head).
BINATTN_HD int bias_key_limit(int64_t off, int row0, int N, int64_t sn, int64_t extent, int first_key, int ec) {
    if (first_key + 128 <= N || (N & (ec - 1)) == 0) return N;
    const int last_row = bias_min(row0 + 32, N) - 1;
    return off + (int64_t)last_row * sn + ((N + ec - 1) & -ec) > extent ? N - (ec - 1) : N;
}

}  // namespace binattn
