// Which rows of V the threads of a single-launch workgroup load.  Index arithmetic only (constexpr: the same on the
// device and in a host program), so that the coverage can be checked without a GPU.
//
// A thread owns one 8-channel chunk (of c16 = d / 8 per row) of quads of four consecutive tokens; consecutive threads take
// consecutive chunks, so nt threads are nt / c16 whole groups with a quad each, and a few threads behind them that
// repeat the first chunks of the next pass.  Rows are read through a buffer descriptor that ends with the last one: what
// lies behind it reads as zeros, as long as its 32-bit byte offset does not wrap.
#pragma once

namespace binattn {

constexpr int HEAD_QUADS = 64;  // token quads of two key blocks

// Passes that cover all quads whatever d in (32 (dk - 1), 32 dk] is: the widest rows leave the fewest groups (nt = 256,
// dk = 3: 21 groups at d = 96, and three passes over 21 quads stop one short of 64).  Narrower rows leave out the
// passes that head_v_pass calls empty.
constexpr int head_v_passes(int nt, int dk) { return (HEAD_QUADS + nt / (4 * dk) - 1) / (nt / (4 * dk)); }
constexpr int head_v_groups(int nt, int c16) { return nt / c16; }
constexpr bool head_v_pass(int pass, int groups) { return pass * groups < HEAD_QUADS; }
// group of a thread, number = thread / c16.  Up to d = 24 there are more than 64 in the one pass: those all take quad
// 64, which no call has.  (Counted on, their rows, up to 2047, would wrap at far pitches.)  Forms that have no such groups
// are built without the minimum (512 heads, N = 256, d = 72 29.74 -> 29.62 us).
constexpr int head_v_group(int number, int nt, int dk) {
    return nt / (4 * dk - 3) <= HEAD_QUADS || number < HEAD_QUADS ? number : HEAD_QUADS;
}
// quad of the thread in group `group`; HEAD_QUADS or more: none
constexpr int head_v_quad(int group, int pass, int groups) { return group + pass * groups; }
// So the largest row whose offset is formed is 4 * 127 + 3, and rows up to 511 at pitches below this many elements have
// 32-bit byte offsets; other pitches take 64-bit addresses.
constexpr int HEAD_FAR_PITCH = 1 << 22;

}  // namespace binattn
