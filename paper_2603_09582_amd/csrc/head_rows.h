// Which rows of V the threads of a single-launch workgroup load.  Index arithmetic only (constexpr: the same on the
// device and in a host program), so that the coverage can be checked without a GPU.
//
// A thread owns one 8-channel chunk (of c16 = d / 8 per row) of quads of four consecutive tokens; consecutive threads take
// consecutive chunks, so nt threads are nt / c16 whole groups with a quad each, and a few threads behind them that
// repeat the first chunks of the next pass.
#pragma once

namespace binattn {

constexpr int HEAD_QUADS = 64;  // token quads of two key blocks

// Passes that cover all quads whatever d in (32 (dk - 1), 32 dk] is: the widest rows leave the fewest groups (nt = 256,
// dk = 3: 21 groups at d = 96, and three passes over 21 quads stop one short of 64).  Narrower rows leave out the
// passes that head_v_pass calls empty.
constexpr int head_v_passes(int nt, int dk) { return (HEAD_QUADS + nt / (4 * dk) - 1) / (nt / (4 * dk)); }
constexpr int head_v_groups(int nt, int c16) { return nt / c16; }
constexpr bool head_v_pass(int pass, int groups) { return pass * groups < HEAD_QUADS; }
// quad of the thread in group `group` (its number / c16); HEAD_QUADS or more: none
constexpr int head_v_quad(int group, int pass, int groups) { return group + pass * groups; }

}  // namespace binattn
