// The grid of psi_kernel: channel slabs of V, and behind them the key blocks it packs or expands.  Plain arithmetic, the
// same in the library and in a host program that checks it.
#pragma once

#include <stdint.h>

namespace binattn {

constexpr int psi_slabs(int C16) { return (C16 + 3) / 4; }  // slabs of a head, of four 8-channel chunks at most
constexpr int psi_threads(int nblk) { return nblk <= 4 ? 256 : 512; }

enum PsiKeys { PSI_V_ONLY, PSI_EXPAND, PSI_PHI };  // nothing else; sign words -> operand rows; Q, K -> signs and operand rows
constexpr int PSI_K_BLOCKS = 4;                    // key blocks whose sign words one workgroup expands
constexpr int PSI_PHI_THREADS = 256;               // threads that take a key block of Q and K

constexpr int64_t psi_key_workgroups(int heads, int nblk, PsiKeys keys) {
    return keys == PSI_PHI      ? (int64_t)heads * ((nblk + psi_threads(nblk) / PSI_PHI_THREADS - 1) / (psi_threads(nblk) / PSI_PHI_THREADS))
           : keys == PSI_EXPAND ? ((int64_t)heads * nblk + PSI_K_BLOCKS - 1) / PSI_K_BLOCKS
                                : 0;
}
// slabs are dealt out to the eight chiplets in equal shares
constexpr int64_t psi_workgroups(int heads, int C16, int nblk, PsiKeys keys) {
    return ((int64_t)heads * psi_slabs(C16) + 7) / 8 * 8 + psi_key_workgroups(heads, nblk, keys);
}
// The most heads of one launch, which the runtime refuses from 2^32 threads on (2.1 million heads of N = 640, d = 8): calls
// with more take several.
constexpr int psi_heads(int C16, int nblk, PsiKeys keys) {
    return (int)((((int64_t)1 << 32) / psi_threads(nblk) - 8) / (psi_slabs(C16) + psi_key_workgroups(1, nblk, keys)));
}

}  // namespace binattn
