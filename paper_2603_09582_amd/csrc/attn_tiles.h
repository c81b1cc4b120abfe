// Device routines shared by the fused attention kernel and the logits export:
// the per-block operand image, its asynchronous copy into LDS, and the QK tile
// on the matrix cores.
//
// Register/lane convention (wave64, 32x32 MFMA tiles, D = A*B + C):
//   lane L feeds row (A) / column (B) number (L & 31) with the k-slots of group
//   g = L >> 5.  A and B use the same slot numbering, so any consistent
//   assignment of channels (or keys) to slots gives the same contraction.
//   D: lane L holds column (L & 31); register r holds row 8(r/4) + 4g + (r%4).
// The kernels put KEYS (resp. value channels) on the A side and QUERIES on the
// B side, so that every lane owns one query row: all softmax statistics are
// lane-local, and the P tile a lane produces is already in B-operand order for
// the P.V contraction (no LDS round trip).
//
// QK runs as v_mfma_f32_32x32x64_f8f6f4 with FP4 (e2m1) operands: +1.0 and -1.0
// are exact in FP4, the products and the fp32 accumulation of at most 128 of
// them are exact, so the result is the integer logit of Sec. 4.1 already in
// fp32 (no int->float conversion), and the accumulator input carries the bias
// term of Eq. 6 for free.  An int8 form of the same tile is kept for comparison.
#pragma once

#include "binattn_internal.h"

namespace binattn {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned u4v __attribute__((ext_vector_type(4)));  // 16-byte register

constexpr int FUSED_THREADS = 256;
constexpr int KT = BV / 32;  // MFMA key tiles per block

// B operand of the QK tile for this lane's query row: FP4 codes of channels
// 64 s + 32 g + [0, 32) in 16 bytes, zero beyond d.  q_words: the row's sign words
// (zero-filled up to 2 * DK2).  `flip` negates the row, `zero` clears it (used for a
// non-positive or vanishing logit multiplier).
template <int DK2>
__device__ __forceinline__ void load_q_operand(const unsigned q_words[2 * DK2], int d, int g,
                                               bool flip, bool zero, v4i qB[DK2]) {
#pragma unroll
    for (int s = 0; s < DK2; ++s) {
        unsigned word = g ? q_words[2 * s + 1] : q_words[2 * s];
        if (flip) word = ~word;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c0 = 32 * (2 * s + g) + 8 * i;
            qB[s][i] = (c0 < d && !zero) ? (int)fp4_pm1_from_bits8((word >> (8 * i)) & 0xFFu) : 0;
        }
    }
}

// A operand rows of QK tile t for this lane (LDS reads only).
template <int DK>
__device__ __forceinline__ void load_k_operand(const char *img, int t, int m, int g,
                                               v4i ka[(DK + 1) / 2]) {
    using L = Image<DK>;
#pragma unroll
    for (int s = 0; s < L::DK2; ++s)
        ka[s] = *reinterpret_cast<const v4i *>(img + L::K_OFF + (32 * t + m) * L::KP +
                                               16 * k_chunk(m, 2 * s + g, L::KP));
}

// QK tile: for this lane's query, register r of the result is
// cin[r] + (s_i . t_j) with key j = block start + 32 t + 16 g + r.
template <int DK2>
__device__ __forceinline__ v16f qk_mfma(const v4i ka[DK2], const v4i qB[DK2], v16f cin) {
#pragma unroll
    for (int s = 0; s < DK2; ++s) {
        const v8i a8 = {ka[s][0], ka[s][1], ka[s][2], ka[s][3], 0, 0, 0, 0};
        const v8i b8 = {qB[s][0], qB[s][1], qB[s][2], qB[s][3], 0, 0, 0, 0};
        cin = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, cin, 4, 4, 0, 0, 0, 0);
    }
    return cin;
}

template <int DK>
__device__ __forceinline__ v16f qk_tile(const char *img, int t, int m, int g,
                                        const v4i qB[(DK + 1) / 2], v16f cin) {
    v4i ka[(DK + 1) / 2];
    load_k_operand<DK>(img, t, m, g, ka);
    return qk_mfma<(DK + 1) / 2>(ka, qB, cin);
}

// LDS byte offset of a pointer into a __shared__ array.
__device__ __forceinline__ unsigned lds_offset(const void *p) {
    return (unsigned)(size_t)(__attribute__((address_space(3))) const char *)p;
}

// A pointer that is the same in every lane, moved into scalar registers.
template <class T>
__device__ __forceinline__ const T *uniform_ptr(const T *p) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    // (the builtin returns int: widen through unsigned, or the low half is sign-extended)
    const uint64_t u = (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((unsigned)a) |
                       ((uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((unsigned)(a >> 32)) << 32);
    return reinterpret_cast<const T *>(u);
}

// One asynchronous 16-byte-per-lane copy global -> LDS: lane L's 16 bytes, read from
// sbase + voff (sbase wave-uniform, kept in scalar registers; voff this lane's byte offset),
// land at lds_base + 16 L (lds_base wave-uniform).  Issued through inline assembly so that
// the compiler does not serialise later LDS reads of OTHER buffers against it; the callers
// order it by hand (wait_vmem + barrier before the data is read).  ONCE: data that no other
// workgroup is about to read ("nt": first to leave the caches).
template <bool ONCE = false>
__device__ __forceinline__ void dma16(const void *sbase, unsigned voff, unsigned lds_base) {
    const uint64_t u = reinterpret_cast<uint64_t>(uniform_ptr(static_cast<const char *>(sbase)));
    if constexpr (ONCE)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                     :
                     : "s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(voff), "s"(u)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :
                     : "s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(voff), "s"(u)
                     : "memory", "m0");
}

// NC consecutive KiB (NC = 1 .. 4) the same way: the instruction's offset moves both addresses, so one base and one
// setting of m0 serve them all.  (A scalar instruction costs the wave as much time as a vector one where two waves share a
// SIMD; copy by copy a block's image took 5 per KiB.)
template <int NC>
__device__ __forceinline__ void dma_kib(const char *sbase, unsigned voff, unsigned lds_base) {
    static_assert(NC >= 1 && NC <= 4, "the offset field ends at 4095");
    const uint64_t u = reinterpret_cast<uint64_t>(uniform_ptr(sbase));
    const unsigned l = __builtin_amdgcn_readfirstlane(lds_base);
#define HEAD "s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, %2"
#define NEXT(o) "\n\tglobal_load_lds_dwordx4 %1, %2 offset:" #o
    if constexpr (NC == 1) asm volatile(HEAD : : "s"(l), "v"(voff), "s"(u) : "memory", "m0");
    if constexpr (NC == 2) asm volatile(HEAD NEXT(1024) : : "s"(l), "v"(voff), "s"(u) : "memory", "m0");
    if constexpr (NC == 3) asm volatile(HEAD NEXT(1024) NEXT(2048) : : "s"(l), "v"(voff), "s"(u) : "memory", "m0");
    if constexpr (NC == 4) asm volatile(HEAD NEXT(1024) NEXT(2048) NEXT(3072) : : "s"(l), "v"(voff), "s"(u) : "memory", "m0");
#undef HEAD
#undef NEXT
}
template <int NC>
__device__ __forceinline__ void dma_run(const char *sbase, unsigned voff, unsigned lds_base) {
    if constexpr (NC > 4) {
        dma_kib<4>(sbase, voff, lds_base);
        dma_run<NC - 4>(sbase + 4096, voff, lds_base + 4096);
    } else if constexpr (NC > 0) {
        dma_kib<NC>(sbase, voff, lds_base);
    }
}

// Asynchronous copy of one block image (L::BYTES, a multiple of 1 KiB) from
// global memory straight into LDS by NW waves (wave = 0 .. NW - 1), each of
// which moves a run of KiB.
template <int DK, int NW = 4>
__device__ __forceinline__ void dma_image(const char *__restrict__ gsrc, unsigned ldst, int wave, int lane) {
    constexpr int NCH = Image<DK>::BYTES / 1024, PER = (NCH + NW - 1) / NW, REST = NCH % PER;
    const int c = wave * PER;
    if (c + PER <= NCH)
        dma_run<PER>(gsrc + c * 1024, lane * 16, ldst + c * 1024);
    else if (REST > 0 && c < NCH)
        dma_run<REST>(gsrc + c * 1024, lane * 16, ldst + c * 1024);
}

// The staged part of a wave's bias tile for one whole key block: row groups j = 0 .. 3, SEGS segments of 128 bytes per row; lane offset
// voff[j] from base[j], each copy to its own KiB of the region, in the order of the region.  (m0 carries minus the
// instruction's offset, which moves both addresses.)
template <int SEGS>
__device__ __forceinline__ void dma_tile(const char *const (&base)[4], const unsigned (&voff)[4], unsigned lds_base) {
    static_assert(SEGS >= 1 && SEGS <= 3, "one to three segments per row");
    const uint64_t b0 = reinterpret_cast<uint64_t>(base[0]), b1 = reinterpret_cast<uint64_t>(base[1]);
    const uint64_t b2 = reinterpret_cast<uint64_t>(base[2]), b3 = reinterpret_cast<uint64_t>(base[3]);
    const unsigned l = __builtin_amdgcn_readfirstlane(lds_base);
#define COPY(v, s, o) "global_load_lds_dwordx4 " v ", " s " offset:" #o "\n\t"
#define STEP(n) "s_add_u32 m0, m0, " #n "\n\ts_nop 0\n\t"
#define ROWS2(v, s) COPY(v, s, 0) STEP(0x380) COPY(v, s, 128)
#define ROWS3(v, s) COPY(v, s, 0) STEP(0x380) COPY(v, s, 128) STEP(0x380) COPY(v, s, 256)
    if constexpr (SEGS == 1)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\t"
                     COPY("%1", "%5", 0) STEP(0x400) COPY("%2", "%6", 0) STEP(0x400) COPY("%3", "%7", 0) STEP(0x400) COPY("%4", "%8", 0)
                     : : "s"(l), "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3]), "s"(b0), "s"(b1), "s"(b2), "s"(b3)
                     : "memory", "m0", "scc");
    else if constexpr (SEGS == 2)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\t"
                     ROWS2("%1", "%5") STEP(0x480) ROWS2("%2", "%6") STEP(0x480) ROWS2("%3", "%7") STEP(0x480) ROWS2("%4", "%8")
                     : : "s"(l), "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3]), "s"(b0), "s"(b1), "s"(b2), "s"(b3)
                     : "memory", "m0", "scc");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\t"
                     ROWS3("%1", "%5") STEP(0x500) ROWS3("%2", "%6") STEP(0x500) ROWS3("%3", "%7") STEP(0x500) ROWS3("%4", "%8")
                     : : "s"(l), "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3]), "s"(b0), "s"(b1), "s"(b2), "s"(b3)
                     : "memory", "m0", "scc");
#undef COPY
#undef STEP
#undef ROWS2
#undef ROWS3
}

__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// max / sum over the two lanes L and L ^ 32 (they share a query row), on the vector ALU.
__device__ __forceinline__ float pair_max(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    float o;  // (fmaxf would quiet both operands first, two instructions more; they are results of maxima)
    asm("v_max_f32 %0, %1, %2" : "=v"(o) : "v"(r[0]), "v"(r[1]));
    return o;
}
__device__ __forceinline__ float pair_sum(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// sum over the lanes i + 16, i + 8, i + 4, i + 2, i + 1 of lane i's pair of rows, added in that order (a lane's partner is the
// one a rotation of its row of 16 brings: the sums of both are the same)
__device__ __forceinline__ float row_tree_sum(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xf, 0xf, false));  // row_ror:8
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xf, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x122, 0xf, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x121, 0xf, 0xf, false));
    return x;
}

}  // namespace binattn
