// Internal declarations shared by the HIP translation units of libbinattn.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "binattn.h"
#include "fast_div.h"
#include "head_split.h"
#include "psi_grid.h"

namespace binattn {

// Key/value block of Alg. 1 (B_v): 128 keys, i.e. four 32-key MFMA tiles.
constexpr int BV = 128;
// Query rows per workgroup (B_r of Alg. 1): 4 waves x 32 rows.
constexpr int BR = 128;
constexpr int ROWS_PER_WAVE = 32;
// Token rows reduced by one workgroup of the V absmax kernel.
constexpr int VCHUNK = 256;

struct Shape {
    int B, H, N, d;
    int BH;    // B * H
    int W;     // sign words per token = ceil(d / 32)
    int DK;    // 32-channel groups = W
    int DKP;   // padded channel count = 32 * DK
    int nblk;  // key blocks = ceil(N / BV)
    int npad;  // nblk * BV
    int nchunk;  // V absmax partials per head = ceil(N / VCHUNK)
};

inline Shape make_shape(int B, int H, int N, int d) {
    Shape s;
    s.B = B; s.H = H; s.N = N; s.d = d;
    s.BH = B * H;
    s.W = (d + 31) / 32;
    s.DK = s.W;
    s.DKP = 32 * s.DK;
    s.nblk = (N + BV - 1) / BV;
    s.npad = s.nblk * BV;
    s.nchunk = (N + VCHUNK - 1) / VCHUNK;
    return s;
}

// Operand image of one key/value block (BV keys) of one head, stored in the
// workspace exactly as the attention kernel wants it in LDS, so that a block is
// one flat asynchronous copy:
//   K  [BV positions][KP bytes]  FP4 codes of the +-1 keys, 32 bytes per 64 channels, rows in
//                                MFMA order; the 16-byte chunks of a row are XOR-swizzled (k_chunk)
//   VT [DKP channels][VP bytes]  V codes, channel-major, BV key bytes per row + 16 pad
//   CS [DKP] int32               PV_MAGIC + 128 * (sum of the row's BV codes)
// What no key or channel fills.  K: expand_k_blocks and expand_k_block (sign words) write zeros for channels beyond d
// and keys beyond N; phi_block (Q, K, V in one pass) writes whole rows, whatever LDS held there; phi_psi1_kernel leaves the
// workspace's old bytes.  V: codes of keys beyond N are 0, rows and seeds beyond d are zeros from prep_head_kernel and old
// bytes from psi_kernel and v_quant_kernel.  The single-launch forms, whose images exist in LDS only, clear nothing: V
// codes of token quads beyond N are old bytes there too, which the seeds include.  So a consumer replaces the
// logits of keys beyond N (their weight is 0, code -128, and the seed takes its share out again), keeps its query
// operand zero beyond d (FP4 has no NaN) and drops the accumulators beyond d.
// Swizzle and padding make the 16-byte reads of 16 consecutive rows fall into 16
// different 16-byte bank groups of the 256-byte LDS row.
template <int DK>
struct Image {
    static constexpr int DK2 = (DK + 1) / 2;       // 64-channel groups of the QK contraction
    static constexpr int DKP = 32 * DK;            // padded channel count of V
    static constexpr int KP = 32 * DK2;
    static constexpr int VP = BV + 16;
    static constexpr int K_OFF = 0;
    static constexpr int V_OFF = BV * KP;
    static constexpr int CS_OFF = V_OFF + DKP * VP;
    static constexpr int BYTES = (CS_OFF + DKP * 4 + 1023) / 1024 * 1024;
};

// Where 16-byte chunk `chunk` (of KP / 16) of K row `pos` is stored inside the row.
__host__ __device__ inline int k_chunk(int pos, int chunk, int KP) {
    return KP == 32 ? (chunk ^ ((pos >> 3) & 1)) : (chunk ^ ((pos >> 2) & 3));
}

// FP4 e2m1 codes of +1.0 and -1.0
constexpr unsigned FP4_PLUS1 = 0x2u, FP4_MINUS1 = 0xAu;

// 8 sign bits -> 8 FP4 nibbles, +1.0 where set, -1.0 where clear.  Bit 2 k goes to nibble k, bit
// 2 k + 1 to nibble 4 + k: the order in which two bf16 values per dword give their signs
// (fp4_pm1_abs).  The order inside a group of 8 channels is free as long as the Q and the K
// operand share it: every FP4 word of the library comes from these two routines.
__device__ __forceinline__ unsigned fp4_pm1_from_bits8(unsigned b) {
    unsigned x = (b & 0x55u) | ((b & 0xAAu) << 15);     // even bits at 2 k, odd bits at 16 + 2 k
    x = (x & 0x00050005u) | ((x & 0x00500050u) << 4);
    x = (x & 0x01010101u) | ((x & 0x04040404u) << 2);   // one bit per nibble, at its lowest position
    return 0xAAAAAAAAu - (x << 3);                      // 0xA - 8 = 0x2 where the bit is set
}

inline int image_bytes(int DK) {
    switch (DK) {
        case 1: return Image<1>::BYTES;
        case 2: return Image<2>::BYTES;
        case 3: return Image<3>::BYTES;
        default: return Image<4>::BYTES;
    }
}

// The int32 P.V accumulator of a block starts from PV_MAGIC + 128 * colsum: read
// as fp32 bits the finished accumulator is then 1.5 * 2^23 + (block result),
// exact while |block result| < 2^22 (128 keys * 255 * 127 = 4 145 280 fits).
constexpr int PV_MAGIC_BITS = 0x4B400000;
constexpr float PV_MAGIC_F = 12582912.0f;

// Private workspace layout (all offsets 256-byte aligned).
//   img   bytes [BH][nblk][Image<DK>::BYTES]
//   delta f32   [BH][DKP]
//   amax  f32   [BH][nblk][DKP]             partial absmax of V (per 256 tokens, or per key
//                                           block on the path that takes Q, K, V themselves)
// and, for that path:
//   mu    f32   [2][BH]                     abs-means of Q and K
//   psum  f32   [BH][nblk][2]               their partial sums per key block
//   qbits u32   [BH][N][W]                  query sign words
struct Workspace {
    size_t img, delta, amax, mu, psum, qbits, total;
    int img_bytes;
};

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

inline Workspace make_workspace(const Shape &s) {
    Workspace w;
    w.img_bytes = image_bytes(s.DK);
    size_t off = 0;
    w.img = off;   off = align256(off + (size_t)s.BH * s.nblk * w.img_bytes);
    w.delta = off; off = align256(off + (size_t)s.BH * s.DKP * 4);
    w.amax = off;  off = align256(off + (size_t)s.BH * s.nblk * s.DKP * 4);
    w.mu = off;    off = align256(off + (size_t)2 * s.BH * 4);
    w.psum = off;  off = align256(off + (size_t)s.BH * s.nblk * 2 * 4);
    w.qbits = off; off = align256(off + (size_t)s.BH * s.N * s.W * 4);
    w.total = off;
    return w;
}

// Up to this many key blocks psi can be one launch whose workgroups hold whole channel slabs of V, and the abs-means of
// the entry point that takes Q, K, V are added up by the attention kernel from their partial sums.
constexpr int PSI_MAX_BLOCKS = 32;
// Above 16 key blocks a wave of that launch takes four in turn, which few slabs do not hide: two passes, with a workgroup
// per key block, are faster there.  us, two passes / one: preparation, d = 64, N = 4096 1 head 7.2 / 9.2, 16 heads 8.5 / 9.9,
// 32 heads 13.0 / 10.7; d = 32, N = 2049 8 heads 7.0 / 7.8, 32 heads 8.6 / 8.2; d = 104, N = 4096 4 heads 9.7 / 10.5, 16 heads 12.9 / 11.5;
// but d = 72, N = 2816 4 heads 9.1 / 8.5.  With phi in the same launch, whole call, N = 4096: d = 32 8 heads 47.0 / 48.1, 24 heads
// 90.9 / 87.9; d = 72 4 heads 59.6 / 60.9, 12 heads 80.3 / 80.2; d = 128 4 heads 67.4 / 66.5.
constexpr bool psi_one_pass(int BH, int C16, int nblk, bool with_phi) {
    if (nblk > PSI_MAX_BLOCKS) return false;
    if (nblk <= 16) return true;
    const int slabs = BH * psi_slabs(C16);
    return with_phi ? C16 > 12 || slabs > 16 : (C16 > 8 && C16 < 12) || slabs > 32;
}

struct Strides3 {
    int64_t b, h, n;
};

// Launchers (each returns BINATTN_OK or BINATTN_ERR_LAUNCH).
int launch_pack_qk(const void *q, Strides3 qs, const void *k, Strides3 ks, const Shape &s,
                   uint32_t *q_bits, uint32_t *k_bits, float *mu_q, float *mu_k,
                   hipStream_t stream);
int launch_expand_k(const uint32_t *k_bits, const Shape &s, char *ws, const Workspace &w,
                    hipStream_t stream);
int launch_prepare(const void *v, Strides3 vs, const uint32_t *k_bits, const Shape &s, char *ws,
                   const Workspace &w, hipStream_t stream);
int launch_phi_psi(const void *q, Strides3 qs, const void *k, Strides3 ks, const void *v, Strides3 vs,
                   const Shape &s, char *ws, const Workspace &w, float *mu_q_out, float *mu_k_out,
                   hipStream_t stream);
int launch_export_vq(const Shape &s, const char *ws, const Workspace &w, int8_t *vq, float *delta,
                     hipStream_t stream);
int launch_logits_popcount(const uint32_t *q_bits, const uint32_t *k_bits, const Shape &s,
                           int row_begin, int row_end, int32_t *logits, bool rowsum, hipStream_t stream);
int launch_logits_fp4(const uint32_t *q_bits, const char *ws, const Workspace &w, const Shape &s,
                      int row_begin, int row_end, int32_t *logits, bool rowsum, hipStream_t stream);
int launch_logits_i8(const uint32_t *q_bits, const uint32_t *k_bits, const Shape &s, int row_begin,
                     int row_end, int32_t *logits, bool rowsum, hipStream_t stream);

int launch_probe_valu(int op, int iters, int blocks, float *out, hipStream_t stream);

enum BiasMode {
    BIAS_NONE = 0,
    BIAS_BF16_VEC = 1,  // rows straight into registers, one block ahead (row pitch >= 2^27; d > 96 with one row block, or with
                        // rows on 4-byte words that are no whole 16-byte chunks)
    BIAS_F32_VEC = 3,   // fp32 rows, 16-byte loads at use (row pitch >= 2^27; d > 96 with one row block)
    BIAS_F32_LDS = 15,  // fp32 rows of any alignment: most of the tile staged global -> LDS, the rest into registers
    BIAS_BF16_LDS = 5,  // rows of any alignment: tile staged global -> LDS asynchronously
    BIAS_BF16_LDS8 = 17, // the same for N a multiple of 8 (4-wave workgroups over a prepared workspace): no copy reads past a row
    BIAS_AXIAL = 7,     // b_ij = y[iy - jy] + x[ix - jx] on a Gy x Gx token grid, tables held in LDS
    BIAS_TABLE = 9,     // b_ij = t[iy - jy][ix - jx]: the full relative-position table of the head in LDS (single-launch forms)
    BIAS_TABLE_BLK = 13, // the same table, only the rows a key block needs, staged per block
    BIAS_LUT = 11       // no bias: 255 exp(S - m) read from a per-head table indexed by (m - I) / 2
};

// largest grid side of BIAS_AXIAL (the tables of one head live in LDS)
constexpr int AXIAL_MAX_G = 256;
// largest grid side of BIAS_TABLE (4 N - 2 Gx <= 1024 entries of a head's table held in LDS)
constexpr int TABLE_MAX_G = 32;

struct FusedParams {
    const uint32_t *q_bits;
    const float *mu_q, *mu_k;  // may be null (taken as 1)
    const float *psum;         // partial sums of the abs-means, [BH][nblk][2] (then nblk <= PSI_MAX_BLOCKS and mu_q, mu_k unused), or null
    float inv_count;           // 1 / (N d)
    const void *bias;          // may be null
    Strides3 bs;               // bias element strides (batch, head, row)
    int64_t bias_end;          // elements of the dense bias from its first to its last one
    float scale;
    uint16_t *out;
    Strides3 os;
    const char *img;     // block images
    const float *delta;
    int B, H, N, d, nblk, nrb, total_wg;
    FastDiv div_inner, div_rows;  // work item number -> (batch, row block, head): by B / nb and nrb; single-launch forms: by H
    int nb;              // batch entries per workgroup (1 or 2)
    int wide;            // 0; 1 / 3 / 8: single-launch forms (8 waves / 4 / 4, three per compute unit); 2: 8-wave workgroups over row-block pairs (nrb counts pairs); 4: paired form, bias copied past the caches
    // single-launch short-sequence kernel: the bf16 inputs, whether mu is applied, optional mu exports
    const uint16_t *xq, *xk, *xv;
    Strides3 xqs, xks, xvs;
    int small_pitch;     // rows of xq, xk, xv less than HEAD_FAR_PITCH elements apart
    int use_mu;
    int phase512;        // 8-wave forms: the accumulator's offset is removed where the 4-wave form on the grid of 512 does
    int split_from;      // 4-wave single launch: heads from this one on take a workgroup per row block (a multiple of 8, or total_wg)
    int split_sums;      // 4-wave single launch: abs-means in the 8-wave form's order
    float *mu_q_out, *mu_k_out;
    const float *ax_y, *ax_x;  // BIAS_AXIAL: fp32 [H][2 Gy - 1], [H][2 Gx - 1]
    const float *table;        // BIAS_TABLE: fp32 [H][2 Gy - 1][2 Gx - 1]
    int Gy, Gx, gx_shift;      // BIAS_AXIAL / BIAS_TABLE: token grid, Gx = 1 << gx_shift
};

// The kernels of a head dimension, DK = ceil(d / 32), defined (and explicitly instantiated) in fused_dk<DK>.hip; FORMS = FORM_HALF, in
// fused_dk<DK>_half.hip, where d ends in the first half of the last 32 channels.
constexpr int FORM_HALF = 16;
constexpr bool half_form(int DK, int d) { return (DK == 2 || DK == 3) && d <= 32 * DK - 16; }
template <int DK, int FORMS>
int launch_fused_dk(const FusedParams &p, int mode, hipStream_t stream);
// The single-launch forms, for at most two key blocks (total_wg = B * H): nb = 2 for one 8-wave workgroup per head, 1 for 4-wave
// workgroups, which calls with more heads than this take (two or three per compute unit).
constexpr int ONEHEAD4_MIN_HEADS = 256;
// Three 4-wave workgroups per compute unit instead of two (32 < d <= 64).  Without a bias they are at least as fast everywhere (us,
// two / three: N = 197 400 heads 19.8 / 19.7, 768 31.6 / 28.1, 1536 54.5 / 48.4, N = 256 1024 42.5 / 38.3, N = 100 768 18.6 / 15.8) and the only form.  With bf16
// tiles a head takes longer: up to 512 heads, one round of either, two are faster (N = 197 24.5 / 26.4).  Above, three / two, each with its best split,
// over N = 129, 160, 180, 197, 224 and d = 40, 48, 64 (mean, least .. most): 513 heads 0.87, 0.81 .. 0.92, 700 0.91, 0.84 .. 0.95, 870 0.97, 0.92 .. 1.03, 960 0.98, 0.94 .. 1.05,
// 1200 0.91, 0.86 .. 0.94, 1480 0.92, 0.88 .. 0.97, 1800 0.90, 0.87 .. 0.94, 2304 0.88, 0.84 .. 0.93, 3500 0.88, 0.82 .. 0.96; between 897 and 1024, where
// 768 leave a last round that is less than a third full and 512 fill theirs, it goes either way with N (d = 40, 960 heads N = 129 30.8 / 32.4, d = 64 N = 224
// 41.9 / 39.4), and two stay.  N <= 128 and N > 224 spill there, and fp32 tiles do not fit.
constexpr bool onehead_three_only(int DK, int mode) { return DK == 2 && mode == BIAS_NONE; }
constexpr bool onehead_three(int DK, int mode, int N, int heads) {
    if (onehead_three_only(DK, mode)) return true;
    return DK == 2 && mode == BIAS_BF16_LDS && N > BV && N <= 2 * BV - 32 && heads > 512 && !(heads > 896 && heads <= 1024);
}
// The first head that is split by row blocks (head_split.h): for rounds of 768 where three workgroups share a compute unit, which
// they do up to 32 channels as well, without a bias and with bf16 tiles.
constexpr int onehead_split_from(int DK, int mode, bool three, int heads, int row_blocks) {
    if (row_blocks != 2) return heads;
    return three || (DK == 1 && (mode == BIAS_NONE || mode == BIAS_BF16_LDS)) ? split_of_768(heads) : split_last(heads, 512);
}
// The 4-wave form is built in the variants whose 256-thread prologue holds a head's loads in registers without spilling
constexpr bool onehead4_built(int DK, int mode) {
    return DK <= 2 || (DK == 3 && (mode == BIAS_NONE || mode == BIAS_F32_VEC || mode == BIAS_F32_LDS || mode == BIAS_BF16_LDS ||
                       mode == BIAS_AXIAL || mode == BIAS_TABLE));
}

template <int DK, int FORMS>
int launch_onehead_dk(const FusedParams &p, int mode, hipStream_t stream);

inline int check_launch() {
    return hipGetLastError() == hipSuccess ? BINATTN_OK : BINATTN_ERR_LAUNCH;
}

}  // namespace binattn
