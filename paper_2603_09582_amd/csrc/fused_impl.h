// The fused loop of Alg. 1 for one (batch, head, 128-query block) per
// workgroup: QK logits on the matrix cores, scale + bias (Eq. 6), online
// softmax, unsigned 8-bit P, int8 P.V with int32 accumulation, fp32 carry.
//
// One wave owns 32 query rows; a lane owns ONE query row and half of the keys
// of every block: of tile t's 32 keys those at 32 t + 16 g + [0, 16), g = lane / 32.
// The vector ALU is the binding unit of this kernel, so the design removes
// vector instructions wherever another unit can do the work.  Per key block of
// BV = 128 keys:
//   0. the next block's operand image is copied global -> LDS asynchronously
//      (no staging registers, no LDS store instructions)
//   1. T = I + b / alpha: the bias is unpacked, divided by the logit multiplier
//      alpha = scale * mu_q * mu_k and handed to the FP4 MFMA as its accumulator
//      input; the MFMA adds the exact integer logit I = s_i . t_j in fp32.
//      (S of Eq. 6 is alpha * T; alpha > 0 after folding its sign into the Q
//      operand, so maxima can be taken on T.)
//   2. block max of T (one cross-lane exchange with lane ^ 32), running max m
//   3. p = 255 * exp(S - m) = exp2(T * alpha*log2(e) + c) with one FMA and one
//      v_exp_f32; row sum in fp32; p rounded to a byte by v_cvt_pk_u8_f32
//      (Eq. 7, scale 1/255, relative to the running maximum as in Alg. 1)
//   4. P.V: the int8 MFMA is signed x signed, so the operand is P - 128 and the
//      accumulator starts from 128 * (column sums of the V block), precomputed
//      by the V quantisation kernel: exact in int32.  The seed also carries the
//      bit pattern of 1.5 * 2^23, so the finished int32 accumulator, read as
//      fp32 bits, IS the float 1.5 * 2^23 + result: no int->float conversion.
//   5. O = exp(m_old - m_new) * O + block result (Alg. 1's rescale line, read as
//      a multiplication) is one FMA per output register; the 1.5 * 2^23 offsets
//      accumulate as 1.5 * 2^23 * rho with rho = sum of the rescale products,
//      tracked per row and subtracted every eighth block and at the end.
// Final: (O - 1.5*2^23*rho) / (sum of 255 * P_hat) * delta_v (Alg. 1 last line;
// the factor 255 is already inside the row sum).
#pragma once

#include <type_traits>

#include "attn_tiles.h"
#include "bias_rows.h"
#include "fast_div.h"
#include "head_rows.h"
#include "quant_v.h"

namespace binattn {

// 16-byte loads from addresses that are only element-aligned (gfx950 under HSA
// supports unaligned vector loads; the compiler still emits one dwordx4 load).
typedef u4v u4v_a2 __attribute__((aligned(2)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef f4v f4v_a4 __attribute__((aligned(4)));

constexpr float LOG2E_F = 1.44269504088896340736f;
constexpr float LOG2_255_F = 7.99435343685885793770f;

__device__ __forceinline__ float bf16_lo(unsigned w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(unsigned w) { return __uint_as_float(w & 0xffff0000u); }

// two fp32 -> two bf16 in one dword, round to nearest even (v_cvt_pk_bf16_f32)
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned pack_bf16x2(float lo, float hi) {
    const f2v v = {lo, hi};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

// NB = batch entries per workgroup.  NB = 2 (only with BIAS_BF16_LDS and a bias shared
// over the batch) puts two batch entries of the same (head, row block) into one
// 8-wave workgroup: waves 0-3 work on entry 2 bp, waves 4-7 on entry 2 bp + 1, and
// both read the SAME bias tile from LDS, so the bias - the dominant HBM stream of
// long sequences - is fetched once per pair and can be double-buffered.
//
// With NB = 1 the grid is persistent: a workgroup walks work items v, v + G, v + 2G, ...
// (G = grid size) and treats all their key blocks as ONE stream, so the asynchronous
// copies for the first block of the next item are already in flight during the last
// block of the current one; only the very first block of a workgroup waits for memory.
// That pays for short sequences (few blocks per item).  NB = 2 is only used for long
// sequences, where the item switch is rare and its bookkeeping at the start of every
// block (all waves of a workgroup pass it together, right after the barrier, so it is
// not hidden behind another wave's arithmetic) costs more than it saves: there a
// workgroup computes one item.
//
// ONEHEAD (8 waves) is the single-launch form for at most two key blocks: one workgroup
// owns a whole (batch, head).  It reads the bf16 Q, K, V itself, makes the sign bits, both
// abs-means, the V codes and both operand images directly in LDS (phi and psi of Alg. 1
// fused into their consumer), then runs the same block loop on its two 128-row blocks
// (waves 0-3 / 4-7).  Nothing but the bias and the inputs is read from memory and only the
// output is written.
//
// WIDE_ROWS2 (8 waves) serves head dimensions whose operand images leave no LDS room for two
// 4-wave workgroups with bias tiles (d > 96): the two halves of the workgroup are the row
// blocks 2 rp, 2 rp + 1 of ONE (batch, head); they share the operand images (one copy stream
// for 256 rows) and keep private bias tiles; the grid is persistent as with NB = 1.
//
// ONEHEAD4 (4 waves) is the single-launch form for launches with more heads than compute units:
// the same prologue with 256 threads, then the head's two 128-row blocks one after the other
// as two items of the persistent stream (the images stay where they are).  Two such workgroups
// share a compute unit, so one head's loads and preparation overlap the other's block loop.
// (The last heads take a workgroup per row block where that fills a round better: head_split.h.)
//
// WIDE_PAIR_ONCE is the paired form (NB = 2) with the bias copies marked as not worth keeping in the
// caches, for biases larger than those.
//
// WIDE_WAVES3 is the ordinary 4-wave form compiled for three waves per SIMD (168 registers), three
// workgroups per compute unit, in the variants of use_waves3.
//
// WIDE_TRI4 and WIDE_TRISHORT4 are ONEHEAD4 (the latter with what WIDE_SHORT4 leaves out) for three workgroups per compute unit:
// 168 registers, 53 KB of LDS.  Of a bf16 tile half the keys are staged, the others loaded into registers a block ahead; V rows are
// read behind the exponentials, the second row's words kept in LDS.  Chosen by onehead_three.
//
// WIDE_SHORT and WIDE_SHORT4 are the single-launch forms for 128 < N <= 224, whose second key block ends at least 32 keys early:
// the 32-key tiles behind N are left out of it, and waves whose rows all lie there out of the second row block.  (us, without / with: N = 197, d = 64 3 heads 12.14 / 11.70, 512 heads 25.2 / 24.2, 768 heads
// 38.1 / 36.3, N = 129 35.4 / 30.5; the branches cost calls whose last tile holds a key 1.2-1.5 %, so those keep the forms without.)
enum { WIDE_NONE = 0, WIDE_ONEHEAD = 1, WIDE_ROWS2 = 2, WIDE_ONEHEAD4 = 3, WIDE_PAIR_ONCE = 4, WIDE_WAVES3 = 5, WIDE_SHORT = 6, WIDE_SHORT4 = 7, WIDE_TRI4 = 8, WIDE_TRISHORT4 = 9 };
//
// FORM is one of these, plus FORM_HALF where at least half of the last 32-channel block lies beyond d (d = 40, 48, 72, 80): its upper two quads
// of channels per lane have no carry, no seeds and no output.  (Attention stage, us, without / with: N = 1024, d = 72, 128 heads, bf16 46.1 / 45.6, table
// 42.1 / 40.7, N = 1370, d = 80, 64 heads 53.2 / 52.0; one launch, N = 256, d = 72, 512 heads 29.8 / 29.2.)
template <int DK, int MODE, int NB, int FORM = WIDE_NONE>
__global__ __launch_bounds__(FUSED_THREADS * NB, ((FORM & 15) == WIDE_WAVES3 || (FORM & 15) >= WIDE_TRI4 ? 3 : 2)) void fused_kernel(const FusedParams p) {
    constexpr int WIDE = FORM & 15;
    using L = Image<DK>;
    constexpr bool TRI = WIDE == WIDE_TRI4 || WIDE == WIDE_TRISHORT4;
    constexpr bool SHORT = WIDE == WIDE_SHORT || WIDE == WIDE_SHORT4 || WIDE == WIDE_TRISHORT4;
    constexpr bool ONEHEAD4 = WIDE == WIDE_ONEHEAD4 || WIDE == WIDE_SHORT4 || TRI;
    constexpr bool ONEHEAD = WIDE == WIDE_ONEHEAD || SHORT || ONEHEAD4, ROWS2 = WIDE == WIDE_ROWS2;
    constexpr bool WAVES3 = WIDE == WIDE_WAVES3;
    static_assert(WIDE == WIDE_NONE || ONEHEAD4 || WAVES3 || NB == 2, "the wide forms use 8 waves");
    static_assert(!ONEHEAD4 || NB == 1, "the 4-wave single-launch form");
    constexpr bool PAIR = NB == 2 && (WIDE == WIDE_NONE || WIDE == WIDE_PAIR_ONCE);  // two batch entries sharing bias tiles
    constexpr int NWI = ROWS2 ? 8 : 4;                   // waves that copy one operand image
    constexpr int NIMG = PAIR ? 2 : 1;          // operand images per buffer
    constexpr bool PERSIST = NB == 1 || ROWS2;
    constexpr int DKP = 32 * DK;
    constexpr bool HALF = (FORM & FORM_HALF) != 0;
    auto live_quads = [](int cb) constexpr -> int { return HALF && cb == DK - 1 ? 2 : 4; };  // of a lane, 4 channels each
    constexpr int DK2 = L::DK2;
    constexpr bool F32L = MODE == BIAS_F32_LDS;
    constexpr bool BF16L = MODE == BIAS_BF16_LDS || MODE == BIAS_BF16_LDS8, LDS_BIAS = BF16L || F32L;
    // A chunk can straddle the end of a row.  Where none can, the block loop is built without the code for it (whole calls, us, with /
    // without: N = 392, 640 heads d = 16 63.8 / 62.2, d = 32 68.1 / 66.6, d = 80 95.3 / 94.1, N = 520, 48 heads d = 72 21.4 / 21.2, N = 1376, 96 heads d = 96
    // 100.1 / 98.4).  It is the ragged last block that gains: over long rows either may be ahead by 1 % (N = 4096, 8 heads d = 96 86.2 / 85.3, d = 72 82.1 / 83.1).
    constexpr bool STRADDLE = MODE != BIAS_BF16_LDS8;
    // Staged bias rows: SEGS segments of 128 bytes per row and block.  A bf16 tile is staged whole
    // (two segments); an fp32 tile would be 16 KiB per wave, so its first SEGS 32-key quarters (one per
    // QK tile) are staged and the others go straight into registers, one block ahead: three
    // quarters where two 4-wave workgroups (or one of 8 waves) fit a compute unit's LDS that way.
    constexpr int SEGS = TRI ? 1 : !F32L ? 2 : (NB == 1 && DK == 3) ? 2 : 3;
    constexpr int ESZ = F32L ? 4 : 2, KSEG = 128 / ESZ, EC = 16 / ESZ;  // element size, keys per segment / 16-byte chunk
    constexpr int REGION = SEGS * 4096;  // bytes of a wave's 32-row tile
    static_assert(!F32L || !PAIR, "fp32 tiles are private");
    constexpr bool BIAS_DB = LDS_BIAS && PAIR;  // bias tiles double-buffered and shared
    // The generated biases leave the memory pipeline idle: there the prefetched channel blocks'
    // matrix instructions of a tile are issued right behind its codes and run under the next
    // tile's exponentials (128 x 128 grid, d = 64: 2155 -> 2083 us; nothing or a loss above d = 64).
    // So are those of all channel blocks, whose V rows are read under the tile's own exponentials, in the 4-wave workgroups with bf16
    // tiles at 64 < d <= 96 and fp32 tiles at 32 < d <= 64 (attention stage, us: N = 1024, d = 72, 128 heads 46.1 / 45.8, N = 1370, 64 heads, d = 80
    // 51.3 / 50.8, d = 88 52.4 / 51.1, fp32, N = 577, 192 heads 35.9 / 35.5; bf16 at d = 64 nothing, d = 128 191 / 200, the paired form 2616 / 2838).
    // The single launch is built without (whole calls, without / with: d = 72, N = 256 512 heads 29.2 / 29.0, 768 43.4 / 43.0, N = 128 600 heads 21.9 / 22.1, d = 96,
    // N = 256 768 heads 49.6 / 50.3, fp32, d = 64, N = 256 768 heads 38.0 / 37.5, N = 128 600 heads 20.0 / 20.1): ahead by 1 % with two blocks, behind with one.
    constexpr bool ALL_EARLY = !ONEHEAD && NB == 1 && ((DK == 3 && BF16L) || (DK == 2 && F32L));
    constexpr bool PV_EARLY = ((MODE == BIAS_AXIAL || MODE == BIAS_TABLE_BLK) && DK <= 2) || ALL_EARLY;
    // V operand rows of this many channel blocks are fetched from LDS before the
    // exponential phase (the rest just before their MFMAs): hides the LDS latency
    // where the register budget allows it.
    constexpr int PRE = ALL_EARLY ? DK : TRI ? 0 : (DK == 2 && WAVES3) ? (PV_EARLY ? 1 : 0) : DK <= 2 ? DK : ((DK == 4 && MODE == BIAS_TABLE_BLK) || MODE == BIAS_F32_LDS) ? 0 : 1;
    // ... and at three waves per SIMD each tile's V rows are read under its own exponentials (the
    // registers do not hold them all).
    constexpr bool VDEMAND = (PV_EARLY && WAVES3) || ALL_EARLY;
    // key blocks between two removals of the accumulator's float-bit offset (a power of two)
    constexpr int REBASE = 8;
    __shared__ __attribute__((aligned(1024))) char bufA[NIMG * L::BYTES];
    __shared__ __attribute__((aligned(1024))) char bufB[NIMG * L::BYTES];
    // Staging of the 32 x 128 bias tiles, REGION bytes per 32-row group.
    // NB = 1: one region per wave, private to it.  NB = 2: two buffers shared by the pair.
    __shared__ __attribute__((aligned(1024))) char biasA[LDS_BIAS ? (NB == 2 ? 8 : 4) * REGION : 1024];
    constexpr unsigned BIAS_B = BIAS_DB ? 4 * REGION : 0;  // the second buffer
    // BIAS_AXIAL: the head's two relative-position tables, already divided by alpha.
    //   axu: four copies of the REVERSED x table, copy j shifted by j entries, so that every
    //        lane finds its 16-entry window (ascending with the key index) 16-byte aligned.
    //        Neighbouring queries use copies 3, 2, 1, 0 at one offset, then the next lower
    //        offset: a copy pitch of 16 entries beyond a multiple of 64 puts the 16-byte reads
    //        of 16 consecutive lanes on 16 different bank groups.
    //   axw: the y table (one entry per lane and 16-key tile), behind zeros for the grid rows past the last one that the last
    //        block's keys beyond N would lie in
    constexpr bool AXIAL = MODE == BIAS_AXIAL;
    constexpr int AXL = 2 * AXIAL_MAX_G + 16;  // pitch of a copy, in entries
    constexpr int AXW0 = 8;
    __shared__ __attribute__((aligned(16))) float axu[AXIAL ? 4 * AXL : 4];
    __shared__ float axw[AXIAL ? AXL : 4];
    // BIAS_TABLE / BIAS_TABLE_BLK: rows of the head's (2 Gy - 1) x (2 Gx - 1) table divided by alpha,
    // reversed in x (a lane's 16-entry window then ascends with the key index), at a pitch of
    // 2 Gx entries, in four copies, copy j shifted by j entries as in axu: a window may start at
    // any entry, and its lane reads it with four 16-byte loads from the copy that aligns it
    // (one copy read entry by entry took 64 dword reads per lane and block and was 12 % slower
    // at the 128 x 128 grid, d = 64).  An entry is written to all four copies; the up to three
    // places before a row's first entry that this touches are the unused tail of the row (or
    // copy) before it.
    //   BIAS_TABLE (single-launch forms, Gy * Gx <= 256): the whole table, 4 N - 2 Gx entries.
    //   BIAS_TABLE_BLK: a 128-key block covers 128 / Gx grid rows (or part of one) and so do the
    //   item's 128 queries, so a block needs only the table rows iy - jy in
    //   [iy_lo - jy_hi, iy_hi - jy_lo]: (256 / Gx - 1) rows, or one, i.e. at most 512 entries.
    //   They are double-buffered: the entries for the next block of the stream are loaded at
    //   the start of a block and written to the other buffer at its end.
    constexpr bool TABLE = MODE == BIAS_TABLE, TBLK = MODE == BIAS_TABLE_BLK;
    constexpr int TB_N = TABLE ? 1024 : 512;           // entries of a copy
    constexpr int TB_CP = TB_N + 16;                   // copy pitch (bank spread as for axu)
    constexpr int TB_PER = TB_N / (FUSED_THREADS * NB); // entries a thread stages
    static_assert(!TBLK || (NB == 1 && (WIDE == WIDE_NONE || WAVES3)), "per-block table rows: 4-wave workgroups");
    static_assert(!TABLE || ONEHEAD, "whole table: single-launch forms");
    __shared__ __attribute__((aligned(16))) float tab[TABLE ? 4 * TB_CP : TBLK ? 2 * 4 * TB_CP : 4];
    // BIAS_LUT (no bias): the logit takes only the d + 1 values alpha * I, I = d, d - 2, ..., -d, and
    // the running maximum is one of them, so 255 * exp(S - m) is one of d + 1 numbers that depend
    // on the head alone: lut[k] = 255 * exp(-2 alpha k) for m - I = 2 k.  Entries d + 1 ... 2 d + 1
    // are 0: keys past the end of the sequence are given the "logit" I = -3 d - 2, below every
    // real one and at most 2 d + 1 table steps under any running maximum.  The exponential and
    // its argument disappear from the per-pair work; what remains is one address addition and
    // one LDS read.
    constexpr bool LUT = MODE == BIAS_LUT;
    constexpr int LUTN = 264;
    __shared__ float lut[LUT ? LUTN : 4];
    // delta_v of the current item (two copies: consecutive items alternate)
    __shared__ __attribute__((aligned(16))) float sdelta[2][NIMG][DKP];
    // partial sums of the abs-means of the next item's head (the decomposed bias has no entry point that leaves them).
    // Two copies as well: the waves read one at an item's end, behind its last barrier, and the first wave through may start
    // the copy for the item after the next at once; the block barriers of an item lie between a copy's uses.
    constexpr bool PSUM = PERSIST && !ONEHEAD && !AXIAL;
    static_assert(PSI_MAX_BLOCKS <= 32, "item_mu adds up one pair of sums per lane of half a wave");
    __shared__ __attribute__((aligned(16))) float spsum[2][PSUM ? 2 * PSI_MAX_BLOCKS + 4 : 4];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 3);  // 32-row group
    const int bsel = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);        // half of the workgroup
    const int isel = PAIR ? bsel : 0;                // which resident image / delta copy
    const int wreg = (NB == 2 && !PAIR) ? 4 * bsel + wave : wave;  // this wave's private bias region / copy share
    const int m = lane & 31, g = lane >> 5;
    const int N = p.N, d = p.d;
    // The kernel's arguments, read again from the argument segment where only the switch from one item to the next needs
    // them: carried through the block loop they (and what is computed from them) did not fit the scalar registers, and
    // 16 to 60 v_readlane per block brought them back from vector lanes.  (Attention stage and its preparation, before / after:
    // 128 x 128 grid, d = 64, 32 heads, decomposed 1927 / 1892 us, table 1941 / 1908; N = 2207, d = 96, 96 heads, fp32 bias
    // 353 / 338; N = 1370, d = 80, 64 heads 72.2 / 70.7.)  The forms that compute one item, or hold one head, have the registers.
    // fp32 tiles up to 64 channels are as fast either way where a workgroup has several items, and with few heads
    // slower reading again (carried / again, d = 64, 1 head N = 2600 59.4 / 60.6, N = 4100 85.9 / 87.6, 192 heads N = 577 51.1 / 51.1).
    constexpr bool COLD_ARGS = PERSIST && !ONEHEAD && !(F32L && DK == 2);
    typedef typename std::conditional<COLD_ARGS, const __attribute__((address_space(4))) FusedParams, const FusedParams>::type Args;
    auto args = [&]() -> Args & {
        if constexpr (COLD_ARGS) {
            uint64_t a = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
            asm volatile("" : "+s"(a));  // (opaque: not hoisted, not kept)
            return *(Args *)a;
        } else {
            return p;
        }
    };
    const int bsb = (MODE == BIAS_F32_VEC || F32L) ? 4 : 2;  // bytes per bias element

    // Work item v -> (batch, head, row block).  Consecutive ids go to different XCDs, so v
    // is first turned into (xcd, slot); items that share a bias slab (same head and row
    // block, different batch entry) are neighbours on one XCD and share it through that
    // XCD's L2.  The grid size is a multiple of 8, so a workgroup stays on its XCD.
    struct Item {
        int b, h, rb, bh;
        int valid;
    };
    // (What takes the arguments as `p`: the loop passes args(), the start of the kernel the arguments themselves, which are all
    // fetched at once then.)
    auto decode = [&](int v, auto &p) -> Item {
        Item t;
        const int nbp = p.B / NIMG, per_xcd = (p.total_wg + 7) >> 3, vmax = 8 * per_xcd;
        int u = (v & 7) * per_xcd + (v >> 3), row_block = 0;
        t.valid = v < vmax && u < p.total_wg;
        if (ONEHEAD4 && p.split_from < p.total_wg) {  // heads from split_from on: a workgroup per row block
            u = split_head(v, p.split_from, p.total_wg);
            row_block = split_row_block(v, p.split_from);
            t.valid = u < p.total_wg;
        }
        const int uu = t.valid ? u : 0;
        const int q1 = fast_div(uu, p.div_inner.m, p.div_inner.s), q2 = ONEHEAD ? 0 : fast_div(q1, p.div_rows.m, p.div_rows.s);  // by H; by nbp, then by nrb
        t.b = ONEHEAD ? q1 : (uu - q1 * nbp) * NIMG + isel;
        t.rb = ONEHEAD4 ? row_block : ONEHEAD ? bsel : ROWS2 ? 2 * (q1 - q2 * p.nrb) + bsel : q1 - q2 * p.nrb;
        t.h = ONEHEAD ? uu - q1 * p.H : q2;
        t.bh = t.b * p.H + t.h;
        t.valid = __builtin_amdgcn_readfirstlane(t.valid);
        return t;
    };

    // (row-block pairs have no register left for more of them at once)
    auto first_args = [&]() -> typename std::conditional<ROWS2, Args, const FusedParams>::type & {
        if constexpr (ROWS2) return args();
        else return p;
    };
    int v = blockIdx.x;
    Item cur = decode(v, first_args());
    if (!cur.valid) return;  // uniform over the workgroup

    // ---- per-item state ---------------------------------------------------------
    const char *imgs;  // block image to be copied next
    int q;             // this lane's query row
    float inv_alpha, a2;
    v4i qB[DK2];
    // fp32 tiles' register quarters are loaded before the exponentials of the block before; where the registers do not hold them then
    // (24 bytes per lane were spilled), behind them, and the bias addresses are formed in every block
    constexpr bool BIAS_LATE = F32L && ONEHEAD4 && DK == 3;
    const char *brow = nullptr;  // this lane's bias row (register modes)
    constexpr bool HI_REGS = TRI && BF16L;  // the second half of a bf16 tile goes straight into registers
    constexpr bool BROW_AHEAD = MODE == BIAS_BF16_VEC || HI_REGS || (F32L && !BIAS_LATE);  // ... that of the block loaded next
    // Dense tiles are fetched with full-cache-line requests (8 lanes cover the 128 bytes of one row
    // segment) straight into LDS; which lane fetches what and where it lands: bias_rows.h.
    // A wave copies RGW of the four 8-row groups of its 32-row tile: all four when the
    // tile is its own (NB = 1), two when the tile is shared with the other batch entry.
    constexpr int RGW = PAIR ? 2 : 4;
    const int rg0 = PAIR ? RGW * bsel : 0;  // first row group of the tile this wave copies
    // The copy address is a wave-uniform base (first row of the group and first key of the block to be copied next,
    // scalar registers, advanced by scalar arithmetic) plus a 32-bit lane offset that is fixed for an item.
    struct BiasSrc {
        const char *base[RGW];
        unsigned voff[RGW];
    };
    BiasSrc bsrc;
    int dma_c[RGW];  // key chunk this lane fetches, per row group
#pragma unroll
    for (int j = 0; j < RGW; ++j) {
        bsrc.base[j] = nullptr;
        bsrc.voff[j] = 0;
        dma_c[j] = bias_copy_chunk(rg0 + j, lane);
    }
    int ax_ub = 0, ax_wb = 0;  // BIAS_AXIAL: this lane's window base in axu (floats), its y-table base
    float m_run, l_run, rho;  // running max (units of T = S / alpha), sum of 255 exp(S - m), rescale sum
    int hb_run = 0x7fffffff;  // BIAS_LUT: running minimum of the bit patterns of 1.5 * 2^23 + (d - I)
    float Of[DK][16];         // output carry, channel 32 cb + 8 (r/4) + 4 g + r % 4

    // registers fetched ahead for the NEXT item
    // (sign words; in the single-launch forms the FP4 operand words themselves)
    constexpr int PQ = ONEHEAD ? 4 * DK2 : 2 * DK2;
    unsigned pend_q[PQ];
    __shared__ __attribute__((aligned(16))) unsigned row2_words[TRI ? FUSED_THREADS : 1][TRI ? PQ : 1];  // (three waves per SIMD keep them in LDS)
    unsigned pend_q2[ONEHEAD4 ? PQ : 1];  // ONEHEAD4: this lane's row in the second row block
    float pend_muq = 1.0f, pend_muk = 1.0f;
    auto fetch_item_regs = [&](const Item &t, auto &p) {
        if constexpr (ONEHEAD4) {  // made by the prologue
#pragma unroll
            for (int w = 0; w < PQ; ++w) pend_q[w] = TRI ? row2_words[TRI ? threadIdx.x : 0][w] : pend_q2[w];
            return;
        }
        const int qc = min(t.rb * BR + wave * ROWS_PER_WAVE + m, N - 1), W = (d + 31) / 32;
        const uint32_t *qw = p.q_bits + ((int64_t)t.bh * N + qc) * W;
#pragma unroll
        for (int w = 0; w < 2 * DK2; ++w) pend_q[w] = w < W ? qw[w] : 0u;
        pend_muq = p.mu_q ? p.mu_q[t.bh] : 1.0f;
        pend_muk = p.mu_k ? p.mu_k[t.bh] : 1.0f;
    };
    // The abs-means of an item from the partial sums of its key blocks: one pair per lane, at most PSI_MAX_BLOCKS, in
    // the tree over lanes i, i + 16, i + 8, i + 4, i + 2, i + 1 (the same bits on every run, and those of the tree in
    // v_quant_kernel); exported with the head's first row block.
    struct MuParts {
        float s[2];
    };
    auto mu_parts = [&](const float *ps, auto &p) -> MuParts {
        MuParts o;
        int ln = lane;  // (opaque: no address is kept for this in the block loop)
        asm volatile("" : "+v"(ln));
#pragma unroll
        for (int i = 0; i < 2; ++i) o.s[i] = ln < p.nblk ? ps[2 * ln + i] : 0.0f;
        return o;
    };
    auto item_mu = [&](const Item &t, const MuParts &parts, auto &p) {
        float s[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            s[i] = row_tree_sum(parts.s[i]);
            s[i] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(s[i]))) * p.inv_count;
        }
        if (t.rb == 0 && wave == 0 && lane == 0) {
            if (p.mu_q_out) p.mu_q_out[t.bh] = s[0];
            if (p.mu_k_out) p.mu_k_out[t.bh] = s[1];
        }
        pend_muq = p.use_mu ? s[0] : 1.0f;
        pend_muk = p.use_mu ? s[1] : 1.0f;
    };
    // bias pointers of an item (no memory access)
    auto bias_row_ptr = [&](const Item &t, auto &p) -> const char * {
        int ln = lane;
        if (TRI) asm volatile("" : "+v"(ln));  // (opaque: the second row block's addresses are formed where it starts)
        const int qc = min(t.rb * BR + wave * ROWS_PER_WAVE + (ln & 31), N - 1);
        return static_cast<const char *>(p.bias) +
               ((int64_t)t.b * p.bs.b + (int64_t)t.h * p.bs.h + (int64_t)qc * p.bs.n) * bsb;
    };
    auto bias_dma_src = [&](const Item &t, auto &p) -> BiasSrc {
        BiasSrc o;
        int ln = lane;
        if (TRI) asm volatile("" : "+v"(ln));
#pragma unroll
        for (int j = 0; j < RGW; ++j) {
            const int rg = rg0 + j;
            const int row0 = bias_group_row(t.rb * BR + wave * ROWS_PER_WAVE, rg, N);  // uniform
            const int row = bias_copy_row(row0, rg, ln, N);
            o.base[j] = uniform_ptr(static_cast<const char *>(p.bias) +
                                    ((int64_t)t.b * p.bs.b + (int64_t)t.h * p.bs.h + (int64_t)row0 * p.bs.n) * ESZ);
            o.voff[j] = (unsigned)(row - row0) * (unsigned)p.bs.n * (unsigned)ESZ + 16u * (TRI ? bias_copy_chunk(rg, ln) : dma_c[j]);
        }
        return o;
    };
    auto image_ptr = [&](const Item &t, auto &p) -> const char * {
        return uniform_ptr(p.img + (int64_t)t.bh * p.nblk * L::BYTES);
    };
    // ---- BIAS_TABLE / BIAS_TABLE_BLK: staging of table rows from row0 on -------------
    // (Clipping the rows of every block against the grid, and a tile's window against its rows, took 105 scalar and 29 vector
    // instructions per block, now 25 and 17.  Attention stage, us: table, 128 x 128, d = 64, 32 heads 1840 / 1774, 32 x 32, d = 72, 128 heads
    // 45.6 / 43.5; decomposed, where the same holds of the tables' windows, 1820 / 1782.)
    // Entry kk of reversed row r is a lane's i = r (2 Gx) + kk.  The loads go through a buffer descriptor that ends with the head's
    // table: places that hold no entry (rows outside the table, the place behind a row) read as zero or as a neighbour, and only
    // keys past the end of the sequence, whose logits are replaced, see them.  So a block takes one number, row0 LX.
    float tstage[TABLE || TBLK ? TB_PER : 1];
    __amdgpu_buffer_rsrc_t trsrc;
    unsigned tvoff[TABLE || TBLK ? TB_PER : 1];
    auto table_place = [&](int i) -> int {  // table entry of stage entry i, from the first row's first on
        const int LX = 2 * p.Gx - 1, sh = p.gx_shift + 1;
        return (i >> sh) * LX + LX - 1 - (i & ((1 << sh) - 1));
    };
    auto table_begin = [&](const Item &t, auto &p) {
        const int LX = 2 * p.Gx - 1, LY = 2 * p.Gy - 1;
        trsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(uniform_ptr(p.table + (int64_t)t.h * LY * LX)), 0, 4 * LY * LX, 0x00020000);
#pragma unroll
        for (int j = 0; j < TB_PER; ++j) tvoff[j] = 4u * (unsigned)table_place(64 * (4 * bsel + wave) + lane + j * FUSED_THREADS * NB);
    };
    auto table_load = [&](int row0) {  // global loads only
        if (DK == 4) {  // (formed here: no registers to carry them)
            int tid = 64 * (4 * bsel + wave) + lane;
            asm volatile("" : "+v"(tid));
#pragma unroll
            for (int j = 0; j < TB_PER; ++j) tvoff[j] = 4u * (unsigned)table_place(tid + j * FUSED_THREADS * NB);
        }
        const unsigned o = 4u * (unsigned)(row0 * (2 * p.Gx - 1));
#pragma unroll
        for (int j = 0; j < TB_PER; ++j)
            tstage[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(trsrc, tvoff[j] + o, 0, 0));
    };
    auto table_store = [&](float *dst, float ia) {
#pragma unroll
        for (int j = 0; j < TB_PER; ++j) {
            const int i = 64 * (4 * bsel + wave) + lane + j * FUSED_THREADS * NB;
            if (TBLK && j > 0 && p.Gx == 128) break;  // one row of 256 entries (the other grids need more than half)
            const float x = tstage[j] * ia;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                dst[c * TB_CP + i - c] = x;
        }
    };
    // BIAS_TABLE_BLK: the rows of one (row block, key block): row 0 is that of the first query row and the last key row
    auto tblk_load = [&](int rb, int blk) {
        table_load(((rb * BR) >> p.gx_shift) + p.Gy - 1 - ((blk * BV + BV - 1) >> p.gx_shift));
    };
    // turn the fetched registers into the item's state
    // (same_head: the head's tables are in LDS already)
    auto begin_item = [&](const Item &t, auto same_head, auto &p) {
        constexpr bool SAME_HEAD = decltype(same_head)::value;
        q = t.rb * BR + wave * ROWS_PER_WAVE + m;
        // Logit multiplier alpha of Eq. 6.  Its sign goes into the Q operand and a vanishing
        // alpha clears the Q operand, so that the loop can assume alpha > 0.
        const float alpha = p.scale * pend_muq * pend_muk;
        const bool a_zero = fabsf(alpha) < 1e-30f;
        const bool a_neg = alpha < 0.0f;
        const float a_abs = a_zero ? 1.0f : fabsf(alpha);
        inv_alpha = 1.0f / a_abs;
        a2 = a_abs * LOG2E_F;  // exponent multiplier in base 2
        // (BIAS_LUT lets the matrix core SUBTRACT the logit from a constant, see the block loop)
        if constexpr (ONEHEAD) {
#pragma unroll
            for (int i = 0; i < PQ; ++i)
                qB[i / 4][i % 4] = a_zero ? 0 : (int)(pend_q[i] ^ ((LUT ? !a_neg : a_neg) && pend_q[i] ? 0x88888888u : 0u));
        } else {
            load_q_operand<DK2>(pend_q, d, g, LUT ? !a_neg : a_neg, a_zero, qB);
        }
        if (LUT && !SAME_HEAD) {
            // (the previous item's last block is behind every wave; the barrier publishes the table)
            for (int i = threadIdx.x; i < LUTN; i += FUSED_THREADS * NB)
                lut[i] = i <= d ? __builtin_amdgcn_exp2f(fmaf(-2.0f * (float)i, a2, LOG2_255_F)) : 0.0f;
            __syncthreads();
        }
        if (LUT) hb_run = 0x7fffffff;
        if (MODE == BIAS_F32_VEC || BIAS_LATE) brow = bias_row_ptr(t, p);
        if (AXIAL && !SAME_HEAD) {
            // every wave is past the previous item's last block (begin_item follows its closing
            // barrier), so the tables can be overwritten; a barrier publishes the new ones
            const int LX = 2 * p.Gx - 1, LY = 2 * p.Gy - 1;
            const float *ux = p.ax_x + (int64_t)t.h * LX, *wy = p.ax_y + (int64_t)t.h * LY;
            // (all loads of a thread go out before the first LDS write: one memory latency)
            constexpr int NTA = FUSED_THREADS * NB;
            constexpr int NU = (4 * AXL + NTA - 1) / NTA, NW = (AXL + NTA - 1) / NTA;
            float tu[NU], tw[NW];
            int tid = 64 * (4 * bsel + wave) + lane;  // (opaque: keeps the index arithmetic out of the block loop's registers)
            asm volatile("" : "+v"(tid));
#pragma unroll
            for (int j = 0; j < NU; ++j) {
                const int i = tid + j * NTA;
                const int kk = (i % AXL) + (i / AXL);  // index into the reversed table
                const bool on = i < 4 * AXL && kk < LX;
                tu[j] = ux[on ? LX - 1 - kk : 0];
                if (!on) tu[j] = 0.0f;
            }
#pragma unroll
            for (int j = 0; j < NW; ++j) {
                const int i = tid + j * NTA;
                const bool on = i >= AXW0 && i < LY + AXW0;
                tw[j] = wy[on ? i - AXW0 : 0];
                if (!on) tw[j] = 0.0f;
            }
#pragma unroll
            for (int j = 0; j < NU; ++j) {
                const int i = tid + j * NTA;
                if (i < 4 * AXL) axu[i] = tu[j] * inv_alpha;
            }
#pragma unroll
            for (int j = 0; j < NW; ++j) {
                const int i = tid + j * NTA;
                if (i < AXL) axw[i] = tw[j] * inv_alpha;
            }
            // vmcnt(0), in the form the compiler counts: some lanes use none of the last loads, and it would wait for those, and
            // with them for the copies just started, at the top of every block (64 x 64 grid, 1 head d = 32 59.3 -> 50.4 us, d = 64
            // 61.1 -> 56.2; 128 x 128 grid, d = 64, 32 heads 1923 -> 1866)
            __builtin_amdgcn_s_waitcnt(0x0F70);
            __syncthreads();
        }
        if (AXIAL) {
            const int qc = min(q, N - 1);
            const int ix = qc & (p.Gx - 1), iy = qc >> p.gx_shift;
            const int s0 = p.Gx - 1 - ix;  // reversed-table index of key column 0
            ax_ub = (s0 & 3) * AXL + (s0 & ~3) + ((16 * g) & (p.Gx - 1));
            ax_wb = iy + p.Gy - 1 + AXW0 - (p.Gx == 16 ? g : 0);
        }
        if (TABLE && !SAME_HEAD) {
            // (as above: the previous item's last block is behind every wave)
            table_begin(t, p);
            table_load(0);
            table_store(tab, inv_alpha);
            __syncthreads();
        }
        if (TABLE) {
            const int qc = min(q, N - 1);
            const int s0 = p.Gx - 1 - (qc & (p.Gx - 1));  // reversed-row index of key column 0
            ax_ub = (s0 & 3) * TB_CP + (s0 & ~3) + (((qc >> p.gx_shift) + p.Gy - 1) << (p.gx_shift + 1));
        }
        if (TBLK) {
            const int qc = min(q, N - 1);
            const int s0 = p.Gx - 1 - (qc & (p.Gx - 1));  // reversed-row index of key column 0
            // ... of the row of a block's last keys (row 0 of the staged rows: iy = iy_lo, jy = jy_hi), plus the step from a 32-key
            // tile's first 16 keys to its last, which is the same in all tiles
            ax_ub = (s0 & 3) * TB_CP + (s0 & ~3) + (((qc >> p.gx_shift) - ((t.rb * BR) >> p.gx_shift)) << (p.gx_shift + 1)) +
                    g * (p.Gx == 16 ? -2 * 16 : 16);
        }
        m_run = -INFINITY;
        l_run = 0.0f;
        rho = 0.0f;
#pragma unroll
        for (int cb = 0; cb < DK; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r) Of[cb][r] = 0.0f;
    };

    // ---- bias access ----------------------------------------------------------
    // The copies' source may start at any element: they take 2-byte-aligned addresses like ordinary
    // loads do.  A chunk that would read behind the tensor's last element is left out and written
    // element by element (bias_tail).
    auto bias_klimit = [&](const Item &t, int blk) -> int {
        if (blk * BV + BV <= N) return N;
        Args &p = args();
        return bias_key_limit((int64_t)t.b * p.bs.b + (int64_t)t.h * p.bs.h, t.rb * BR + wave * ROWS_PER_WAVE, N, p.bs.n,
                              p.bias_end, blk * BV, EC);
    };
    auto bias_tail = [&](const Item &t, int blk, unsigned region) {
        typedef typename std::conditional<F32L, uint32_t, uint16_t>::type elem;
        Args &p = args();
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int rg = ln >> 3, k0 = (N & -EC) - blk * BV;  // the chunk's first key inside the block
        if (rg < rg0 || rg >= rg0 + RGW || k0 >= SEGS * KSEG) return;
        const int row = min(t.rb * BR + wave * ROWS_PER_WAVE + ln, N - 1);
        const elem *src = static_cast<const elem *>(p.bias) + (int64_t)t.b * p.bs.b + (int64_t)t.h * p.bs.h +
                          (int64_t)row * p.bs.n + (N & -EC);
        const unsigned dst = region + bias_lds_chunk(ln, k0 / KSEG, k0 / EC & 7, SEGS);
#pragma unroll 1
        for (int i = 0; i < (N & (EC - 1)); ++i)
            *reinterpret_cast<__attribute__((address_space(3))) elem *>((size_t)(dst + ESZ * i)) = src[i];
    };
    auto dma_bias_one = [&](const BiasSrc &src, int blk, int klim, unsigned region, int idx) {  // copy idx = SEGS j + segment
        const int j = idx / SEGS, seg = idx % SEGS;
        int ln = lane;
        if (TRI) asm volatile("" : "+v"(ln));
        const int key0 = blk * BV + KSEG * seg + EC * (TRI ? bias_copy_chunk(rg0 + j, ln) : dma_c[j]);
        if (key0 < klim)
            dma16<WIDE == WIDE_PAIR_ONCE>(src.base[j] + 128 * seg, src.voff[j], region + ((rg0 + j) * SEGS + seg) * 1024);
    };
    // block blk of item t into the LDS offset `region`; src is at that block and moves on to the next.  Blocks that end inside
    // the row, all but the last, need no look at any lane's keys: eight lane masks, branches and 64-bit addresses per block
    // held the wave as long as its vector work did (190 scalar instructions per block; with them and those of the switch of items
    // gone from the ordinary block, attention stage, before / after, us: N = 1024, d = 72, 128 heads 51.9 / 48.5, N = 1370, d = 80, 64
    // heads 58.4 / 52.6, fp32 bias, N = 577, d = 64, 192 heads 39.9 / 36.1, N = 2048, d = 128, 128 heads 213.5 / 195.6).
    // `ends`: where the caller's code knows it, and the other copy routine is left out of it.  The single launch runs through its
    // code once, cold, and pays for its length.  Its first tile takes the ragged routine whatever its length (us, both / so: bf16, 300 heads
    // d = 32, N = 50 9.62 / 9.37, d = 64, N = 50 11.85 / 11.43, d = 96, N = 100 15.9 / 15.7, 360 heads d = 96, N = 128 16.1 / 16.3).  The second block of
    // the short forms is ragged, the first block of a second row block whole.  N > 224 has both (N = 256, 384 heads, one / both: fp32, d = 32
    // 18.4 / 17.7, d = 64 25.2 / 24.2, bf16, d = 64 23.5 / 23.1).
    constexpr int ENDS_INSIDE = 1, ENDS_RAGGED = 2;
    auto dma_bias = [&](const Item &t, BiasSrc &src, int blk, unsigned region, int ends) {
        if constexpr (!PAIR) {
            if (ends ? ends == ENDS_INSIDE : blk * BV + BV <= N) {
                dma_tile<SEGS>(src.base, src.voff, region);
            } else {
                const int klim = STRADDLE ? bias_klimit(t, blk) : N;
                if (STRADDLE && klim != N) bias_tail(t, blk, region);
#pragma unroll
                for (int idx = 0; idx < SEGS * RGW; ++idx) dma_bias_one(src, blk, klim, region, idx);
            }
        } else {
            const int klim = STRADDLE ? bias_klimit(t, blk) : N;
            if (STRADDLE && klim != N) bias_tail(t, blk, region);
#pragma unroll
            for (int idx = 0; idx < SEGS * RGW; ++idx) dma_bias_one(src, blk, klim, region, idx);
        }
#pragma unroll
        for (int j = 0; j < RGW; ++j) src.base[j] += BV * ESZ;
    };
    f4v fraw[F32L ? SEGS : 1][4];      // F32L: the staged quarters of the current block
    f4v freg[F32L ? 4 - SEGS : 1][4];  // F32L: this lane's values of the quarters that are not staged
    auto load_bias_quarters = [&](const char *row, int blk) {
        const float *src = reinterpret_cast<const float *>(row) + blk * BV + 16 * g;
#pragma unroll
        for (int t = SEGS; t < KT; ++t) {
            if (blk * BV + 32 * t + 32 <= N) {
#pragma unroll
                for (int i = 0; i < 4; ++i) freg[t - SEGS][i] = *reinterpret_cast<const f4v_a4 *>(src + 32 * t + 4 * i);
            } else if (blk * BV + 32 * t < N) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int o = 32 * t + 4 * i + j;
                        freg[t - SEGS][i][j] = blk * BV + 16 * g + o < N ? src[o] : 0.0f;
                    }
            }
        }
    };
    u4v braw[8];  // the 64 bf16 bias values of this lane for the current block
    auto load_bias_vec = [&](const char *row, int blk) {  // BIAS_BF16_VEC: registers straight from global memory
        const int k0 = blk * BV + 16 * g;
        const uint16_t *src = reinterpret_cast<const uint16_t *>(row) + k0;
        if (blk * BV + BV <= N) {
#pragma unroll
            for (int i = 0; i < 8; ++i) braw[i] = *reinterpret_cast<const u4v_a2 *>(src + 32 * (i >> 1) + 8 * (i & 1));
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int o = 32 * (i >> 1) + 8 * (i & 1);
                if (k0 + o + 8 <= N) {
                    braw[i] = *reinterpret_cast<const u4v_a2 *>(src + o);
                } else {
                    unsigned e[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) e[j] = (k0 + o + j < N) ? src[o + j] : 0u;
                    braw[i] = u4v{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16),
                                  e[6] | (e[7] << 16)};
                }
            }
        }
    };
    // HI_REGS: this lane's values of keys 64 .. 127 of a block.  Chunks may read on behind a row's end, but not behind the tensor's.
    auto load_bias_hi = [&](const char *row, int blk) {
        const uint16_t *src = reinterpret_cast<const uint16_t *>(row) + blk * BV + 16 * g;
        const uint16_t *end = static_cast<const uint16_t *>(p.bias) + p.bias_end;
#pragma unroll
        for (int i = 4; i < 8; ++i) {
            if (blk * BV + 32 * (i >> 1) >= N) continue;  // (uniform)
            const int o = 32 * (i >> 1) + 8 * (i & 1);
            if (src + o + 8 <= end) {
                braw[i] = *reinterpret_cast<const u4v_a2 *>(src + o);
            } else {
                const uint16_t *s2 = src + o;
                asm volatile("" : "+v"(s2));  // (opaque: nothing of this rare way is kept in registers)
                unsigned e[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) e[j] = s2 + j < end ? s2[j] : 0u;
                braw[i] = u4v{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
            }
        }
    };
    // accumulator input of QK tile t: bias / alpha for keys blk*BV + 32 t + 16 g + [0, 16)
    auto bias_tile = [&](int blk, int t) -> v16f {
        const int k0 = blk * BV + 32 * t + 16 * g;
        v16f bt;
        if (MODE == BIAS_NONE) {
#pragma unroll
            for (int r = 0; r < 16; ++r) bt[r] = 0.0f;
        } else if (MODE == BIAS_BF16_VEC || BF16L) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const u4v w = braw[2 * t + i];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    bt[8 * i + 2 * j] = bf16_lo(w[j]) * inv_alpha;
                    bt[8 * i + 2 * j + 1] = bf16_hi(w[j]) * inv_alpha;
                }
            }
        } else if (F32L) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f4v w = t < SEGS ? fraw[t < SEGS ? t : 0][i] : freg[t < SEGS ? 0 : t - SEGS][i];
#pragma unroll
                for (int j = 0; j < 4; ++j) bt[4 * i + j] = w[j] * inv_alpha;
            }
        } else {  // BIAS_F32_VEC: 16-byte loads at float alignment, guarded at the row end
            const float *src = reinterpret_cast<const float *>(brow) + k0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (k0 + 4 * i + 4 <= N) {
                    const f4v w = *reinterpret_cast<const f4v_a4 *>(src + 4 * i);
#pragma unroll
                    for (int j = 0; j < 4; ++j) bt[4 * i + j] = w[j] * inv_alpha;
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        bt[4 * i + j] = (k0 + 4 * i + j < N) ? src[4 * i + j] * inv_alpha : 0.0f;
                }
            }
        }
        return bt;
    };

    // ---- epilogue of an item: (O - magic * rho) / (255 l) * delta_v, bf16 store ----
    // A lane holds 4 consecutive channels per (cb, q4) and its partner lane ^ 32 the next 4.
    // One permlane32 swap per dword regroups two such quads so that the lower lane owns 8
    // consecutive channels of quad 2k and the upper lane those of quad 2k + 1: 16-byte stores.
    auto finish_item = [&](const Item &t, const float *dl) {
        Args &p = args();
        const float l_tot = pair_sum(l_run);
        const float inv = 1.0f / l_tot;
        const float off = PV_MAGIC_F * rho;
        uint16_t *orow = p.out + (int64_t)t.b * p.os.b + (int64_t)t.h * p.os.h + (int64_t)min(q, N - 1) * p.os.n;
#pragma unroll
        for (int cb = 0; cb < DK; ++cb)
#pragma unroll
            for (int k = 0; k < live_quads(cb) / 2; ++k) {
                unsigned w[2][2];  // [quad 2k / 2k+1][dword]
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int q4 = 2 * k + e;
                    const float4 d4 = *reinterpret_cast<const float4 *>(dl + 32 * cb + 8 * q4 + 4 * g);
                    w[e][0] = pack_bf16x2((Of[cb][4 * q4 + 0] - off) * inv * d4.x,
                                          (Of[cb][4 * q4 + 1] - off) * inv * d4.y);
                    w[e][1] = pack_bf16x2((Of[cb][4 * q4 + 2] - off) * inv * d4.z,
                                          (Of[cb][4 * q4 + 3] - off) * inv * d4.w);
                }
                // lower lanes: {own quad 2k, partner's quad 2k}; upper: {partner's 2k+1, own 2k+1}
                const auto s0 = __builtin_amdgcn_permlane32_swap(w[0][0], w[1][0], false, false);
                const auto s1 = __builtin_amdgcn_permlane32_swap(w[0][1], w[1][1], false, false);
                const int c = 32 * cb + 16 * k + 8 * g;  // first of this lane's 8 channels
                if (q < N && c < d)
                    *reinterpret_cast<u4v *>(orow + c) = u4v{s0[0], s1[0], s0[1], s1[1]};
            }
    };

    // Where this lane reads its tile row: chunk c of the row sits at row + 16 (c ^ (m & 7)) = (row + 16 (m & 7)) ^ 16 c (rows are
    // 128-byte aligned).  Four addresses, which stay in registers: forming them in every block took 14 instructions.
    // (fp32 tiles above 64 channels have no registers left for them.)
    const char *bA = biasA + wreg * REGION;
    constexpr bool BADDR_LATE = F32L && DK == 3;
    unsigned baddr[LDS_BIAS ? 4 : 1];
    auto bias_addresses = [&](int ln) {
        const int mm = ln & 31, gg = ln >> 5;
        const unsigned row = lds_offset(bA) + (mm >> 3) * (SEGS * 1024) + 128 * ((mm & 7) ^ ((mm >> 3) & 1));
#pragma unroll
        for (int i = 0; i < 4; ++i)  // F32L: chunks 4 g + i of a segment; else chunks 2 g, 2 g + 1 of either 32-key half of it
            baddr[i] = (row + 16 * ((mm & 7) ^ (F32L ? 4 * gg : 2 * gg))) ^ (F32L ? 16u * i : 16u * (4 * (i >> 1) + (i & 1)));
    };
    if (LDS_BIAS && !BADDR_LATE) bias_addresses(lane);

    // The persistent forms end inside the loop: a way out of it to the function's end leaves ten moves between scalar registers (and
    // as many through vector registers) in every block.  (Attention stage, us: N = 1024, d = 72, 128 heads 48.4 / 47.2, N = 1370, d = 80, 64
    // heads 52.4 / 51.4, fp32 bias, N = 577, d = 64, 192 heads 36.1 / 35.7.  Where registers are at their limit it spills one.  Above 64
    // channels fp32 tiles lose by it, whole calls, us, way out / so: d = 96 N = 10000 4 heads 444 / 455, N = 2207 32 heads 169.8 / 172.9, N = 6000 1 head
    // 131.7 / 135.7, d = 80 N = 1370 64 heads 80.9 / 81.9.)
    constexpr bool ENDS = PERSIST && !WAVES3 && DK < 4 && !(F32L && DK == 3);
    // ---- stream position --------------------------------------------------------
    int it = 0;        // key block inside the current item
    // 8-wave single launch (up to 128 tokens leave half of its waves without rows): a wave whose 32 rows all lie beyond N
    // only copies.  12 heads, N = 125 11.0 -> 10.4 us; the branch around the block costs the other forms 1-3 %.
    const bool live = !(ONEHEAD && NB == 2) || cur.rb * BR + wave * ROWS_PER_WAVE < N;
    // (Flags of the loop are integers in scalar registers that the compiler cannot look into: it makes lane masks out of them
    // otherwise, five to ten instructions per block for each.)
    int younger = 0;
    if constexpr (NB == 1 && !ONEHEAD) {
        const int flag = WAVES3 && gridDim.x > 512 ? 3 * blockIdx.x >= 2 * gridDim.x : 2 * blockIdx.x >= gridDim.x;
        younger = __builtin_amdgcn_readfirstlane(flag);
        asm volatile("" : "+s"(younger));
    }
    int parity = 0;    // items alternate between the two delta_v copies
    Item nxt = {0, 0, 0, 0, false};
    if (ONEHEAD4) {  // a head's two row blocks, one workgroup
        nxt = cur;
        nxt.rb = 1;
        nxt.valid = p.nrb > 1 && (p.split_from == p.total_wg || v < p.split_from);
    } else if (PERSIST) {
        nxt = decode(v + gridDim.x, first_args());
    }

    // (-infinity that the compiler cannot see: a maximum of two matrix results alone first quiets both, two instructions more)
    float ninf = -INFINITY;
    if (AXIAL) asm volatile("" : "+s"(ninf));
    // The block before which the accumulator's offset is next removed (see the loop).  A 4-wave item that
    // starts on buffer B (an odd number of blocks per item, after an odd number of items) is rebased before
    // blocks 9, 17, ... instead of 8, 16, ...: which it is shows in the last bits of the carry.  The grid of
    // three workgroups per compute unit deals items out differently, and the 8-wave forms deal out pairs of
    // them: they follow the grid of 512, where the item with index u is the (u % per / 64)-th of its
    // workgroup, so that a row block has the same bits whichever form serves it.  (Rows of whole 16-byte chunks,
    // which the 8-wave forms have always served, keep those forms' own order.)
    constexpr bool PHASE = WAVES3 || PAIR || ROWS2;
    auto first_rebase = [&]() -> int {
        if (!PHASE) return 0;
        Args &p = args();
        if (WAVES3) return REBASE + ((v >> 9) & p.nblk & 1);
        if (!p.phase512) return REBASE + (ROWS2 ? (v >> 8) & p.nblk & 1 : 0);
        const int nrb1 = (N + BR - 1) / BR, per = (p.B * p.H * nrb1 + 7) >> 3;
        const int u = (cur.h * nrb1 + min(cur.rb, nrb1 - 1)) * p.B + cur.b;
        return REBASE + (((u % per) >> 6) & p.nblk & 1);
    };
    int next_rebase = PAIR ? 0 : first_rebase();

    // Copies of an item's small data, outside the block loop: delta_v of the item that starts (for its epilogue), and the partial
    // sums of the abs-means of the item after it (for item_mu).  Its first block's end waits for them.
    auto copy_item_data = [&](auto &p) {
        if (ONEHEAD || (ROWS2 ? wreg : wave) != 0) return;
        if (lane < DKP / 4) dma16(p.delta + (int64_t)cur.bh * DKP, 16 * lane, lds_offset(&sdelta[parity][isel][0]));
        if (PSUM && p.psum && nxt.valid && 2 * lane < p.nblk)
            dma16(p.psum + (int64_t)nxt.bh * p.nblk * 2, 16 * lane, lds_offset(&spsum[parity][0]));
    };

    constexpr bool FETCH_AFTER = MODE == BIAS_BF16_VEC && DK == 4;  // (spills 84 bytes otherwise)
    // One key/value block of the stream: compute block `it` of item `cur` from the image at
    // `ibuf` (and bias tile `bcur` bytes behind the first), prefetch the next block of the stream into the LDS
    // offsets `inxt` / `bnxt`.  Returns false after the last block of the last item.
    auto step = [&](const char *ibuf, unsigned inxt, unsigned bcur, unsigned bnxt, int tpar) -> bool {
        // 0. start the copies for the next block of the stream
        int nblkidx = it + 1;  // its number in its item
        int more = PERSIST ? 1 : p.nblk - nblkidx;  // not 0: the stream goes on
        if (__builtin_expect(nblkidx == p.nblk, 0)) {  // the last block of this item: the next one belongs to the next item
            if (PERSIST) more = nxt.valid;
            nblkidx = 0;
            if (PERSIST && more) {
                if (!ONEHEAD) imgs = image_ptr(nxt, args());
                if (!FETCH_AFTER) fetch_item_regs(nxt, args());
                if (LDS_BIAS && !BIAS_DB && !BIAS_LATE) bsrc = bias_dma_src(nxt, args());
                if (BROW_AHEAD) brow = bias_row_ptr(nxt, args());
            }
        }
        if (!ONEHEAD && !ROWS2) asm volatile("" : "+s"(more));
        if (!ONEHEAD && PERSIST && !ROWS2) asm volatile("" : "+s"(nblkidx));
        const bool sw = PERSIST && nblkidx == 0;
        if (!ONEHEAD && more) {
            dma_image<DK, NWI>(imgs, inxt + isel * L::BYTES, ROWS2 ? wreg : wave, lane);
            imgs += L::BYTES;
        }
        if (BIAS_LATE && more) {
            bsrc = bias_dma_src(sw ? nxt : cur, args());
#pragma unroll
            for (int j = 0; j < RGW; ++j) bsrc.base[j] += nblkidx * (BV * ESZ);
        }
        if (FETCH_AFTER && sw && more) fetch_item_regs(nxt, args());
        int nklim = N;  // key limit of the shared bias tile's copies below
        const bool whole = nblkidx * BV + BV <= N;
        if (BIAS_DB && more && !whole) {
            nklim = bias_klimit(cur, nblkidx);
            if (nklim != N) bias_tail(cur, nblkidx, bnxt);
        }
        if (TBLK && more) {  // land during this block, stored at its end
            if (sw) table_begin(nxt, args());
            tblk_load(sw ? nxt.rb : cur.rb, nblkidx);
        }

        // Two 4-wave workgroups share a CU, and the SIMDs issue the older wave first: the
        // workgroup dispatched first then runs ~25 % faster than the other and leaves the CU
        // half empty at the end.  The second half of the grid (dispatched after every CU has
        // its first workgroup) therefore raises its priority on every other block.  Only a
        // scheduling hint: results do not depend on it.  With three workgroups per CU the last third does
        // (128 x 128 grid, d = 64: table 1968 us with the second half, 1912 with the last third, 2143 without).
        // The single launch has at most two blocks an item: one of at most 128 keys has nothing to raise, and the flag formed for it cost
        // 0.1 .. 0.6 us (us, with / without: d = 64, bf16, N = 128 896 heads 24.4 / 23.9, N = 100 768 heads 20.0 / 19.5).  The second block is raised where
        // all of it counts (N > 224; us, never raised / so: d = 32, fp32 N = 240 260 heads 20.4 / 19.2, d = 64 24.2 / 22.9, d = 96, N = 256 384 heads
        // 34.4 / 33.8); where it ends early, and with three workgroups per unit, it goes either way (N = 197, no bias, d = 32 500 heads 13.9 / 13.6,
        // 768 18.6 / 18.9, fp32, d = 64 768 heads 37.7 / 38.1).
        if constexpr (NB == 1 && !ONEHEAD) {
            if (!tpar) __builtin_amdgcn_s_setprio(0);
            else if (younger) __builtin_amdgcn_s_setprio(1);
        } else if constexpr (ONEHEAD4 && !SHORT && !TRI) {
            if (!tpar) __builtin_amdgcn_s_setprio(0);
            else if (2 * blockIdx.x >= gridDim.x) __builtin_amdgcn_s_setprio(1);
        }
        // WIDE_SHORT: tile t of the second block holds no key (its weights are 0, code -128)
        auto dead_tile = [&](int t) -> bool { return SHORT && tpar == 1 && t > 0 && BV + 32 * t >= N; };
        if ((live && (!(SHORT && ONEHEAD4) || cur.rb * BR + wave * ROWS_PER_WAVE < N))) {
        // 1. all LDS reads of the logit phase go out together: bias tile, key rows
        if (LDS_BIAS) {
            if (BADDR_LATE) {
                int ln = lane;  // (opaque: the addresses are formed here)
                asm volatile("" : "+v"(ln));
                bias_addresses(ln);
            }
            if (F32L) {
#pragma unroll
                for (int t = 0; t < SEGS; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        fraw[t][i] = *reinterpret_cast<const __attribute__((address_space(3))) f4v *>((size_t)(baddr[i] + 1024u * t));
            } else {
#pragma unroll
                for (int i = 0; i < (HI_REGS ? 4 : 8); ++i)  // chunk 2 gg + 4 (t & 1) + i % 2 of the 64-key half t / 2, t = i / 2
                    braw[i] = *reinterpret_cast<const __attribute__((address_space(3))) u4v *>((size_t)(baddr[2 * ((i >> 1) & 1) + (i & 1)] + bcur + 1024u * (i >> 2)));
            }
        }
        v4i ka[KT][DK2];
        int kln = lane;
        if (DK == 4 && (TBLK || LUT)) asm volatile("" : "+v"(kln));  // (addresses formed here: carried, they were spilled)
#pragma unroll
        for (int t = 0; t < KT; ++t) load_k_operand<DK>(ibuf, t, kln & 31, kln >> 5, ka[t]);
        __builtin_amdgcn_sched_barrier(0);  // all of them in flight before the first use
        //    T = I + b / alpha
        v16f T[KT];
        float wt[KT];  // BIAS_AXIAL: the y term of tile t (constant over its 16 keys), else 0
        if (AXIAL) {
            // A block starts on a grid row up to Gx = 128, so a tile's place in it does not depend on the block (Gx = 256: two blocks
            // to a row); the first keys' places are in the lane's bases.
            const int xb = (it * BV) & (p.Gx - 1), yb = (it * BV) >> p.gx_shift;
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                const float *win = axu + ax_ub + xb + ((32 * t) & (p.Gx - 1));
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const f4v x = *reinterpret_cast<const f4v *>(win + 4 * i);
                    T[t][4 * i] = x[0]; T[t][4 * i + 1] = x[1]; T[t][4 * i + 2] = x[2]; T[t][4 * i + 3] = x[3];
                }
                wt[t] = axw[ax_wb - yb - ((32 * t) >> p.gx_shift)];
            }
#pragma unroll
            for (int t = 0; t < KT; ++t) T[t] = qk_mfma<DK2>(ka[t], qB, T[t]);
        } else if (TABLE || TBLK) {
            // Windows of 16 keys of one grid row (16 <= Gx).  A block starts on a grid row up to Gx = 128, so a tile's place in the
            // staged rows does not depend on the block (Gx = 256: two blocks to a row).
            const float *tcur = tab + (TBLK ? tpar * 4 * TB_CP : 0) + ax_ub + (TBLK ? (it * BV) & (p.Gx - 1) : 0);
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                int o0, o1;
                if (TBLK) {
                    o0 = o1 = ((32 * t) & (p.Gx - 1)) + (((BV - 1) >> p.gx_shift) - ((32 * t) >> p.gx_shift)) * (2 * p.Gx);
                } else {
                    auto window = [&](int key0) { return (key0 & (p.Gx - 1)) - min(key0 >> p.gx_shift, p.Gy - 1) * (2 * p.Gx); };
                    o0 = window(it * BV + 32 * t), o1 = window(it * BV + 32 * t + 16);
                }
                const float *win = tcur + (TBLK ? o0 : g ? o1 : o0);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const f4v x = *reinterpret_cast<const f4v *>(win + 4 * i);
                    T[t][4 * i] = x[0]; T[t][4 * i + 1] = x[1]; T[t][4 * i + 2] = x[2]; T[t][4 * i + 3] = x[3];
                }
                wt[t] = 0.0f;
            }
#pragma unroll
            for (int t = 0; t < KT; ++t) T[t] = qk_mfma<DK2>(ka[t], qB, T[t]);
        } else if (LUT) {
            // 1.5 * 2^23 + d - I: an integer in [0, 2 d] on top of the float-bit offset, so the bit
            // pattern read as an integer is PV_MAGIC_BITS + (d - I) and all further logit
            // arithmetic (minimum, table address) is integer arithmetic on it
            const float cm = PV_MAGIC_F + (float)d;
            v16f cin;
#pragma unroll
            for (int r = 0; r < 16; ++r) cin[r] = cm;
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                wt[t] = 0.0f;
                T[t] = qk_mfma<DK2>(ka[t], qB, cin);
            }
        } else {
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                wt[t] = 0.0f;
                if (!dead_tile(t)) T[t] = qk_mfma<DK2>(ka[t], qB, bias_tile(it, t));
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (F32L && !BIAS_LATE && more) load_bias_quarters(brow, nblkidx);
        if (HI_REGS && more) load_bias_hi(brow, nblkidx);  // (braw is free again)
        if (MODE == BIAS_BF16_VEC && more)  // braw is free again
            load_bias_vec(brow, nblkidx);
        if (LDS_BIAS && !BIAS_DB && more) {
            wait_lds();                       // this block's tile has been read into registers
            dma_bias(sw ? nxt : cur, bsrc, nblkidx, bnxt, !(SHORT || (ONEHEAD && NB == 2)) ? 0 : tpar ? ENDS_INSIDE : ENDS_RAGGED);    // refill the wave's own region
        }
        //    the LDS reads of the P.V phase go out now and land during the exponentials
        v16i acc[DK];
        v4i va[PRE > 0 ? PRE : 1][KT];
#pragma unroll
        for (int cb = 0; cb < PRE; ++cb) {
#pragma unroll
            for (int q4 = 0; q4 < live_quads(cb); ++q4) {
                const v4i c4 = *reinterpret_cast<const v4i *>(ibuf + L::CS_OFF + 4 * (32 * cb + 8 * q4 + 4 * g));
                acc[cb][4 * q4] = c4[0]; acc[cb][4 * q4 + 1] = c4[1];
                acc[cb][4 * q4 + 2] = c4[2]; acc[cb][4 * q4 + 3] = c4[3];
            }
#pragma unroll
            for (int t = 0; t < (VDEMAND ? 0 : KT); ++t)
                va[cb][t] = *reinterpret_cast<const v4i *>(ibuf + L::V_OFF + (32 * cb + m) * L::VP + 32 * t + 16 * g);
        }

        const bool ragged = it * BV + BV > N;
        // (Tile by tile costs branches in the 8-wave forms over a workspace, and where DK = 3 has no bias: us, by tile / at once, d = 128,
        // fp32 bias, 18 heads N = 10122 1288 / 1279, d = 64, bf16, 32 heads N = 8192 709.6 / 706.9; no bias, d = 72, 1 head N = 8284
        // 108.5 / 107.7, 40 heads N = 4100 220.2 / 217.2.)
        constexpr bool AT_ONCE = !ONEHEAD && (NB == 2 || (MODE == BIAS_NONE && DK == 3));
        if (AT_ONCE && ragged) {
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (it * BV + 32 * t + 16 * g + r >= N) T[t][r] = -INFINITY;
        } else if (ragged) {  // ragged last block: keys beyond N never count
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                const int left = N - it * BV - 32 * t;
                if (left >= 32 || dead_tile(t)) continue;  // uniform
                const int lim = left - 16 * g;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (r >= lim) T[t][r] = LUT ? PV_MAGIC_F + (float)(4 * d + 2) : -INFINITY;
            }
        }

        float resc;
        float ls0 = 0.0f, ls1 = 0.0f;
        v4i pk[KT];
        if constexpr (LUT) {
            // 2. running maximum of I = running minimum of the bit patterns (a block always holds
            //    a key inside the sequence, so the minimum is a real logit)
            int hb = __float_as_int(T[0][0]);
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) hb = min(hb, __float_as_int(T[t][r]));
            {
                const auto sw2 = __builtin_amdgcn_permlane32_swap((unsigned)hb, (unsigned)hb, false, false);
                hb = min((int)sw2[0], (int)sw2[1]);
            }
            const int hb_new = min(hb_run, hb);
            // e^{m_old - m_new} with m = alpha (d - h): the first block of an item has nothing to carry
            resc = hb_run == 0x7fffffff ? 0.0f : __builtin_amdgcn_exp2f((float)(hb_new - hb_run) * a2);
            hb_run = hb_new;
            // 3. 255 * exp(S - m) = lut[(h - h_min) / 2]: byte address 2 (h - h_min) past the table
            const unsigned abase = lds_offset(lut) - 2u * (unsigned)hb_new;
#pragma unroll
            for (int t = 0; t < KT; ++t) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    unsigned w = 0;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const unsigned a = ((unsigned)__float_as_int(T[t][4 * i + j]) << 1) + abase;
                        const float pe = *reinterpret_cast<const __attribute__((address_space(3))) float *>((size_t)a);
                        if (j & 1) ls1 += pe; else ls0 += pe;
                        w = __builtin_amdgcn_cvt_pk_u8_f32(pe, j, w);
                    }
                    pk[t][i] = (int)(w ^ 0x80808080u);
                }
            }
        } else {
        // 2. running maximum (Alg. 1: m_ij = max(m_i,j-1, rowmax S_ij); both lanes of a row hold the same m_run)
        float mx = m_run;
        if (AXIAL) {  // per-tile maxima, each shifted by the tile's y term
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                float mt = ninf;
#pragma unroll
                for (int r = 0; r < 16; ++r) mt = fmaxf(mt, T[t][r]);
                mx = fmaxf(mx, mt + wt[t]);
            }
        } else {
#pragma unroll
            for (int t = 0; t < KT; ++t)
                if (!dead_tile(t))
#pragma unroll
                    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, T[t][r]);
        }
        const float m_new = pair_max(mx);
        const float m_use = (MODE != BIAS_NONE && m_new == -INFINITY) ? 0.0f : m_new;  // whole row masked so far
        resc = __builtin_amdgcn_exp2f((m_run - m_use) * a2);  // e^{m_old - m_new}
        const float cexp = LOG2_255_F - m_use * a2;
        m_run = m_new;

        // 3. p = 255 * exp(S - m), its row sum, and the byte codes
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            if (t == 0) __builtin_amdgcn_sched_barrier(0);
            if (dead_tile(t)) {
                pk[t] = v4i{(int)0x80808080u, (int)0x80808080u, (int)0x80808080u, (int)0x80808080u};
                continue;
            }
            if constexpr (VDEMAND) {
#pragma unroll
                for (int cb = 0; cb < PRE; ++cb)
                    va[cb][t] = *reinterpret_cast<const v4i *>(ibuf + L::V_OFF + (32 * cb + m) * L::VP + 32 * t + 16 * g);
            }
            const float ce = AXIAL ? fmaf(wt[t], a2, cexp) : cexp;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                unsigned w = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float pe = __builtin_amdgcn_exp2f(fmaf(T[t][4 * i + j], a2, ce));
                    if (!(ONEHEAD && DK == 4) && t == 0 && i == 0 && j < 2) (j ? ls1 : ls0) = pe;  // (there one register too many)
                    else if (j & 1) ls1 += pe; else ls0 += pe;
                    w = __builtin_amdgcn_cvt_pk_u8_f32(pe, j, w);
                }
                pk[t][i] = (int)(w ^ 0x80808080u);  // code - 128 as signed bytes
            }
            // (the sums are finished here: the compiler would keep all 64 terms until the block's end and spill)
            if (TBLK && DK == 2 && WAVES3) asm volatile("" : "+v"(ls0), "+v"(ls1));
            if constexpr (PV_EARLY) {
#pragma unroll
                for (int cb = 0; cb < PRE; ++cb)
                    acc[cb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(va[cb][t], pk[t], acc[cb], 0, 0, 0);
                if (AXIAL || WAVES3 || ALL_EARLY) __builtin_amdgcn_sched_barrier(0);
            }
            // The shared bias tile of the next block (BIAS_DB), one copy per tile of exponentials:
            // issued in one burst at the start of the block, beside the image copies, they fill
            // the memory pipeline's queue and hold the wave there (1.5 % of the block time).
            if (BIAS_DB && more && t < 2 * RGW) {
                if (whole)
                    dma16<WIDE == WIDE_PAIR_ONCE>(bsrc.base[t / 2] + 128 * (t & 1), bsrc.voff[t / 2], bnxt + ((rg0 + t / 2) * 2 + (t & 1)) * 1024);
                else
                    dma_bias_one(bsrc, nblkidx, nklim, bnxt, t);
                if (t & 1) bsrc.base[t / 2] += BV * ESZ;
            }
        }
        }
        if (BIAS_LATE) {
            __builtin_amdgcn_sched_barrier(0);
            if (more) load_bias_quarters(bias_row_ptr(sw ? nxt : cur, args()), nblkidx);
        }
        l_run = fmaf(l_run, resc, ls0 + ls1);
        rho = fmaf(rho, resc, 1.0f);

        // 4. P~ . V~ : the prefetched channel blocks as interleaved MFMA chains ...
        if (!PV_EARLY)
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int cb = 0; cb < PRE; ++cb)
                acc[cb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(va[cb][t], pk[t], acc[cb], 0, 0, 0);
        //    ... then the remaining ones
#pragma unroll
        for (int cb = PRE; cb < DK; ++cb) {
#pragma unroll
            for (int q4 = 0; q4 < live_quads(cb); ++q4) {
                const v4i c4 = *reinterpret_cast<const v4i *>(ibuf + L::CS_OFF + 4 * (32 * cb + 8 * q4 + 4 * g));
                acc[cb][4 * q4] = c4[0]; acc[cb][4 * q4 + 1] = c4[1];
                acc[cb][4 * q4 + 2] = c4[2]; acc[cb][4 * q4 + 3] = c4[3];
            }
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                const v4i a = *reinterpret_cast<const v4i *>(ibuf + L::V_OFF + (32 * cb + m) * L::VP + 32 * t + 16 * g);
                acc[cb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, pk[t], acc[cb], 0, 0, 0);
            }
        }
        // 5. O = e^{m_old - m_new} O + block result
#pragma unroll
        for (int cb = 0; cb < DK; ++cb)
#pragma unroll
            for (int r = 0; r < 4 * live_quads(cb); ++r) Of[cb][r] = fmaf(Of[cb][r], resc, __int_as_float(acc[cb][r]));
        }
        if (TBLK && more && !sw) table_store(tab + (tpar ^ 1) * 4 * TB_CP, inv_alpha);
        __builtin_amdgcn_sched_barrier(0);  // keep the wait at the very end of the block
        if (TBLK) __builtin_amdgcn_s_waitcnt(0x0F70);  // (vmcnt(0) in the form the compiler counts: see the decomposed bias's tables)
        else wait_vmem();  // this wave's copies for the next block have landed
        // everyone is done with this block's buffers, the next ones are complete (the single-launch forms have nothing
        // but tiles of a wave's own to fill again)
        if (!ONEHEAD) __syncthreads();

        if (nblkidx != 0) {
            ++it;
            return true;
        }
        finish_item(cur, &sdelta[parity][isel][0]);
        if (!PERSIST || !nxt.valid) {
            if (ENDS) __builtin_amdgcn_endpgm();
            return false;
        }
        cur = nxt;
        v += gridDim.x;
        if (ONEHEAD4) nxt.valid = false;  // (two row blocks)
        else nxt = decode(v + gridDim.x, args());
        if (PSUM && args().psum) item_mu(cur, mu_parts(&spsum[parity][0], args()), args());
        if (!ONEHEAD4) parity ^= 1;  // (the single-launch forms keep one copy of delta_v)
        copy_item_data(args());
        begin_item(cur, std::integral_constant<bool, ONEHEAD4>{}, args());
        if (TBLK) {  // (the next item's first rows: divided by ITS alpha)
            table_store(tab + (tpar ^ 1) * 4 * TB_CP, inv_alpha);
            __syncthreads();
        }
        it = 0;
        if (!PAIR) next_rebase = first_rebase();
        return true;
    };

    // ---- prologue: first block of the first item --------------------------------
    if constexpr (ONEHEAD) {
        // phi and psi of Alg. 1 for this head, straight into the two LDS images.
        constexpr int NT = FUSED_THREADS * NB;
        __shared__ int sabs[NT / 64][DKP];   // per-channel absmax of V (bit patterns), a wave's own
        __shared__ __attribute__((aligned(16))) float srcp[DKP];  // the quantiser's multipliers
        // |q| and |k| partial sums.  The 4-wave form adds what a lane sees of both row blocks in one
        // sum (kept in the second of two, the first stays 0); with p.split_sums it keeps what waves w
        // and w + 4 of the 8-wave form add apart, which gives the 8-wave form's abs-means to the last bit.
        constexpr bool SPLIT_BUILT = ONEHEAD4 && DK == 3 && (MODE == BIAS_TABLE || MODE == BIAS_BF16_LDS);
        constexpr int NS = SPLIT_BUILT ? 2 : 1;
        constexpr int NSUM = NS * NT / 64;
        __shared__ float ssum[2][NSUM];
        const int C16 = d / 8;
        const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        auto imgp = [&](int blk) -> char * { return blk ? bufB : bufA; };
        const uint16_t *qb_ = p.xq + (int64_t)cur.b * p.xqs.b + (int64_t)cur.h * p.xqs.h;
        const uint16_t *kb_ = p.xk + (int64_t)cur.b * p.xks.b + (int64_t)cur.h * p.xks.h;
        const uint16_t *vb_ = p.xv + (int64_t)cur.b * p.xvs.b + (int64_t)cur.h * p.xvs.h;

        // Every global load of the head goes out before the first one is used, oldest first in
        // the order of use: the bias tile, this lane's query chunks, the V rows, the key chunks.
        if (LDS_BIAS) {
            bsrc = bias_dma_src(cur, first_args());
            dma_bias(cur, bsrc, 0, lds_offset(bA), ENDS_RAGGED);
        }
        if (BROW_AHEAD) brow = bias_row_ptr(cur, first_args());
        if (HI_REGS) load_bias_hi(brow, 0);
        if (MODE == BIAS_BF16_VEC) load_bias_vec(brow, 0);
        if (F32L && !BIAS_LATE) load_bias_quarters(brow, 0);
        // Row loads go through buffer descriptors that end with the tensor's last row: rows beyond N read as zeros (no effect on
        // a sum or a maximum, code 0), an address is one 32-bit offset, and nothing is clamped or masked.  (Pitches from
        // HEAD_FAR_PITCH elements on do not fit the offsets and take 64-bit addresses.)  With that, nothing cleared that no result
        // depends on, passes without work left out, wave sums by lane swaps and no barrier between the key blocks: 3 heads,
        // N = 197, d = 64 13.3 -> 12.1 us, 768 heads 41.5 -> 37.9, 768 heads, N = 100 22.0 -> 20.0, 512 heads, N = 256, d = 72
        // 30.5 -> 29.7 (its load phase, 7 of 28 us, is at the memory's rate).
        struct Rows {
            __amdgpu_buffer_rsrc_t r;
            unsigned pitch;  // bytes
            const uint16_t *base;
            int64_t pitch64;
        };
        auto rows_of = [&](const uint16_t *base, int64_t pitch) {
            Rows o;
            o.base = base;
            o.pitch64 = pitch;
            o.pitch = N > 1 ? 2u * (unsigned)pitch : 2u * (unsigned)d;  // (a single row may have any pitch)
            o.r = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(base), 0, (N - 1) * o.pitch + 2 * d, 0x00020000);
            return o;
        };
        const Rows rq = rows_of(qb_, p.xqs.n), rk = rows_of(kb_, p.xks.n), rv = rows_of(vb_, p.xvs.n);
        // 8 channels from channel c0 of a row; off: byte offset row * pitch + 2 c0
        auto load_chunk = [&](auto fast, const Rows &src, unsigned off, int row, int c0) -> u4 {
            if constexpr (decltype(fast)::value) return __builtin_amdgcn_raw_buffer_load_b128(src.r, off, 0, 0);
            return row < N && c0 < d ? *reinterpret_cast<const u4 *>(src.base + (int64_t)row * src.pitch64 + c0) : u4{0u, 0u, 0u, 0u};
        };
        // this lane's query row: the chunks of the sign words its B operand needs (channels 64 s + 32 g + 8 j)
        const int qrow = (ONEHEAD4 ? 0 : cur.rb * BR) + wave * ROWS_PER_WAVE + m;
        u4 qx[ONEHEAD4 ? 2 : 1][DK2][4];  // (4-wave form: and its row in the second row block)
        float qsum[NS] = {}, ksum[NS] = {};
        auto load_q_row = [&](auto fast, int rb) {
            const int row = qrow + rb * BR;
            const unsigned o0 = (unsigned)row * rq.pitch + 64 * g;
#pragma unroll
            for (int sI = 0; sI < DK2; ++sI)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (64 * sI + 8 * j < d)  // uniform
                        qx[rb][sI][j] = load_chunk(fast, rq, o0 + 128 * sI + 16 * j, row, 64 * sI + 32 * g + 8 * j);
        };
        auto q_row_words = [&](int rb, unsigned *words, float &sum) {  // FP4 words of the loaded row, |q| into sum
            const int row = qrow + rb * BR;
#pragma unroll
            for (int sI = 0; sI < DK2; ++sI)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int c0 = 64 * sI + 8 * j;  // of the lower lanes
                    unsigned word = 0u;
                    if (c0 + 32 < d || (c0 < d && g == 0)) word = fp4_pm1_abs(qx[rb][sI][j], sum);
                    words[4 * sI + j] = word;
                }
            if (sum != sum && row < N) {  // a NaN among this lane's queries: the words once more, exactly
#pragma unroll
                for (int i = 0; i < PQ; ++i)
                    if (words[i] != 0u)
                        words[i] = fp4_pm1_exact(*reinterpret_cast<const u4 *>(
                            qb_ + (int64_t)row * p.xqs.n + 32 * (2 * (i / 4) + g) + 8 * (i % 4)));
            }
        };
        // V rows into registers: a thread owns quads of consecutive tokens of one 8-channel
        // chunk; consecutive lanes take consecutive chunks (whole-row loads)
        // i / C16 for 0 <= i < 2^12 and C16 <= 16 without the integer-division sequence:
        // (i + 0.5) / C16 is at least 1/32 away from every integer, far more than the error
        // of the fp32 product
        const float rc16 = 1.0f / (float)C16;
        auto div_c16 = [&](int i) { return (int)(((float)i + 0.5f) * rc16); };
        const int RT = head_v_groups(NT, C16);  // thread groups = token quads per pass
        const int vn = div_c16(threadIdx.x), vr = head_v_group(vn, NT, DK), vc = threadIdx.x - vn * C16;
        constexpr int KQ = head_v_passes(NT, DK);
        u4 vw[KQ][4];
        // this thread's key chunks (8 channels of one key each): chunk i = thread + kk NT belongs to key group i / C16
        constexpr int KPT = (2 * BV * 4 * DK + NT - 1) / NT;  // chunks per thread, at most
        const int kpt = (2 * BV * C16 + NT - 1) / NT;
        // All rows are loaded, those beyond N as zeros.  At 64 < d <= 96 the words of the second key block and of the second query
        // row are left out where N <= 128, or more than 256 heads are slower than with the clamped rows before the descriptors
        // (us, clamped / all / half: 1080 heads, N = 128, d = 96 35.6 / 36.8 / 34.3, d = 88 34.5 / 35.4 / 33.0; N = 1, d = 96 28.7 / 30.9 /
        // 28.5).  Narrower and wider heads are not; leaving out loads as well gives 6 % more there, and costs 1 % above 128 tokens.
        const int rows = DK == 3 && N <= BV ? BV : 2 * BV;
        const int kwords = (rows * C16 + NT - 1) / NT;
        u4 kx[KPT];
        unsigned kdst[KPT];  // where its FP4 word goes (LDS offset), 0xffffffff for a chunk that does not exist
        auto issue = [&](auto fast) {
            load_q_row(fast, 0);
            const unsigned v0 = (unsigned)(4 * vr) * rv.pitch + 16 * vc;
#pragma unroll
            for (int kq = 0; kq < KQ; ++kq)
                if (head_v_pass(kq, RT))  // uniform
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        vw[kq][t] = load_chunk(fast, rv, v0 + (unsigned)(4 * kq * RT + t) * rv.pitch, 4 * head_v_quad(vr, kq, RT) + t, 8 * vc);
#pragma unroll
            for (int kk = 0; kk < KPT; ++kk)
                if (kk < kpt) {  // uniform
                    const int i = threadIdx.x + kk * NT;
                    const int ic = div_c16(i), c8 = i - ic * C16;
                    const int o = key_of_chunk(ic % BV), pos = position_of_key(o), key = (ic & BV) + o;
                    kdst[kk] = lds_offset(bufA) + (ic & BV ? lds_offset(bufB) - lds_offset(bufA) : 0u) + L::K_OFF + pos * L::KP +
                               16 * k_chunk(pos, c8 >> 2, L::KP) + 4 * (c8 & 3);
                    if ((2 * BV * 4 * DK) % NT != 0 || NB == 2) kdst[kk] = ic < 2 * BV ? kdst[kk] : 0xffffffffu;
                    kx[kk] = load_chunk(fast, rk, (unsigned)key * rk.pitch + 16 * c8, ic < 2 * BV ? key : N, 8 * c8);
                }
            if constexpr (ONEHEAD4) load_q_row(fast, 1);
        };
        if (p.small_pitch) issue(std::true_type{});
        else issue(std::false_type{});
        for (int i = lane; i < DKP; i += 64) sabs[wid][i] = 0;
        // (Nothing else is cleared: logits of keys beyond N are replaced, the query operand is zero in channels beyond d and
        // FP4 has no NaN, accumulators of channels beyond d are dropped, and a V code that no key fills meets the weight 0,
        // code -128, whose share the accumulator seed takes out again.)
        // the sign words of the query row (the oldest loads: V and K may still be in flight)
        q_row_words(0, pend_q, qsum[0]);
        // keys: sign bits -> FP4 codes of +-1 at the row position the QK tile reads
#pragma unroll
        for (int kk = 0; kk < KPT; ++kk) {
            if (kk < kwords && kdst[kk] != 0xffffffffu) {
                const bool first = NS == 1 || (kk % 2 == 0 && p.split_sums);
                float sum = first ? ksum[0] : ksum[NS - 1];
                *reinterpret_cast<__attribute__((address_space(3))) unsigned *>((size_t)kdst[kk]) =
                    fp4_pm1_abs(kx[kk], sum);
                ksum[0] = first ? sum : ksum[0];
                ksum[NS - 1] = first ? ksum[NS - 1] : sum;
            }
        }
        if (ksum[0] != ksum[0] || ksum[NS - 1] != ksum[NS - 1]) {  // a NaN among this thread's keys: its words once more, exactly
            for (int i = threadIdx.x; i < 2 * BV * C16; i += NT) {
                const int ic = div_c16(i), c8 = i - ic * C16;
                const int o = key_of_chunk(ic % BV), pos = position_of_key(o), key = (ic & BV) + o;
                if (key < N)
                    *reinterpret_cast<unsigned *>(imgp(ic / BV) + L::K_OFF + pos * L::KP +
                                                  16 * k_chunk(pos, c8 >> 2, L::KP) + 4 * (c8 & 3)) =
                        fp4_pm1_exact(*reinterpret_cast<const u4 *>(kb_ + (int64_t)key * p.xks.n + 8 * c8));
            }
        }
        if constexpr (ONEHEAD4) {
            if (NS == 2 && !p.split_sums) {
                qsum[NS - 1] = qsum[0];
                qsum[0] = 0.0f;
            }
            if (rows > BR) q_row_words(1, pend_q2, qsum[NS - 1]);
            if (cur.rb == 1) {  // (uniform)
#pragma unroll
                for (int i = 0; i < PQ; ++i) pend_q[i] = pend_q2[i];
            }
            if (TRI) {
#pragma unroll
                for (int i = 0; i < PQ; ++i) row2_words[threadIdx.x][i] = pend_q2[i];
            }
        }
        // V: absmax per channel through LDS integer maxima
        {
            unsigned mb[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int kq = 0; kq < KQ; ++kq)
                if (head_v_pass(kq, RT))
#pragma unroll
                    for (int t = 0; t < 4; ++t) absmax_acc(mb, vw[kq][t]);
            float mf[8];
            absmax_floats(mb, mf);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (mf[i] > 0.0f) atomicMax(&sabs[wid][8 * vc + i], __float_as_int(mf[i]));
        }
        // abs-means: wave sums, then the eight partials
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            qsum[i] = row_tree_sum(pair_sum(qsum[i]));
            ksum[i] = row_tree_sum(pair_sum(ksum[i]));
        }
        if (lane == 0) {
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                ssum[0][(threadIdx.x >> 6) + 4 * i] = qsum[i];
                ssum[1][(threadIdx.x >> 6) + 4 * i] = ksum[i];
            }
        }
        __syncthreads();
        if (threadIdx.x < 8 * C16) {
            float dl;
            int am = 0;
#pragma unroll
            for (int i = 0; i < NT / 64; ++i) am = max(am, sabs[i][threadIdx.x]);
            quant_consts(__int_as_float(am), &dl, &srcp[threadIdx.x]);
            sdelta[0][0][threadIdx.x] = dl;
        }
        float tq = 0.0f, tk = 0.0f;
#pragma unroll
        for (int i = 0; i < NSUM; ++i) {
            tq += ssum[0][i];
            tk += ssum[1][i];
        }
        const float inv_cnt = 1.0f / ((float)N * (float)d);
        pend_muq = p.use_mu ? tq * inv_cnt : 1.0f;
        pend_muk = p.use_mu ? tk * inv_cnt : 1.0f;
        if (threadIdx.x == 0 && (!ONEHEAD4 || cur.rb == 0)) {
            if (p.mu_q_out) p.mu_q_out[cur.bh] = tq * inv_cnt;
            if (p.mu_k_out) p.mu_k_out[cur.bh] = tk * inv_cnt;
        }
        __syncthreads();
        // V codes, channel-major, into the images
        {
            const QuantConsts8 kc = load_quant_consts8(srcp, vc);
#pragma unroll
            for (int kq = 0; kq < KQ; ++kq) {
                const int quad = head_v_quad(vr, kq, RT);
                if (head_v_pass(kq, RT) && 4 * quad < N && quad < HEAD_QUADS) {
                    unsigned packed[8];
                    quant_quad(vw[kq], kc, &sdelta[0][0][0], vc, packed);
                    char *imgq = imgp(quad / (BV / 4));
                    char *dstv = imgq + L::V_OFF + 4 * (quad % (BV / 4));
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        *reinterpret_cast<unsigned *>(dstv + (8 * vc + i) * L::VP) = packed[i];
                }
            }
        }
    } else {
        // Everything the first block needs is under way before the first of it is waited for: the kernel's arguments fetched at once, the
        // item's number divided by products, the tiles not behind the abs-means (4.6 us from the start to the first block before,
        // N = 1024, d = 72, 128 heads; attention stage, us, before / after: 64 heads, N = 128, d = 72 9.1 / 8.6, 512 heads 16.0 / 15.3, N = 1024, 128 heads 53.1 / 52.0).
        MuParts parts = {};
        if (!AXIAL && p.psum) parts = mu_parts(p.psum + (int64_t)cur.bh * p.nblk * 2, first_args());
        fetch_item_regs(cur, first_args());
        imgs = image_ptr(cur, first_args());
        dma_image<DK, NWI>(imgs, lds_offset(bufA) + isel * L::BYTES, ROWS2 ? wreg : wave, lane);
        imgs += L::BYTES;
        if (LDS_BIAS) {
            bsrc = bias_dma_src(cur, first_args());
            dma_bias(cur, bsrc, 0, lds_offset(bA), 0);
        }
        if (!AXIAL && p.psum) item_mu(cur, parts, first_args());
    }
    begin_item(cur, std::false_type{}, first_args());
    if (BIAS_LATE) load_bias_quarters(brow, 0);
    if (!ONEHEAD) {
        if (BROW_AHEAD) brow = bias_row_ptr(cur, first_args());
        if (MODE == BIAS_BF16_VEC) load_bias_vec(brow, 0);
        if (F32L) load_bias_quarters(brow, 0);
        copy_item_data(first_args());
    }
    if (TBLK) {
        table_begin(cur, p);
        tblk_load(cur.rb, 0);
        table_store(tab, inv_alpha);
    }
    wait_vmem();
    __syncthreads();
    if constexpr (ONEHEAD) {
        // accumulator seeds of the two images: float-bit offset + 128 * (column sums of the V
        // codes), one thread per (block, channel) over the finished tiles
        if ((int)threadIdx.x < p.nblk * DKP) {
            char *imgq = threadIdx.x / DKP ? bufB : bufA;
            const int ch = threadIdx.x % DKP;
            int sum = 0;
#pragma unroll
            for (int j = 0; j < BV / 16; ++j) {
                const u4 x = *reinterpret_cast<const u4 *>(imgq + L::V_OFF + ch * L::VP + 16 * j);
#pragma unroll
                for (int n = 0; n < 4; ++n) sum = __builtin_amdgcn_sdot4((int)x[n], 0x01010101, sum, false);
            }
            reinterpret_cast<int *>(imgq + L::CS_OFF)[ch] = PV_MAGIC_BITS + 128 * sum;
        }
        __syncthreads();
    }

    const char *imgA = bufA + isel * L::BYTES, *imgB = bufB + isel * L::BYTES;
    // The carried offset 1.5 * 2^23 * rho sets the carry's rounding unit: it is taken out once
    // in REBASE blocks (one FMA per output register), so that rho stays below REBASE + 2 and a
    // block result is rounded to at most 8 units of the integer accumulator whatever N is.  (At
    // the loop's back edge: inside the block body the extra branch cost the four-channel-block
    // kernels their registers.)
    auto rebase = [&]() {
#pragma unroll
        for (int cb = 0; cb < DK; ++cb)
#pragma unroll
            for (int r = 0; r < 4 * live_quads(cb); ++r) Of[cb][r] = fmaf(-PV_MAGIC_F, rho, Of[cb][r]);
        rho = 0.0f;
        if (!PAIR) next_rebase += REBASE;
    };
    // (paired form: one item, its phase formed here: 2 % faster than a running block number)
    const int phase = PAIR ? first_rebase() - REBASE : 0;
    auto rebase_now = [&]() -> bool {  // `it`: the block that comes next
        if (PAIR) return it >= REBASE && (it & (REBASE - 1)) == phase;
        return PHASE ? it == next_rebase : it >= REBASE && (it & (REBASE - 2)) == 0;
    };
    for (;;) {
        if (!step(imgA, lds_offset(bufB), 0, lds_offset(bA) + BIAS_B, 0)) break;
        if (PHASE && rebase_now()) rebase();
        if (!step(imgB, lds_offset(bufA), BIAS_B, lds_offset(bA), 1)) break;
        if (rebase_now()) rebase();
    }
}

// Three waves per SIMD instead of two hide more of a block's LDS and matrix latencies where the biases are
// generated (two / three waves: decomposed, d = 64, N = 16384 2073 / 1918 us, N = 4096, 96 heads 436 / 412; table,
// d = 32 120 / 110, d = 64 2170 / 1987), but not where all items fit two workgroups per compute unit (table, 24 items,
// d = 64 26.5 / 26.9; decomposed, attention stage, d = 32, N = 2048, 128 items 24.4 / 25.2, d = 64, N = 16384, 256 items 188 / 192,
// N = 1024, 384 items 20.8 / 21.2, though d = 32, N = 2048, 384 items 32.8 / 32.2).  Without a bias or with dense tiles (up to 32
// channels: LDS) a workgroup's block takes as much longer as there are more of them, and what counts is
// the last round, which leaves the chip less idle unless the 512 slots of two waves fill theirs: 96 heads,
// N = 1024, d = 64 43.6 / 41.1 us (768 items), 480 heads, N = 600, d = 48 88.8 / 84.1 (2400), 36 heads, N = 2048, d = 32, bf16
// bias 80.9 / 67.5 (576), but 96 heads, N = 2048, d = 32 97.2 / 98.5 (1536), 12 heads, N = 4096 69.0 / 72.0 (384).  Between
// 769 and 896 items, where both take two rounds, and over tens of rounds three waves stay ahead (whole calls):
// N = 1024, d = 64 97 heads 48.5 / 46.6, 112 heads 49.6 / 48.1, d = 32 112 heads 42.2 / 41.2, bf16 bias 60.0 / 59.2; N = 600, d = 48
// 1501 heads (7505 items) 258 / 245, N = 1000, d = 64 1501 heads (12008) 574 / 555.  At a remainder of 0 or above 384 it goes
// either way (attention stage: d = 64, N = 1024 1024 heads 240 / 231, but d = 32, bf16 bias, N = 1000 1024 heads 452 / 460, 128 heads
// 51.8 / 55.4).
constexpr bool use_waves3(int DK, int mode, int items) {
    const bool generated = (mode == BIAS_AXIAL && DK <= 2 && items > 512) || (mode == BIAS_TABLE_BLK && (DK == 1 || (DK == 2 && items > 512)));
    const bool other = (mode == BIAS_NONE && DK <= 2) || ((mode == BIAS_BF16_LDS || mode == BIAS_BF16_LDS8) && DK == 1);
    return generated || (other && items > 512 && items % 512 != 0 && items % 512 <= 384);
}
// Dense tiles up to 32 channels are built once: both forms take 162 registers and run alike on the grid of two (N = 1024,
// 63 heads 26.1 / 26.0 us).  Without a bias the accumulator's offset removal between the two blocks of the loop costs the
// three-wave form 4 % there (4 heads, N = 8192 73.9 / 76.9).
constexpr bool waves2_built(int DK, int mode) {
    return !use_waves3(DK, mode, 1) && !(DK == 1 && (mode == BIAS_BF16_LDS || mode == BIAS_BF16_LDS8));
}

template <int DK, int FORMS>
int launch_fused_dk(const FusedParams &p, int mode, hipStream_t stream) {
    // NB = 1, persistent grid: as many workgroups as fit on the chip at once (two 4-wave
    // workgroups per CU, 256 CUs), a multiple of 8 so that a workgroup's items stay on one
    // XCD; fewer if there is less work.  NB = 2: one workgroup per item.
    const int needed = ((p.total_wg + 7) / 8) * 8;
    if (p.wide == WIDE_ROWS2) {  // persistent, one 8-wave workgroup per CU
        if constexpr (DK == 4) {
            const dim3 grid((unsigned)(needed < 256 ? needed : 256)), block(FUSED_THREADS * 2);
            if (mode == BIAS_BF16_LDS)
                hipLaunchKernelGGL((fused_kernel<DK, BIAS_BF16_LDS, 2, WIDE_ROWS2 | FORMS>), grid, block, 0, stream, p);
            else if (mode == BIAS_F32_LDS)
                hipLaunchKernelGGL((fused_kernel<DK, BIAS_F32_LDS, 2, WIDE_ROWS2 | FORMS>), grid, block, 0, stream, p);
            else
                return BINATTN_ERR_DTYPE;
            return check_launch();
        }
        return BINATTN_ERR_SHAPE;
    }
    const bool waves3 = p.nb == 1 && use_waves3(DK, mode, p.total_wg);
    const int slots = waves3 ? 768 : 512;
    const dim3 grid((unsigned)(p.nb == 2 || needed < slots ? needed : slots));
    const dim3 block(FUSED_THREADS * p.nb);
    if (p.nb == 2) {
        if constexpr (DK <= 2) {
            if (mode != BIAS_BF16_LDS) return BINATTN_ERR_DTYPE;
            if (p.wide == WIDE_PAIR_ONCE)
                hipLaunchKernelGGL((fused_kernel<DK, BIAS_BF16_LDS, 2, WIDE_PAIR_ONCE | FORMS>), grid, block, 0, stream, p);
            else
                hipLaunchKernelGGL((fused_kernel<DK, BIAS_BF16_LDS, 2, FORMS>), grid, block, 0, stream, p);
            return check_launch();
        }
        return BINATTN_ERR_SHAPE;
    }
    switch (mode) {
// (the form of three waves per SIMD where use_waves3 may choose it or is the only one)
#define CASE(M)                                                                                       \
    case M:                                                                                           \
        if constexpr (use_waves3(DK, M, 513)) {                                                       \
            if (waves3 || !waves2_built(DK, M)) {                                                     \
                hipLaunchKernelGGL((fused_kernel<DK, M, 1, WIDE_WAVES3 | FORMS>), grid, block, 0, stream, p); \
                break;                                                                                \
            }                                                                                         \
        }                                                                                             \
        if constexpr (waves2_built(DK, M)) hipLaunchKernelGGL((fused_kernel<DK, M, 1, FORMS>), grid, block, 0, stream, p); \
        break;
        CASE(BIAS_NONE) CASE(BIAS_LUT) CASE(BIAS_BF16_VEC) CASE(BIAS_F32_VEC) CASE(BIAS_AXIAL) CASE(BIAS_TABLE_BLK)
        case BIAS_BF16_LDS:
        case BIAS_BF16_LDS8:
            if constexpr (DK <= 3) {
                switch (mode) { CASE(BIAS_BF16_LDS) CASE(BIAS_BF16_LDS8) }
                break;
            }
            return BINATTN_ERR_SHAPE;
#undef CASE
        case BIAS_F32_LDS:
            if constexpr (DK <= 3) {
                hipLaunchKernelGGL((fused_kernel<DK, BIAS_F32_LDS, 1, FORMS>), grid, block, 0, stream, p);
                break;
            }
            return BINATTN_ERR_SHAPE;
        default: return BINATTN_ERR_DTYPE;
    }
    return check_launch();
}

// WIDE_SHORT and WIDE_SHORT4: the biases that come with token counts like 197
constexpr bool short_built(int mode) { return mode == BIAS_NONE || mode == BIAS_BF16_LDS || mode == BIAS_F32_LDS; }

template <int DK, int FORMS>
int launch_onehead_dk(const FusedParams &p, int mode, hipStream_t stream) {
    const int needed = ((p.total_wg + 7) / 8) * 8;
    const bool ends_early = p.N > BV && p.N <= 2 * BV - 32;
    if (p.nb == 1) {  // 4-wave form: the variants onehead4_built() names
        const dim3 grid((unsigned)(p.split_from < p.total_wg ? split_grid(p.split_from, p.total_wg) : needed)), block(FUSED_THREADS);
#define CASE(M)                                                                                          \
    case M:                                                                                              \
        if constexpr (onehead_three_only(DK, M)) {                                                       \
            if (ends_early) hipLaunchKernelGGL((fused_kernel<DK, M, 1, WIDE_TRISHORT4 | FORMS>), grid, block, 0, stream, p); \
            else hipLaunchKernelGGL((fused_kernel<DK, M, 1, WIDE_TRI4 | FORMS>), grid, block, 0, stream, p);     \
            return check_launch();                                                                       \
        } else if constexpr (onehead4_built(DK, M)) {                                                    \
            if constexpr (DK == 2 && M == BIAS_BF16_LDS) {                                               \
                if (p.wide == WIDE_TRI4) {                                                               \
                    hipLaunchKernelGGL((fused_kernel<DK, M, 1, WIDE_TRISHORT4 | FORMS>), grid, block, 0, stream, p); \
                    return check_launch();                                                               \
                }                                                                                        \
            }                                                                                            \
            if constexpr (short_built(M)) {                                                              \
                if (ends_early) {                                                                        \
                    hipLaunchKernelGGL((fused_kernel<DK, M, 1, WIDE_SHORT4 | FORMS>), grid, block, 0, stream, p); \
                    return check_launch();                                                               \
                }                                                                                        \
            }                                                                                            \
            hipLaunchKernelGGL((fused_kernel<DK, M, 1, WIDE_ONEHEAD4 | FORMS>), grid, block, 0, stream, p);     \
            return check_launch();                                                                       \
        }                                                                                                \
        return BINATTN_ERR_SHAPE;
        switch (mode) {
            CASE(BIAS_NONE) CASE(BIAS_LUT) CASE(BIAS_BF16_VEC) CASE(BIAS_F32_VEC) CASE(BIAS_AXIAL) CASE(BIAS_TABLE)
            CASE(BIAS_BF16_LDS) CASE(BIAS_F32_LDS)
            default: return BINATTN_ERR_DTYPE;
        }
#undef CASE
    }
    const dim3 grid((unsigned)needed), block(FUSED_THREADS * 2);
    switch (mode) {
#define CASE(M)                                                                                          \
    case M:                                                                                              \
        if constexpr (short_built(M)) {                                                                  \
            if (ends_early) {                                                                            \
                hipLaunchKernelGGL((fused_kernel<DK, M, 2, WIDE_SHORT | FORMS>), grid, block, 0, stream, p);     \
                break;                                                                                   \
            }                                                                                            \
        }                                                                                                \
        hipLaunchKernelGGL((fused_kernel<DK, M, 2, WIDE_ONEHEAD | FORMS>), grid, block, 0, stream, p);           \
        break;
        CASE(BIAS_NONE) CASE(BIAS_LUT) CASE(BIAS_BF16_VEC) CASE(BIAS_F32_VEC) CASE(BIAS_AXIAL) CASE(BIAS_TABLE)
        CASE(BIAS_BF16_LDS) CASE(BIAS_F32_LDS)
#undef CASE
        default: return BINATTN_ERR_DTYPE;
    }
    return check_launch();
}

}  // namespace binattn
