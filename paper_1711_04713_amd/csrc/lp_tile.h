// Pieces shared by the convolution and inner-product kernels: the kernel argument block, exact
// index division by run-time values, and the tile epilogue (limb combine, corrections, bias, LPAct,
// counters; Sec. 2 and 2.1 of the paper) that follows every int8-MFMA main loop.
#pragma once
#include <type_traits>

#include "lp_device.h"

namespace lp {

constexpr int kCUs = 256;    // compute units of the chip the launch geometry is tuned for
constexpr int kXCDs = 8;     // consecutive workgroup ids go round-robin to this many dies

static inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// --------------------------------------------------------------------- kernel arguments

struct ConvArgs {
    const void *x;
    const unsigned char *wp;
    const int64_t *corr;
    const void *bias;
    int bias16, bias_shift;
    int64_t *acc_out;
    void *y;
    int y16;
    unsigned long long *zero_count, *sat_count; // either may be null
    unsigned *zero_partial; // per workgroup (MFMA path): [grid] zero counts, then [grid] counts of clipped
                            // values; summed by a second kernel
    int partial_stride;     // = grid
    int direct_counts;      // no partials: every workgroup adds its counts to zero_count / sat_count itself (small grids)
    int count_sat;          // sat_count is wanted: the epilogue also counts the values it clips
    int N, H, W, Cin, Cout, R, S, stride, pad;
    int Ho, Wo, Hp, FR;
    int RH, TW, PW, NPIXA, NTAB, APLANE, PITCH;
    int tiles_c, tiles_n, CoutP, nchunks, taps, ksteps, Kflat;
    // window-row kernel: K = 32 pieces per window row / in all (a multiple of 4), 16-code units per
    // patch row / per window row / per pixel
    int KHR, KHP, UPR, SU, CU;
    int total_work, per_xcd, full_per_xcd, split;
    unsigned char *partials; // tail tiles' partial accumulators, part_bytes per (tile, part)
    int part_bytes;
    // floor(2^32 / d) for the divisors the kernel's index arithmetic uses (see udivmod)
    unsigned mg_tiles_n, mg_tiles_c, mg_Ho, mg_Hp, mg_PW, mg_TW, mg_taps, mg_S, mg_Cin, mg_SC, mg_rowlen, mg_UPR, mg_CU;
    // Skipping of all-zero input (Sec. 3.1: the sparsity the low-precision layers produce is there
    // to be skipped).  zin: flags written by the layer that produced x, one byte per (pixel tile,
    // channel tile) of ITS output, 1 = the tile holds a nonzero code; its geometry: z_rh x z_tw
    // pixels (rows of the stacked output rows), z_tiles_c tiles per row of tiles, z_tiles_n channel
    // tiles of z_bn channels; z_scale = 2 when x is the 2x2-pooled output.  zout: this layer's own
    // flags [tiles_m][tiles_n].  skipped: += (tile, 64-channel chunk) pairs not multiplied.
    // wsum: [nchunks][CoutP] sums of the weight codes per chunk, for the correction of skipped chunks.
    const unsigned char *zin;
    int z_rh, z_tw, z_tiles_c, z_tiles_n, z_bn, z_scale;
    unsigned char *zout;
    unsigned long long *skipped;
    const int *wsum;
    int fast; // 32-bit requantization is exact for this call (see epilogue)
    int pool; // store the 2x2 maxima of the codes (planner guarantees the tile geometry)
    ActParams act;
};

// x / d and x % d for 0 <= x < 2^31, d >= 1, with m = floor(2^32 / d) from the host: the high half
// of x * m is the quotient or one below it, one compare settles it.  Five cheap operations
// instead of the float-reciprocal sequence a division by a run-time value compiles to (on scalars
// they run on the scalar unit).
__host__ inline unsigned udiv_magic(int d) { return d <= 1 ? 0xffffffffu : (unsigned)((1ull << 32) / (unsigned)d); }
__device__ __forceinline__ void udivmod(int x, int d, unsigned m, int &q, int &r)
{
    unsigned qq = __umulhi((unsigned)x, m);
    unsigned rr = (unsigned)x - qq * (unsigned)d;
    if (rr >= (unsigned)d) {
        ++qq;
        rr -= (unsigned)d;
    }
    q = (int)qq;
    r = (int)rr;
}

__device__ __forceinline__ int64_t bias_term(const ConvArgs &a, int co)
{
    if (!a.bias) return 0;
    const int b = a.bias16 ? (int)((const int16_t *)a.bias)[co] : (int)((const int8_t *)a.bias)[co];
    return (int64_t)b * ((int64_t)1 << a.bias_shift);
}

// One workgroup's count (which: 0 zero codes, 1 clipped values) goes to its slot of the partials, or,
// on small grids, straight to the caller's counter.
__device__ __forceinline__ void publish_count(const ConvArgs &a, int which, unsigned total)
{
    if (a.zero_partial) {
        a.zero_partial[which * a.partial_stride + blockIdx.x] = total;
    } else if (a.direct_counts && total) {
        unsigned long long *c = which ? a.sat_count : a.zero_count;
        if (c) atomicAdd(c, (unsigned long long)total);
    }
}

// Limbs of two-limb weights.  The plain form is that of the activations, b = 256 * bh + bl + 128, whose offset makes every
// output owe 128 times the sum of the codes under its window.  With a signed low limb, b = 256 * bh + bl, nothing is owed
// but the constant 128 * sum(b) (the activations' offset): no code sums are gathered, added up or carried along.  bh then
// is (b + 128) >> 8 and fits a byte for codes below 32640.  A tile of 64 channels takes the signed form unless one of
// its weights is as large as that (the top 128 codes, where a format that clips weights puts them); bit 0 of its
// channels' corrections, otherwise multiples of 128, says so.  us, plain : signed form, batch 32: 112x112 128 -> 128 3x3 192.8 :
// 185.1, 56x56 256 -> 256 187.2 : 180.0, 28x28 512 -> 512 182.5 : 175.1, 22x22 64 -> 64 5x5 18.1 : 15.5, 112x112 16 -> 16 7x7 45.1 : 40.6.
constexpr int64_t kSignedForm = 1;
__device__ __forceinline__ void weight_limbs(int code, bool signed_form, int &hi, int &lo)
{
    lo = signed_form ? (int)(signed char)code : (code & 255) - 128;
    hi = signed_form ? (code - lo) >> 8 : code >> 8;
}
__device__ __forceinline__ bool needs_code_sums(const ConvArgs &a, int ntile) { return (a.corr[(size_t)ntile * 64] & kSignedForm) == 0; }

__device__ __forceinline__ v16i mfma_i8(v4i a, v4i b, v16i c)
{
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
}

// min(max(q, 0), cmax) for 0 <= cmax as the one instruction the hardware has for it (with cmax in
// a scalar register the compiler emits a max and a min).
__device__ __forceinline__ int clamp_code(int q, int cmax)
{
    int r;
    asm("v_med3_i32 %0, %1, 0, %2" : "=v"(r) : "v"(q), "s"(cmax));
    return r;
}

// Requantization of v = 65536*hi + lo16 (hi = floor(v / 65536), 0 <= lo16 < 65536) to
// floor((v + 2^(s-1)) / 2^s) in 32-bit arithmetic, 1 <= s <= 31; the caller clamps to [0, cmax]
// (negative v give 0: ReLU).  The value returned is exact wherever it lies inside the code range
// and stays on the same side of it wherever it does not.  S16: 0 for s >= 17 (lo16 cannot
// matter), 1 for s == 16, 2 for s <= 15.
template <int S16>
__device__ __forceinline__ int requant_relu32(int hi, int lo16, int s)
{
    int q;
    if (S16 == 0) {
        q = (hi + (1 << (s - 17))) >> (s - 16);
    } else if (S16 == 1) {
        q = hi + (lo16 >> 15);
    } else {
        // beyond 32768 the result saturates anyway, below 0 it is 0 anyway: kept inside, the
        // shifted value cannot leave 32 bits
        const int h = min(max(hi, -1), 32768);
        q = (h << (16 - s)) + ((lo16 + (1 << (s - 1))) >> s);
    }
    return q;
}

// Per-channel constants of a tile (weight correction + bias) into LDS, in the form the epilogue
// wants: three int32 planes (bits 16.., 8..15, 0..7) for the 32-bit epilogue, else int64.
// deadmask: chunks of 64 input channels that were skipped as all-zero; their share of the weight
// correction, 128 * sum(w over the chunk) - 16384 * (positions of the chunk), is taken out again
// (their limb products, which it would have cancelled, were never formed).  With 8-bit weights under
// 16-bit activations (limbs 2, wlimbs 1), and with signed low limbs, the correction has no 16384 * K term: the weights carry no offset.
// threads: of the workgroup, a constant where the kernel knows it (blockDim comes from memory, and
// that read is as long as all else here: 0.5 us of a one-limb layer of one round)
template <int BN>
__device__ __forceinline__ void build_colterms(const ConvArgs &a, int ntile, int *ctab, int threads, int limbs, int wlimbs,
                                              unsigned deadmask = 0)
{
    for (int c = threadIdx.x; c < BN; c += threads) {
        const int colg = ntile * BN + c;
        const int64_t corr = colg < a.Cout ? a.corr[colg] : 0;
        int64_t t = colg < a.Cout ? (corr & ~kSignedForm) + bias_term(a, colg) : 0;
        if (limbs == 2 && deadmask && colg < a.Cout) {
            for (unsigned rem = deadmask; rem; rem &= rem - 1) {
                const int ch = __builtin_ctz(rem);
                const int kc = a.taps * min(64, a.Cin - 64 * ch);
                t -= (int64_t)128 * a.wsum[(size_t)ch * a.CoutP + colg] - (wlimbs == 2 && !(corr & kSignedForm) ? (int64_t)16384 * kc : 0);
            }
        }
        if (a.fast) {
            // (shifts 9..16: the epilogue's rounding half 2^(s-1) rides in the constants, as 2^(s-9)
            // at the scale of v / 256; one weight limb: the top plane arrives clamped and at that scale,
            // the middle plane holds the low 16 bits)
            const bool mid = a.act.s >= 9 && a.act.s <= 16;
            const int half9 = mid ? 1 << (a.act.s - 9) : 0;
            if (mid && wlimbs == 1) {
                const int64_t top = t >> 16;
                const int topc = (int)(top > (1 << 22) ? (1 << 22) : top < -(1 << 22) ? -(1 << 22) : top);
                ctab[c] = topc * 256 + half9;
                ctab[BN + c] = (int)(t & 65535);
                ctab[2 * BN + c] = 0;
            } else {
                ctab[c] = (int)(t >> 16);
                ctab[BN + c] = (int)((t >> 8) & 255) + (wlimbs == 2 ? half9 : 0);
                ctab[2 * BN + c] = (int)(t & 255);
            }
        } else {
            ((int64_t *)ctab)[c] = t;
        }
    }
}

// Epilogue of one tile of output pixels x BN channels: combine limbs exactly, add corrections and
// bias, LPAct (or raw accumulators), count zeros.  The MFMAs are issued with the weights as the
// row operand, so in the 32x32 result layout a lane holds one output pixel (tile row row0 + mb*32
// + (lane & 31), row0 being the first tile row of the calling wave) and, in register v, channel
// 8*(v/4) + 4*(lane/32) + v%4 of its 32-channel block (the wave's blocks start at channel col0w
// of the tile): four consecutive channels per group of four registers, which leave as one 8-byte
// (4-byte) store.
// row_sum(m): sum of the codes under tile row m's window (two-limb weights of the plain form, else 0); outoff and ctab (see
// build_colterms) are LDS tables, complete and visible.  Returns the lane's counts of zero codes
// and (when a.count_sat) of values clipped at an end of the code range; see wave_total.
// The accumulators passed in cover MBL of the wave's MB row blocks, starting at block mb0, and GL
// of the four channel groups, starting at group g0 (register 4*gl + e = channel 8*(g0+gl) +
// 4*(lane/32) + e): the main kernel passes everything (MBL = MB, GL = 4, mb0 = g0 = 0), the
// finishing kernel one (row block, channel group) at a time.
struct TileCounts {
    unsigned zeros, sats;
};

// The wave's totals of its lanes' counts (the same in every lane), for lanes of at most 64 of each: both
// halves of a word go through one tree of DPP adds.
__device__ __forceinline__ TileCounts wave_total(TileCounts c)
{
    int v = (int)(c.zeros | (c.sats << 16));
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false); // row_shr:1, 2, 4, 8: sums of the 16-lane rows in their last lanes
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false); // row_bcast:15, 31
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    const unsigned t = (unsigned)__builtin_amdgcn_readlane(v, 63);
    return {t & 0xffffu, t >> 16};
}

// LIMBS / WL: 8-bit limbs of the activations and of the weights; LIMBS + WL - 1 accumulator planes, the
// most significant first (2, 2: HH, HL + LH, LL; 2, 1: H, L; 1, 1: one).
// PIECES: 8-bit codes may leave in pieces of 16 bytes (below).
template <int LIMBS, int WL, int NB, int BN, int MBL, int GL, bool PIECES = true, typename RowSum>
__device__ __forceinline__ TileCounts tile_epilogue(const ConvArgs &a, v16i (&acc)[MBL][NB][LIMBS + WL - 1],
                                                  RowSum row_sum, const int *outoff, const int *pooloff,
                                                  const int *ctab, int ntile, int row0, int col0w, int mb0, int g0)
{
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31, kg = lane >> 5;
    unsigned nz = 0, ns = 0; // zero codes written / values clipped by this lane (at most 16 * MB * NB <= 64 each)
    int oo[MBL], po[MBL], rs[MBL];
#pragma unroll
    for (int mb = 0; mb < MBL; ++mb) {
        const int m = row0 + (mb0 + mb) * 32 + l32;
        oo[mb] = outoff[m];
        po[mb] = a.pool ? pooloff[m] : -1; // pooled output pixel, at the window's top-left lane only
        rs[mb] = (WL == 2) ? row_sum(m) : 0;
    }
    if (a.fast) {
        // v = 2^16*A + 2^8*B + C with every piece in int32: the channel constant is split the same
        // way, 128*rowsum = 2^8*(rowsum >> 1) + 128*(rowsum & 1); then carries are pushed upward.
        // Shift class, code width and store mode are compile-time: about ten VALU operations per
        // value.  Stores go through a buffer descriptor that starts at the tile's first output
        // pixel (the smallest address of the tile) with 32-bit offsets from there; a lane with
        // nothing to store (a row outside the image, a padded channel, a lane that is not the
        // top-left of its pooling window) gets an offset past the descriptor and its store is
        // dropped: no branches, no 64-bit address arithmetic.
        const int s = a.act.s, cmax = a.act.hi;
        __builtin_assume(cmax >= 0);
        constexpr unsigned NOWHERE = 0x80000000u; // the descriptor never covers more than 2^31 - 1 bytes
        auto requant_tile = [&](auto s16c, auto y16c, auto modec, auto satc) __attribute__((always_inline)) {
            constexpr int S16 = decltype(s16c)::value;
            constexpr bool Y16 = decltype(y16c)::value;
            constexpr int MODE = decltype(modec)::value; // 0: four codes per store, 1: fused 2x2 max-pool, 2: ragged channels, 3: 16 bytes of codes per store
            constexpr bool SAT = decltype(satc)::value;  // also count the values clipped at cmax (with ReLU the only end)
            constexpr int ESZ = Y16 ? 2 : 1;
            const int first = __builtin_amdgcn_readfirstlane(MODE == 1 ? pooloff[0] : outoff[0]);
            const size_t pixels = MODE == 1 ? (size_t)a.N * (a.Ho >> 1) * (a.Wo >> 1) : (size_t)a.N * a.Ho * a.Wo;
            const size_t left = (pixels - (size_t)first) * a.Cout * ESZ;
            const __amdgpu_buffer_rsrc_t yrsrc = __builtin_amdgcn_make_buffer_rsrc(
                (unsigned char *)a.y + (size_t)first * a.Cout * ESZ, 0, (int)(left < 0x7fffffffu ? left : 0x7fffffffu), 0x00020000);
            unsigned rel[MBL]; // byte offset of the lane's output pixel from the tile's first one
            unsigned nnz[MBL]; // the lane's codes that are not zero (16-bit codes: two counts of 16 bits)
#pragma unroll
            for (int mb = 0; mb < MBL; ++mb) {
                const int o = MODE == 1 ? po[mb] : oo[mb];
                rel[mb] = o >= 0 ? (unsigned)((o - first) * a.Cout * ESZ) : NOWHERE;
                nnz[mb] = 0;
            }
            // the output pixel of a row of a block, read where it is needed (kept, it would cost the loop below a register)
            auto pixel_at = [&](int mb, int row) __attribute__((always_inline)) {
                int m = row0 + (mb0 + mb) * 32 + row;
                asm volatile("" : "+v"(m));
                return outoff[m];
            };
            auto exists = [&](int mb) __attribute__((always_inline)) { return MODE == 1 ? pixel_at(mb, l32) >= 0 : rel[mb] != NOWHERE; };
            // 8-bit codes of whole blocks of 32 channels, of tensors whose pixels start on 16-byte boundaries, are stored together.  A lane holds four neighbouring channels of each
            // group of eight, of one pixel: stored as they are, an instruction touches 32 lines with 8 bytes each, and the
            // memory system takes a step per line and instruction.  Swapping halves and rows of lanes between registers
            // first gives every lane 16 neighbouring bytes, four lanes to a pixel: with the counting below, 64x56x56, 128 -> 256 3x3
            // 72.0 -> 62.7 us, 256 -> 256 119.8 -> 109.6.  (16-bit codes, twice the bytes per line as they are, gain at most 2 % on large
            // layers, but small ones then wait for their stores at the end: 18x18, 64 -> 64 batch 32 10.2 -> 10.45 us.  Four 8-bit codes
            // that cannot join such a piece leave as they are made for the same reason: 24x180x9, 192 -> 232 3x3 26.2 us with their
            // stores at the end, 24.6.)
            constexpr bool BLOCKS = MODE == 3;
            unsigned word[MBL][NB][GL];
            // Counting.  A wave that is not multiplying issues one instruction at a time beside the others' MFMAs,
            // on whichever unit, so what a count costs is its instructions, scalar ones included.  Zeros: codes are
            // not negative, so min(code, 1) says whether one is nonzero, two packed codes at a time (8-bit codes:
            // the top bits of code + 127, four at a time): one instruction a code where a compare, a mask, a popcount and
            // an add took four.  Clipped values: only where the largest rounded value of a group lies above the
            // range (half an instruction a code) are they counted one by one.
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int gl = 0; gl < GL; ++gl) {
                    // a group of eight channels that lies past Cout altogether has nothing to write
                    // or count (uniform: a scalar branch)
                    if (ntile * BN + col0w + nb * 32 + 8 * (g0 + gl) >= a.Cout) {
                        if constexpr (BLOCKS)
#pragma unroll
                            for (int mb = 0; mb < MBL; ++mb) word[mb][nb][gl] = 0;
                        continue;
                    }
                    const int cl = col0w + nb * 32 + 8 * (g0 + gl) + 4 * kg; // channel within the tile
                    const int col0 = ntile * BN + cl;
                    const bool col_ok = col0 < a.Cout;
                    // what a code that exists may add to the lane's count
                    const unsigned one = !col_ok ? 0u : Y16 ? 0x00010001u : 0x80808080u;
                    const v4i cA = *(const v4i *)(ctab + cl);
                    const v4i cB = *(const v4i *)(ctab + BN + cl);
                    const v4i cC = *(const v4i *)(ctab + 2 * BN + cl);
                    int rounded[MBL][4], peak = 0; // the rounded values before clipping, the largest of them
#pragma unroll
                    for (int mb = 0; mb < MBL; ++mb) {
                        int q[4], own[4];
                        int (&raw)[4] = MODE == 2 ? own : rounded[mb]; // (read by a run-time count there: of four values, not of every block's)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int v = 4 * gl + e;
                            int hi, lo16 = 0;
                            if constexpr (WL == 2 && S16 == 3) {
                                // Shifts 9..16 (above, only the top plane matters and the class-0 form is
                                // shorter).  With W = floor(v / 256) the code is (W + 2^(s-9)) >> (s-8):
                                // the dropped low byte of v cannot carry into a multiple of 256.  W =
                                // 256*A + B + (C >> 8) + (rowsum >> 1) in 32 bits: A is clamped to +-2^22
                                // first (beyond that the code saturates for every s <= 22, and |B + ...|
                                // stays below 2^29 for K <= 8192); the half is part of cB.
                                const int C = acc[mb][nb][2][v] + cC[e] + ((rs[mb] & 1) << 7);
                                const int T = acc[mb][nb][1][v] + cB[e] + (C >> 8);
                                const int A = min(max(acc[mb][nb][0][v] + cA[e], -(1 << 22)), 1 << 22);
                                const int W = (A << 8) + T + (rs[mb] >> 1);
                                raw[e] = W >> (s - 8);
                                q[e] = clamp_code(raw[e], cmax);
                                continue;
                            } else if constexpr (S16 == 3) {
                                // one weight limb, shifts 9..16: the same with v = 65536*cA + 256*H + (L +
                                // low 16 bits of the constant); cA arrives clamped, times 256, plus the
                                // half.  |H|, |L| <= 2^27 for K <= 8192: W stays inside 32 bits
                                int W = ((acc[mb][nb][LIMBS - 1][v] + cB[e]) >> 8) + cA[e];
                                if constexpr (LIMBS == 2) W += acc[mb][nb][0][v];
                                raw[e] = W >> (s - 8);
                                q[e] = clamp_code(raw[e], cmax);
                                continue;
                            } else if constexpr (LIMBS == 2) {
                                const int C = acc[mb][nb][WL][v] + cC[e] + (WL == 2 ? (rs[mb] & 1) << 7 : 0);
                                const int B = acc[mb][nb][WL - 1][v] + cB[e] + (WL == 2 ? rs[mb] >> 1 : 0) + (C >> 8);
                                hi = cA[e] + (B >> 8);
                                if constexpr (WL == 2) hi += acc[mb][nb][0][v];
                                if constexpr (S16 != 0) lo16 = ((B & 255) << 8) | (C & 255);
                            } else {
                                // one limb: the plane split is 2^16*cA + (2^8*cB + cC)
                                const int C = acc[mb][nb][0][v] + (cB[e] << 8) + cC[e];
                                hi = cA[e] + (C >> 16);
                                lo16 = C & 65535;
                            }
                            raw[e] = requant_relu32<S16 == 3 ? 2 : S16>(hi, lo16, s);
                            q[e] = clamp_code(raw[e], cmax);
                        }
                        const bool counted = oo[mb] >= 0 && col_ok; // the lane's codes exist in the output tensor
                        if constexpr (SAT && MODE != 2) {
                            peak = max(max(peak, raw[0]), raw[1]);
                            peak = max(max(peak, raw[2]), raw[3]);
                        }
                        if constexpr (MODE == 2) { // ragged channel tail: code by code
                            if (counted) {
                                unsigned char *dst = (unsigned char *)a.y + ((size_t)oo[mb] * a.Cout + col0) * ESZ;
                                const int ncodes = min(4, a.Cout - col0);
                                for (int e = 0; e < ncodes; ++e) {
                                    if constexpr (Y16) ((int16_t *)dst)[e] = (int16_t)q[e];
                                    else ((int8_t *)dst)[e] = (int8_t)q[e];
                                    nz += (q[e] == 0);
                                    if constexpr (SAT) ns += (raw[e] > cmax);
                                }
                            }
                        } else if constexpr (Y16) {
                            // codes are in [0, cmax]: packing needs no masks
                            unsigned w0 = (unsigned)q[0] | ((unsigned)q[1] << 16);
                            unsigned w1 = (unsigned)q[2] | ((unsigned)q[3] << 16);
                            const v2us ones = __builtin_bit_cast(v2us, one);
                            nnz[mb] = __builtin_bit_cast(unsigned, (v2us)(__builtin_bit_cast(v2us, nnz[mb]) + __builtin_elementwise_min(__builtin_bit_cast(v2us, w0), ones)));
                            nnz[mb] = __builtin_bit_cast(unsigned, (v2us)(__builtin_bit_cast(v2us, nnz[mb]) + __builtin_elementwise_min(__builtin_bit_cast(v2us, w1), ones)));
                            if constexpr (MODE == 1) {
                                // 2x2 maximum across lanes: the horizontal neighbour is the next lane,
                                // the vertical one sits TW lanes further in the same 32-row block.
                                // Every lane takes part; only the window's top-left lane stores.
                                auto pkmax = [](unsigned x, unsigned y) __attribute__((always_inline)) {
                                    return __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(v2s, x),
                                                                                                  __builtin_bit_cast(v2s, y)));
                                };
                                w0 = pkmax(w0, (unsigned)__builtin_amdgcn_mov_dpp((int)w0, 0xB1, 0xF, 0xF, true));
                                w1 = pkmax(w1, (unsigned)__builtin_amdgcn_mov_dpp((int)w1, 0xB1, 0xF, 0xF, true));
                                const int below = ((lane + a.TW) & 63) * 4;
                                w0 = pkmax(w0, (unsigned)__builtin_amdgcn_ds_bpermute(below, (int)w0));
                                w1 = pkmax(w1, (unsigned)__builtin_amdgcn_ds_bpermute(below, (int)w1));
                            }
                            const unsigned at = col_ok ? rel[mb] + (unsigned)col0 * 2u : NOWHERE;
                            __builtin_amdgcn_raw_buffer_store_b64((v2u){w0, w1}, yrsrc, (int)at, 0, 0);
                        } else {
                            const unsigned w0 = (unsigned)q[0] | ((unsigned)q[1] << 8) | ((unsigned)q[2] << 16) | ((unsigned)q[3] << 24);
                            nnz[mb] += __builtin_popcount((w0 + 0x7f7f7f7fu) & one);
                            if constexpr (BLOCKS) {
                                word[mb][nb][gl] = w0;
                            } else {
                                const unsigned at = col_ok ? rel[mb] + (unsigned)col0 : NOWHERE;
                                __builtin_amdgcn_raw_buffer_store_b32(w0, yrsrc, (int)at, 0, 0);
                            }
                        }
                    }
                    if (SAT && MODE != 2 && __builtin_amdgcn_ballot_w64(peak > cmax)) {
#pragma unroll
                        for (int mb = 0; mb < MBL; ++mb) {
                            const int most = col_ok && exists(mb) ? cmax : 0x7fffffff;
#pragma unroll
                            for (int e = 0; e < 4; ++e) ns += rounded[mb][e] > most;
                        }
                    }
                }
            if constexpr (BLOCKS) {
                const auto swap32 = [](unsigned &x, unsigned &y) __attribute__((always_inline)) { // upper half of x with lower half of y
                    const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
                    x = r[0];
                    y = r[1];
                };
                const auto swap16 = [](unsigned &x, unsigned &y) __attribute__((always_inline)) { // odd rows of x with even rows of y
                    const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
                    x = r[0];
                    y = r[1];
                };
                const int colw = ntile * BN + col0w;
                const auto store = [&](const v4u &piece, int o, int ch) __attribute__((always_inline)) {
                    const unsigned at = o >= 0 && ch < a.Cout ? (unsigned)((o - first) * a.Cout + ch) : NOWHERE;
                    __builtin_amdgcn_raw_buffer_store_b128(piece, yrsrc, (int)at, 0, 0);
                };
                const int l16 = lane & 15, row = lane >> 4;
#pragma unroll
                for (int mb = 0; mb < MBL; ++mb) {
                    unsigned(&w)[NB][GL] = word[mb];
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                        for (int p = 0; p < 2; ++p) swap32(w[nb][p], w[nb][p + 2]); // lower lanes: groups 0 and 1, upper lanes: 2 and 3
                    if constexpr (NB == 2) {
#pragma unroll
                        for (int p = 0; p < 4; ++p) swap16(w[0][p], w[1][p]); // rows: channels 0, 32, 16, 48 of sixteen pixels
                        const int ch = colw + 32 * (row & 1) + 16 * (row >> 1);
                        store((v4u){w[0][0], w[0][2], w[0][1], w[0][3]}, pixel_at(mb, l16), ch);
                        store((v4u){w[1][0], w[1][2], w[1][1], w[1][3]}, pixel_at(mb, 16 + l16), ch);
                    } else {
                        const int ch = colw + 16 * kg;
                        __builtin_amdgcn_raw_buffer_store_b128((v4u){w[0][0], w[0][2], w[0][1], w[0][3]}, yrsrc,
                                                               (int)(ch < a.Cout ? rel[mb] + (unsigned)ch : NOWHERE), 0, 0);
                    }
                }
            }
            if constexpr (MODE != 2) {
                // groups of four channels that the lane has: 8 channels apart, over all blocks or one per block
                constexpr int STEP = GL == 4 ? 8 : 32;
                static_assert(GL == 4 || GL == 1, "groups are evenly spaced");
                const int left = a.Cout - (ntile * BN + col0w + 8 * g0 + 4 * kg);
                const unsigned codes = 4u * (unsigned)min(max((left + STEP - 1) / STEP, 0), NB * GL);
#pragma unroll
                for (int mb = 0; mb < MBL; ++mb)
                    nz += exists(mb) ? codes - (Y16 ? (nnz[mb] & 0xffffu) + (nnz[mb] >> 16) : nnz[mb]) : 0u;
            }
        };
        using std::integral_constant;
        auto by_sat = [&](auto s16c, auto y16c, auto modec) __attribute__((always_inline)) {
            if (a.count_sat) requant_tile(s16c, y16c, modec, integral_constant<bool, true>{});
            else requant_tile(s16c, y16c, modec, integral_constant<bool, false>{});
        };
        auto by_mode = [&](auto s16c, auto y16c) __attribute__((always_inline)) {
            if constexpr (decltype(y16c)::value) {
                if (a.pool) return by_sat(s16c, y16c, integral_constant<int, 1>{});
            }
            if constexpr (!decltype(y16c)::value && GL == 4 && PIECES) {
                if ((a.Cout & 15) == 0) return by_sat(s16c, y16c, integral_constant<int, 3>{});
            }
            if ((a.Cout & 3) == 0) by_sat(s16c, y16c, integral_constant<int, 0>{}); // every group of four channels is aligned
            else by_sat(s16c, y16c, integral_constant<int, 2>{});
        };
        // shift classes: 9..16 (the usual ones) -> 3; else >= 17 -> 0, 16 -> 1, <= 15 -> 2
        const bool mid = s >= 9 && s <= 16;
        if (a.y16) {
            if (mid) {
                by_mode(integral_constant<int, 3>{}, integral_constant<bool, true>{});
            } else if (s >= 17) by_mode(integral_constant<int, 0>{}, integral_constant<bool, true>{});
            else if (s == 16) by_mode(integral_constant<int, 1>{}, integral_constant<bool, true>{});
            else by_mode(integral_constant<int, 2>{}, integral_constant<bool, true>{});
        } else {
            if (mid) {
                by_mode(integral_constant<int, 3>{}, integral_constant<bool, false>{});
            } else if (s >= 17) by_mode(integral_constant<int, 0>{}, integral_constant<bool, false>{});
            else if (s == 16) by_mode(integral_constant<int, 1>{}, integral_constant<bool, false>{});
            else by_mode(integral_constant<int, 2>{}, integral_constant<bool, false>{});
        }
    } else {
        const int64_t *ct64 = (const int64_t *)ctab;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int gl = 0; gl < GL; ++gl) {
                const int cl = col0w + nb * 32 + 8 * (g0 + gl) + 4 * kg;
                const int col0 = ntile * BN + cl;
#pragma unroll
                for (int mb = 0; mb < MBL; ++mb) {
                    const int64_t rt = (WL == 2) ? (int64_t)rs[mb] * 128 : 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int v = 4 * gl + e;
                        int64_t val;
                        if constexpr (LIMBS == 2 && WL == 1)
                            val = ((int64_t)acc[mb][nb][0][v] << 8) + (int64_t)acc[mb][nb][1][v] + ct64[cl + e];
                        else if constexpr (LIMBS == 2)
                            val = ((int64_t)acc[mb][nb][0][v] << 16) + ((int64_t)acc[mb][nb][1][v] << 8) +
                                  (int64_t)acc[mb][nb][2][v] + rt + ct64[cl + e];
                        else
                            val = (int64_t)acc[mb][nb][0][v] + ct64[cl + e];
                        if (oo[mb] >= 0 && col0 + e < a.Cout) {
                            const size_t idx = (size_t)oo[mb] * a.Cout + col0 + e;
                            if (a.acc_out) a.acc_out[idx] = val;
                            if (a.y) {
                                bool sat;
                                const int c = act_one(val, a.act, sat);
                                if (a.y16) ((int16_t *)a.y)[idx] = (int16_t)c;
                                else ((int8_t *)a.y)[idx] = (int8_t)c;
                                nz += (c == 0);
                                ns += sat;
                            }
                        }
                    }
                }
            }
    }
    return {nz, ns};
}


// corr[co] = 128 * sum_k w[co][k] for two-limb activations, 0 otherwise: the weight half of the offset correction, computed
// once when the weights are packed.  One wave per output channel (blockIdx.x = co, 64 threads), lanes striding over K.
// Two-limb weights: plus kSignedForm if none of the channel's weights is too large for it (padded channels have none).
template <typename WT>
__global__ __launch_bounds__(64) void weight_corr_kernel(const WT *__restrict__ w, int64_t *__restrict__ corr, int Cout,
                                                        int CoutP, int K, int limbs, int wlimbs)
{
    const int co = blockIdx.x;
    if (co >= CoutP) return;
    long long s = 0;
    bool large = false;
    if (limbs == 2 && co < Cout)
        for (int k = threadIdx.x; k < K; k += 64) {
            const int v = (int)w[(size_t)co * K + k];
            s += v;
            large |= v >= 32640;
        }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_down(s, off, 64);
    const int64_t form = wlimbs == 2 && !__any(large) ? kSignedForm : 0;
    if (threadIdx.x == 0) corr[co] = 128 * s | form;
}

// A tile of 64 channels (blockIdx.x, 64 threads) takes the signed form if all of them can; else the corrections get the
// plain form's - 16384 * K.  Between weight_corr_kernel and the packing kernel, which reads the form there.
static __global__ __launch_bounds__(64) void weight_form_kernel(int64_t *__restrict__ corr, int Cout, int K)
{
    const int co = blockIdx.x * 64 + threadIdx.x;
    const int64_t v = corr[co];
    if (__all((v & kSignedForm) != 0)) return;
    corr[co] = co < Cout ? (v & ~kSignedForm) - (int64_t)16384 * K : 0;
}

// Adds n per-workgroup counts (zeros at partials[0..n), clipped values at partials[n..2n)) to the
// caller's counters (either may be null); defined with the convolution kernels.
lp_status launch_sum_partials(const unsigned *partials, int n, unsigned long long *zero_count,
                              unsigned long long *sat_count, hipStream_t st);

// LPInnerProduct through the convolution kernels (a 1x1 convolution over 1x1 images): the route
// for operand widths the inner-product kernel does not take.
lp_status fc_conv_packed_bytes(int M, int K, int Nout, lp_qfmt qx, lp_qfmt qw, size_t *bytes_host);
lp_status fc_conv_pack_weights(int M, int K, int Nout, lp_qfmt qx, lp_qfmt qw, const void *w_codes_dev,
                               void *packed_dev, size_t packed_bytes, void *stream);
lp_status fc_conv_workspace_bytes(int M, int K, int Nout, lp_qfmt qx, lp_qfmt qw, size_t *bytes_host);
lp_status fc_conv_fwd(int M, int K, int Nout, const void *x_codes_dev, lp_qfmt qx, const void *w_packed_dev,
                      lp_qfmt qw, const void *bias_codes_dev, lp_qfmt qb, int64_t *acc_out_dev,
                      void *y_codes_dev, lp_qfmt qy, int relu, lp_round r, uint64_t *zero_count_dev,
                      uint64_t *sat_count_dev, void *workspace_dev, size_t workspace_bytes, void *stream);

} // namespace lp
