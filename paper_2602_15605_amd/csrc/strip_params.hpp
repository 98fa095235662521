// Parameters of the strip kernels and the packed-triangle indexing they share
// with the fill, bin and batched kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace couple {

// Lanes of a wavefront on CDNA4.
constexpr int kWave = 64;

// Number of consecutive l1 values a lane of the strip kernel owns.  The
// G/H windows slide by one per l3 step, so each step loads one new G and
// one new H value per lane for R terms.
constexpr int kStripR = 4;
// The TT-only sum costs two operations per term, so there the two window
// reads per step dominate; eight rows per lane halve them per term.
constexpr int kStripRTT = 8;
// Launches that would have fewer work items of 64 R rows than these take
// kStripRSmall rows per lane, four times as many items with a quarter of the
// staircase each: float32 below 8192 items (full triangle: lmax <= 1918),
// float64 below 4096 (lmax <= 1321), where the measured crossovers lie; above them the
// longer rows per lane win.
constexpr int kStripRSmall = 2;
constexpr long long kStripSmallItemsF32 = 8192;
constexpr long long kStripSmallItemsF64 = 4096;

// Band-limited grids run in phases of this many consecutive diagonals, the
// phases in order of d and each phase block by block.  A diagonal's trip,
// (l3_hi - d)/2 steps for all but its lowest-l1 block, falls with d, so the
// phases run longest first; inside a phase, waves dispatched together share
// their block's g and h windows.  Measured on the 10^4 / l3 <= 1000 band
// (FP32C, FP64 strip per mask): 0.406 / 0.708 ms with all diagonals of a block
// in turn, 0.394 / 0.707 diagonal by diagonal, 0.383 / 0.680 with 256-diagonal
// phases and 0.377 / 0.677 with 64.
constexpr int kBandPhase = 64;

// l3 steps staged in LDS per chunk by the float64 and float32 strip kernels.
constexpr int kStripChunkF64 = 256;
constexpr int kStripChunkF32 = 256;
// Masks per launch of the multi-mask float32 kernel: at most 4 (one float4
// lane each).  Its sums take 16 VGPRs per mask and spectrum (four rows, block,
// mid and Kahan pair).  TT + EE with four masks needs 230 VGPRs (two waves per
// SIMD, as the 14 KB of LDS would allow at most 2.75): on the 8-mask 10^4 band
// it ran 1.75 ms against 2.18 ms with two masks per launch (156 VGPRs, three
// waves).  TT + TE + EE takes three (228 VGPRs; four would need 256, one
// wave): the 32-mask batched call's strip ran 12.5 ms against 13.4 ms with two.
constexpr int kBandMasks = 4;
constexpr int kMasksPolEE = 4;
constexpr int kMasksPol = 3;
// The float64 multi-mask kernel (one float64 sum per mask, spectrum and row;
// 248 VGPRs for TT + EE with four masks, two waves per SIMD).  On the 8-mask
// 10^4 band (strip per call): 2.45 ms with four masks per launch and 128-step
// chunks, 2.49 ms with 64-step chunks, 3.07 / 3.39 ms with three / two masks,
// against 5.37 ms for one launch per mask.
constexpr int kMasksPolEEF64 = 4;
constexpr int kMasksPolF64 = 2;
constexpr int kStripChunkF64Masks = 128;

// float32 strip kernel: steps per exact split of t = c - (a + b - 1).  Within
// one split the staged D(k) = c(l3) - c(l3 at the split) is below
// 254 (2 l3 + 255) < 2^24 for l3 <= 2 x 16384, hence exact in float32.
constexpr int kStripRebase = 128;

// Above this lmax the float64 strip kernels form N' by n_shift and n_rest below
// (one more operation per step), since a(a-2) + b(b-2) no longer fits 2^53.
constexpr int kNarrowLmax = 8000;

// The float64 whole-triangle kernels (tile.hip) against the diagonal strips, per
// strip mode, in us per call of couple_matrix (strips / tiles):
//   lmax                        1000       1200       1500       2000        3000
//   TT                          -          98 / 52    130 / 70   227 / 110   584 / 276
//   TT + TE + EE                119 / 147  168 / 179  261 / 248  511 / 443   1526 / 1271
//   TT + EE                     99 / 104   138 / 132  220 / 186  434 / 348   -
//   EE                          79 / 99    114 / 118  179 / 162  369 / 285   1090 / 797
//   EB                          89 / 87    127 / 102  200 / 153  407 / 268   1220 / 748
// Small triangles leave the tiles' longer patches without enough waves; TT's stay
// ahead at every size.
constexpr int kTileMinPol = 1400, kTileMinPolEE = 1150, kTileMinEE = 1250, kTileMinEB = 1000;
// lmax from which a thread takes 4 x 2 and 4 x 4 (s, d) values instead of 2 x 2 (us at lmax
// 2200 / 2400 / 2800 / 3000 with 2 x 2, 4 x 2 and 4 x 4:
//   TT + TE + EE   547 703 1098 1339,   566 674 1028 1253,   725 836 1074 1254
//   TT + EE        437 559  862 1042,   463 551  827 1000,   586 674  850  982
//   EE             361 457  702  848,   375 440  667  803,   469 537  673  777
//   EB             327 426  642  776,   366 425  630  760,   450 513  636  732),
// and a wave of the TT kernel 2 x 2 and 4 x 2 MFMA tiles instead of one (2000 / 3000 /
// 10^4: 110 / 286 / 8499 us with one, 153 / 276 / 6785 with 2 x 2, 209 / 361 / 6652 with 4 x 2).
constexpr int kTilePolMid = 2400, kTilePolBig = 2900;
constexpr int kTileTTMid = 2700, kTileTTBig = 6000;

// Zero guard band around the device copies of g(p) and 1/((2p+1)g(p)).
constexpr int kTablePad = 64;

// Offset of diagonal d of the packed upper-triangle store for lmax:
// diagonal d holds Xi(l1, l1 + d) for l1 = 0 .. lmax - d.
__host__ __device__ inline long long diag_offset(int lmax, int d) {
    return (long long)d * (lmax + 1) - (long long)d * (d - 1) / 2;
}
__host__ __device__ inline long long tri_size(int lmax) {
    return (long long)(lmax + 1) * (lmax + 2) / 2;
}

// The (-2 2 0) polynomial as a product and a rest (tile.hip): with s = l1 + l2, d =
// l2 - l1 and any integer a,
//     N' = (c - (s+1)^2 + 1 + a)(c - d^2 + 2 - a) + rest(s, d, a).
// For a near (1 - 1/sqrt 2)/2 ((s+1)^2 - d^2) the rest nearly vanishes, and over a
// patch of 512 rows of a diagonal, or 128 values of s and of d, around the (s, d)
// that a is taken from it stays below 2^52 up to lmax = 16384 (with a = 0 it passes
// 2^53 beyond lmax = 8000): exact in float64, so that N' is one fused
// multiply-add, rounded once.
__device__ inline long long n_shift(long long s, long long d) {
    const long long x = (s + 1) * (s + 1) - d * d;
    return x > 0 ? (long long)(0.14644660940672624 * (double)x) : 0;
}
__device__ inline long long n_rest(long long s, long long d, long long a) {
    const long long S = (s + 1) * (s + 1), D = d * d;
    return ((S - D) * (S - D) + 6 * S - 2 * D - 7) / 8 - a * (S - D + 1) + a * a;
}

// Strip kernel modes: Xi_TT; Xi_TT, Xi_TE, Xi_EE (even L); Xi_EB (odd L).
enum { kStripTT = 0, kStripPol = 1, kStripEB = 2, kStripPolEE = 3, kStripEE = 4 };

}  // namespace couple
