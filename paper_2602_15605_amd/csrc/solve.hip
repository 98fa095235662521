// Binned MASTER solve (Sec. 2, eq. pseudo_cl).
//
// The expectation of the pseudo-spectra is linear in the true spectra:
//   <C~^TT> = K^TT C^TT,
//   <C~^EE> = K^EE C^EE + K^EB C^BB,   <C~^BB> = K^EB C^EE + K^BB C^BB
// (the B-mode line by the structure App. A states: Xi_BB has the form of
// Xi_EE and Xi_BE = Xi_EB).  With the binning of couple_band (row-bin
// average, column-bin sum, C_l constant inside a bin) the binned system is
// K_{b b'} C_{b'} = C~_b, C~_b = (1/n_b) sum_{l in b} C~_l.
//
// bin_spectra_kernel: one thread per (spectrum, bin), the bin's sum in l order.
//
// The solve is Gaussian elimination with partial pivoting (largest |pivot|,
// the first row on ties) on the augmented matrix [K | C~] (TT, or the 2 x 2
// block system for E/B) in the caller's workspace, then back substitution.
// The workspace holds the matrix by columns (entry (r, c) at c m + r), so that
// threads over rows, which the panels, the updates and the back substitution
// all have, read consecutive addresses.
//
// Panels are factorised in registers (factor_rows): a thread owns whole rows of
// the panel (RPT rows of NB columns, 64 doubles at most), so a column step
// needs the pivot search and one broadcast row.  Per column, each wave finds its
// largest entry (16-lane DPP maxima of the high words; the low words and the row
// numbers only on ties) and leaves its row in LDS, one barrier, and every wave
// picks the winner among the waves' candidates; two LDS buffers in turn need no
// second barrier.  Rows are not moved: a thread keeps
// the position its row has after the exchanges.
//
// Systems of up to kTinyMax unknowns are one panel: each work-group factorises it for
// its share of the right-hand sides (master_solve_tiny_kernel).
// Small systems (m < kMultiMin and few right-hand sides) run in one work-group
// (master_solve_kernel), with L21 and U12 staged in LDS and the trailing update on the
// matrix cores.
// Others split the matrix into outer panels of kOuterNB columns:
//   solve_assemble_kernel     [K | C~] into the workspace, by columns;
//   solve_panel_kernel        one work-group factorises NB columns (32 while the
//                             panel has at most 1024 rows, 16, 8, 4, 2 for taller
//                             ones) and applies their exchanges and U12 to the
//                             outer panel's other columns; a panel of fewer than
//                             kOuterNB columns is followed by an update of the
//                             outer panel's later columns; the other work-groups of
//                             its launches do the update that the previous outer
//                             panel left waiting (below);
//   solve_swap_trsm_kernel    right of the outer panel, one thread per column:
//                             the panel's row exchanges, composed into one
//                             permutation of the touched rows, then
//                             U12 = L11^-1 A12;
//   solve_update_kernel       A22 -= L21 U12 in 64 x 64 tiles on the float64
//                             matrix cores (v_mfma_f64_16x16x4: each entry is a
//                             chain of fused multiply-adds in column order), for the
//                             next outer panel's columns; the columns right of those
//                             wait and are updated beside that panel's factorisation,
//                             which keeps one compute unit busy and leaves 255;
//   solve_back_block_kernel,  back substitution: one work-group solves a block of
//   solve_back_above_kernel   kBackRows rows, then every row above it is updated.
// The panel's pivots travel from the panel kernel to the swap kernel in the
// first kOuterNB entries of x, and x[kOuterNB] is a singular flag that every
// later kernel reads first; the last swap kernel copies it to the workspace's
// entry (m - 1, 0), an entry of L that is no longer read, for the back
// substitution, which overwrites x.
// A zero pivot (a singular system) gives NaN in every output.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "couple_internal.hpp"

namespace couple {
namespace {

constexpr int kSolveThreads = 512;
constexpr int kSolveWaves = kSolveThreads / kWave;
constexpr int kTallThreads = 1024;           // the panel kernel for more than 16 x kSolveThreads rows
constexpr int kMostWaves = kTallThreads / kWave;
typedef double d4v __attribute__((ext_vector_type(4)));

struct BinSpecArgs {
    const double* cl;            // [n_spec][cl_stride]
    long long cl_stride;
    double* out;                 // [n_spec][n_bins]
    const int* edges_dev;        // n_bins + 1 edges on the device (n_bins > kInlineBins)
    int inline_edges;
    int edges_in[kInlineBins + 1];
    int n_spec, n_bins;
};

__global__ void __launch_bounds__(256) bin_spectra_kernel(BinSpecArgs a) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= a.n_spec * a.n_bins) return;
    const int s = t / a.n_bins, b = t - s * a.n_bins;
    const int* E = a.inline_edges ? a.edges_in : a.edges_dev;
    const int lo = E[b], hi = E[b + 1];
    const double* c = a.cl + (long long)s * a.cl_stride;
    double acc = 0.0;
    for (int l = lo; l < hi; ++l) acc += c[l];
    a.out[(long long)s * a.n_bins + b] = acc / (double)(hi - lo);
}

struct SolveArgs {
    const double* K;             // TT: [n][n]; E/B: [3][n][n] in the order EE, BB, EB
    const double* rhs;           // [n_rhs][m]
    double* work;                // [m + n_rhs][m]: the augmented matrix by columns
    double* x;                   // [n_rhs][m]
    int n, m, n_rhs, pol;
};


// Entry (r, c) of the augmented matrix [K | C~]: TT, or [EE EB; EB BB] for E/B.
__device__ inline double assembled(const SolveArgs& a, int r, int c) {
    if (c >= a.m) return a.rhs[(long long)(c - a.m) * a.m + r];
    if (!a.pol) return a.K[(long long)r * a.n + c];
    const int n = a.n, br = r / n, bc = c / n;
    const int blk = br != bc ? 2 : br;
    return a.K[((long long)blk * n + (r - br * n)) * n + (c - bc * n)];
}

// The value of lane i (the same i in every lane) in every lane, from registers.
__device__ inline double lane_value(double v, int i) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), i);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), i);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The value of lane i of each row of 16 lanes, in every lane of the row
// (row_newbcast; i a constant once the caller's loop is unrolled).
template <int I>
__device__ __forceinline__ double row16_lane(double v) {
    return __builtin_amdgcn_update_dpp(0.0, v, 0x150 + I, 0xf, 0xf, true);
}
__device__ __forceinline__ double row16_bcast(double v, int i) {
    switch (i & 15) {
    case 0: return row16_lane<0>(v);
    case 1: return row16_lane<1>(v);
    case 2: return row16_lane<2>(v);
    case 3: return row16_lane<3>(v);
    case 4: return row16_lane<4>(v);
    case 5: return row16_lane<5>(v);
    case 6: return row16_lane<6>(v);
    case 7: return row16_lane<7>(v);
    case 8: return row16_lane<8>(v);
    case 9: return row16_lane<9>(v);
    case 10: return row16_lane<10>(v);
    case 11: return row16_lane<11>(v);
    case 12: return row16_lane<12>(v);
    case 13: return row16_lane<13>(v);
    case 14: return row16_lane<14>(v);
    default: return row16_lane<15>(v);
    }
}

// Largest of v over each row of 16 lanes (all lanes active), by rotations of 8, 4, 2 and 1.
__device__ inline unsigned row16_max(unsigned v) {
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, true));   // row_ror:8
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, true));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xf, 0xf, true));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xf, 0xf, true));
    return v;
}

// Largest of v over the wave: over each row of 16 lanes, then the four rows' results on the scalar unit.
__device__ inline unsigned wave_max(unsigned v) {
    v = row16_max(v);
    const unsigned a = __builtin_amdgcn_readlane((int)v, 0), b = __builtin_amdgcn_readlane((int)v, 16);
    const unsigned c = __builtin_amdgcn_readlane((int)v, 32), d = __builtin_amdgcn_readlane((int)v, 48);
    return max(max(a, b), max(c, d));
}

// Whether the high word of a magnitude has an exponent in [-1000, 1000]: its
// reciprocal and the correction step of a quotient are then finite and normal.
__device__ inline bool plain_exponent(unsigned hi) { return (hi >> 20) - 23u <= 2000u; }

// LDS of factor_rows.
template <int NB>
struct PivotLds {
    double blk[NB][NB + 2];       // row j of the factorised top block (L11 and U11), in the register order of step j
    double cand[2][NB < 4 ? kMostWaves : kSolveWaves][NB + 2];   // each wave's candidate row
    int4 key[2][kMostWaves];      // high and low word of its |pivot|, its position
    int piv[NB];                  // row exchanged with row j at step j (panel rows)
    int sing;                     // the panel met a zero pivot
};

// The rows of a panel that a thread holds: row threadIdx.x + q stride in a[q].
// A row leaves when it becomes a pivot (step = its column; its live columns go
// to PivotLds::blk); from then on it takes no part: in panels of 32 columns the
// search and the multiplier skip it, in narrower ones, which have more rows than
// columns per thread, its live columns are set to 0.  step is -1 before that, and
// NB where there is no row.  pos is the position of row q = 0, which only an
// exchange with one of the panel's first NB rows changes.  Other rows stay
// where they are until they leave.
template <int NB, int RPT>
struct PanelRows {
    double a[RPT][NB];
    int step[RPT];
    int stride, pos;
    __device__ __forceinline__ int row(int q) const { return (int)threadIdx.x + q * stride; }
    __device__ __forceinline__ int position(int q) const { return q == 0 ? pos : row(q); }
};

// Column jj of factor_rows, J of its block of GB in the register window, whose
// first live entries are the block's columns and those after it.
template <int NB, int RPT, int GB, int J>
__device__ __forceinline__ void factor_column(PanelRows<NB, RPT>& R, int jj, int live, int waves, PivotLds<NB>& S) {
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    // the wave's largest entry (high words, low words only on ties), its lane w
    constexpr bool kSkip = NB == 32;          // rows that left are skipped, not zeroed
    double mx = 0.0;
#pragma unroll
    for (int q = 0; q < RPT; ++q) mx = fmax(mx, kSkip && R.step[q] >= 0 ? 0.0 : fabs(R.a[q][J]));
    const long long bits = __double_as_longlong(mx);
    const unsigned hi = (unsigned)(bits >> 32), lo = (unsigned)bits;
    unsigned kh = wave_max(hi);
    bool in = hi == kh;
    unsigned long long cand = __ballot(in);
    if (cand & (cand - 1)) {
        const unsigned ml = wave_max(in ? lo : 0u);
        in = in && lo == ml;
        cand = __ballot(in);
        if (cand & (cand - 1)) {
            int bp = 0x7fffffff;                      // the first row on ties
#pragma unroll
            for (int q = 0; q < RPT; ++q)
                if (fabs(R.a[q][J]) == mx && R.step[q] < 0) bp = min(bp, R.position(q));
            const unsigned key = 0x7fffffffu - (unsigned)bp, best = wave_max(in ? key : 0u);
            cand = __ballot(in && key == best);
        }
    }
    const int w = __ffsll((long long)cand) - 1;
    unsigned kl = __builtin_amdgcn_readlane((int)lo, w);
    // which of the lane's rows, and its position
    int wq = 0, p = 0x7fffffff;
    if (RPT == 1) {
        p = __builtin_amdgcn_readlane(R.pos, w);
    } else {
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const bool is = __ballot(fabs(R.a[q][J]) == mx && R.step[q] < 0) >> w & 1;
            const int pq = q == 0 ? __builtin_amdgcn_readlane(R.pos, w) : wave * kWave + w + q * R.stride;
            if (is && pq < p) {
                p = pq;
                wq = q;
            }
        }
    }
    // the wave's candidate row and its key
    constexpr int buf = J & 1;
    double* mine_row = S.cand[buf][wave];
#pragma unroll
    for (int q = 0; q < RPT; ++q)
        if (q == wq) {
            if (lane == w) {
#pragma unroll
                for (int g = 0; g < NB; g += GB) {
                    if (g > 0 && g >= live) continue;
#pragma unroll
                    for (int c = g; c < g + GB; ++c) mine_row[c] = R.a[q][c];
                }
            }
            // the branches stay apart: merged, they would index a in scratch
            if (RPT > 1) asm volatile("; row %0" ::"s"(q));
        }
    int cw = 0;
    if (waves > 1) {
        if (lane == 0) S.key[buf][wave] = make_int4((int)kh, (int)kl, p, 0);
        __syncthreads();
        const int4 k = S.key[buf][lane < waves ? lane : 0];
        // the candidates' largest (at most 16: one row of lanes; copies of the first fill it up)
        const unsigned h = row16_max((unsigned)k.x);
        const unsigned mh = __builtin_amdgcn_readfirstlane((int)h);
        bool on = lane < waves && (unsigned)k.x == mh;
        unsigned long long c = __ballot(on);
        if (c & (c - 1)) {
            const unsigned ml = __builtin_amdgcn_readfirstlane((int)row16_max(on ? (unsigned)k.y : 0u));
            on = on && (unsigned)k.y == ml;
            c = __ballot(on);
            if (c & (c - 1)) {
                const unsigned key = 0x7fffffffu - (unsigned)k.z;
                const unsigned best = __builtin_amdgcn_readfirstlane((int)row16_max(on ? key : 0u));
                c = __ballot(on && key == best);
            }
        }
        cw = __ffsll((long long)c) - 1;
        kh = mh;
        kl = __builtin_amdgcn_readlane(k.y, cw);
        p = __builtin_amdgcn_readlane(k.z, cw);
    } else {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    const double* r = S.cand[buf][cw];
    const double r0 = r[lane % (NB < 16 ? NB : 16)];
    const double r1 = NB > 16 ? r[16 + lane % 16] : 0.0;
    // the pivot row leaves
    if (cw == wave) {
        if (lane < (NB < 16 ? NB : 16)) {
            S.blk[jj][lane] = r0;
            if (NB > 16) S.blk[jj][16 + lane] = r1;
        }
        if (lane == 0) {
            S.piv[jj] = p;
            if ((kh | kl) == 0) S.sing = 1;
        }
        if (kSkip) {
#pragma unroll
            for (int q = 0; q < RPT; ++q) R.step[q] = q == wq && lane == w ? jj : R.step[q];
        } else if (lane == w) {
#pragma unroll
            for (int q = 0; q < RPT; ++q)
                if (q == wq) {
#pragma unroll
                    for (int g = 0; g < NB; g += GB) {
                        if (g > 0 && g >= live) continue;
#pragma unroll
                        for (int c = g; c < g + GB; ++c) R.a[q][c] = 0.0;
                    }
                    R.step[q] = jj;
                    if (RPT > 1) asm volatile("; row %0" ::"s"(q));
                }
        }
    }
    R.pos = R.pos == jj ? p : R.pos;
    // a / |pivot|: from the reciprocal with one correction step, or by division
    const double apv = __longlong_as_double(((long long)kh << 32) | kl);
    const double inv = 1.0 / apv;
    double l[RPT];
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        l[q] = R.a[q][J] * inv;
        l[q] = __builtin_fma(__builtin_fma(-l[q], apv, R.a[q][J]), inv, l[q]);
    }
    if (!plain_exponent(kh)) {
#pragma unroll
        for (int q = 0; q < RPT; ++q) l[q] = R.a[q][J] / apv;
    }
    const double pv = row16_bcast(r0, J);
    const long long sign = __double_as_longlong(pv) & (1LL << 63);
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        R.a[q][J] = __longlong_as_double(__double_as_longlong(l[q]) ^ sign);
        l[q] = kSkip && R.step[q] >= 0 ? 0.0 : -R.a[q][J];
    }
    // the columns after jj, block by block
#pragma unroll
    for (int g = 0; g < NB; g += GB) {
        if (g > 0 && g >= live) continue;
        double u[GB];
#pragma unroll
        for (int c = g; c < g + GB; ++c)
            if (c > J) u[c - g] = row16_bcast(c < 16 ? r0 : r1, c);
#pragma unroll
        for (int c = g; c < g + GB; ++c)
#pragma unroll
            for (int q = 0; q < RPT; ++q)
                if (c > J) R.a[q][c] = __builtin_fma(l[q], u[c - g], R.a[q][c]);
    }
}

template <int NB, int RPT, int GB, int J>
__device__ __forceinline__ void factor_block(PanelRows<NB, RPT>& R, int j0, int nb, int waves, PivotLds<NB>& S) {
    if constexpr (J < GB) {
        if (j0 + J < nb) factor_column<NB, RPT, GB, J>(R, j0 + J, NB - j0, waves, S);
        factor_block<NB, RPT, GB, J + 1>(R, j0, nb, waves, S);
    }
}

// Factorise a panel of nb <= NB columns held in registers by the first `waves`
// waves, with partial pivoting.  Afterwards the rows that have not left hold
// their multipliers, S.blk the top block (entry (j, c) by top_entry) and S.piv
// the exchanges.  Every thread of the work-group calls this (waves beyond
// `waves` only keep the barriers company).  S.sing is set if a pivot column was
// zero or NaN: the caller checks it first, since positions and exchanges (never
// used as an address in here) then hold nothing of use.
// Columns run in blocks of 8 through one copy of the code, the registers rotated
// by a block after each (a copy per column would be 90 KB for 32 columns, more
// than the instruction cache holds).  What bounds it: the dependent chain of a
// column (search, one LDS exchange with a barrier, then the update): 3000 clocks for
// 8 waves of 2 x 32 or 8 x 8 entries per thread.
template <int NB, int RPT>
__device__ __forceinline__ void factor_rows(PanelRows<NB, RPT>& R, int nb, int waves, PivotLds<NB>& S) {
    constexpr int GB = NB < 8 ? NB : 8;
    if ((int)(threadIdx.x / kWave) >= waves) {
        if (waves > 1)
            for (int j = 0; j < nb; ++j) __syncthreads();
        __syncthreads();
        return;
    }
#pragma unroll 1
    for (int j0 = 0; j0 < NB; j0 += GB) {
        factor_block<NB, RPT, GB, 0>(R, j0, nb, waves, S);
        if (NB > GB) {
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                double t[GB];
#pragma unroll
                for (int c = 0; c < GB; ++c) t[c] = R.a[q][c];
#pragma unroll
                for (int c = 0; c < NB - GB; ++c) R.a[q][c] = R.a[q][c + GB];
#pragma unroll
                for (int c = 0; c < GB; ++c) R.a[q][NB - GB + c] = t[c];
            }
        }
    }
    __syncthreads();
}

// The factorised panel: put(r, c, v) for every entry that it holds, row
// positions r and columns c < nb.  The rows that have not left and the finished
// columns of the pivot rows (L11 left of the block of GB they left in) come
// from the registers, the rest of the top block from blk (at step j its columns
// had been rotated by whole blocks).
template <int NB, int RPT, class Put>
__device__ __forceinline__ void put_rows(const PanelRows<NB, RPT>& R, const PivotLds<NB>& S, int nb, Put put) {
    constexpr int GB = NB < 8 ? NB : 8;
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        if (R.step[q] < 0) {
            const int r = R.position(q);
#pragma unroll
            for (int c = 0; c < NB; ++c)
                if (c < nb) put(r, c, R.a[q][c]);
        } else if (NB > GB && R.step[q] >= GB && R.step[q] < NB) {
#pragma unroll
            for (int c = 0; c < NB - GB; ++c)
                if (c < R.step[q] / GB * GB) put(R.step[q], c, R.a[q][c]);
        }
    }
    for (int e = threadIdx.x; e < NB * NB; e += blockDim.x) {
        const int j = e % NB, c = e / NB;
        if (j < nb && c < nb && c >= j / GB * GB) put(j, c, S.blk[j][c - j / GB * GB]);
    }
}

// Panel rows (mr rows from row k0 on, columns k0 .. k0 + nb - 1) into the
// registers of the first `waves` waves; columns nb .. NB - 1 zero.
template <int NB, int RPT>
__device__ __forceinline__ void load_rows(PanelRows<NB, RPT>& R, const double* A, long long m, int k0, int mr, int nb,
                                          int waves) {
    R.stride = waves * kWave;
    R.pos = threadIdx.x;
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const bool in = R.row(q) < mr && (int)threadIdx.x < R.stride;
        const double* Ar = A + k0 * m + k0 + (in ? R.row(q) : 0);
        R.step[q] = in ? -1 : NB;
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            const double v = Ar[min(c, nb - 1) * m];
            R.a[q][c] = (in && c < nb) ? v : 0.0;
        }
    }
}

// The panel's exchanges for its other columns: src[i] = the row whose old values
// land in position i < nb, dst[i] = the position that old row i moves down to
// (-1 if it stays among the first nb); moved (cleared a barrier earlier) where
// any row moved.  One wave composes them from S.piv, lane i holding row i.
template <int NB>
__device__ inline void compose_moves(const PivotLds<NB>& S, int nb, int* src, int* dst, int* moved) {
    static_assert(NB <= 32, "two rows per lane pair");
    if (threadIdx.x >= kWave) return;
    const int l = threadIdx.x;
    // lanes 0 .. nb - 1: positions 0 .. nb - 1; lanes from nb on: positions below, as they are met
    int at = l < nb ? l : -1, from = at;      // position, and the row it holds
    int n = nb;
    bool any = false;
    const int piv = l < nb ? S.piv[l] : 0;
    for (int j = 0; j < nb; ++j) {
        const int p = __builtin_amdgcn_readlane(piv, j);
        if (p == j) continue;
        any = true;
        unsigned long long h = __ballot(at == p);
        if (!h) {
            if (l == n) at = from = p;
            h = 1ull << n++;
        }
        const int ip = __ffsll((long long)h) - 1;
        const int fj = __builtin_amdgcn_readlane(from, j), fp = __builtin_amdgcn_readlane(from, ip);
        if (l == j) from = fp;
        if (l == ip) from = fj;
    }
    if (l < nb) {
        src[l] = from;
        dst[l] = -1;
    }
    if (any && l == 0) *moved = 1;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (l >= nb && l < n && from < nb) dst[from] = at;
}

// u = L^-1 u for a unit lower triangle: row j, column i of it at lp[i ls + j], times sign.
template <int NB>
__device__ __forceinline__ void solve_lower(const double* lp, int ls, double sign, double (&u)[NB]) {
    int ofs = 0;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        asm volatile("" : "+v"(ofs), "+v"(u[i]));   // a column of L is read when its turn comes, not before
#pragma unroll
        for (int j = i + 1; j < NB; ++j) u[j] = __builtin_fma(sign * lp[ofs + i * ls + j], u[i], u[j]);
    }
}

// Column Ac of the matrix (from the panel's first row on): the panel's
// exchanges, then with `solve` U12 = L11^-1 A12, L11 read as lp[i ls + j] (row
// j, column i) times sign.  Every touched row is loaded before any is stored;
// u returns the first nb rows (rows nb .. NB - 1 hold nothing of use).
template <int NB>
__device__ inline void move_and_solve(double* Ac, int nb, bool moved, const int* src, const int* dst, const double* lp,
                                      int ls, double sign, bool solve, double (&u)[NB]) {
    if (moved) {
        double d[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            u[i] = Ac[src[min(i, nb - 1)]];
            d[i] = Ac[min(i, nb - 1)];
        }
#pragma unroll
        for (int i = 0; i < NB; ++i)
            if (i < nb && dst[i] >= 0) Ac[dst[i]] = d[i];
    } else {
#pragma unroll
        for (int i = 0; i < NB; ++i) u[i] = Ac[min(i, nb - 1)];
    }
    if (solve) solve_lower<NB>(lp, ls, sign, u);
#pragma unroll
    for (int i = 0; i < NB; ++i)
        if (i < nb) Ac[i] = u[i];
}

// 32 rows x 32 columns of A22 -= L21 U12 by one wave on the float64 matrix
// cores: load, multiply, store.  sl: -L21, depth k and row r at k ls + r; su:
// U12, depth k and column c at k us + c; nd: the depth, a multiple of 4.  CHAIN:
// the products are added to A22 one by one, as the elimination of a pivot row
// adds them, so that equal rows stay equal; else they are summed by themselves
// and added once (one rounding of A22 per panel, not one per column).  The tile is formed transposed (matrix columns as the MFMA's
// rows), so that an access's 16 lanes are 16 consecutive rows of one column: 128
// bytes.
template <bool CHAIN>
struct UpdateTile {
    d4v c22[2][2], acc[2][2];
    __device__ __forceinline__ void load(const double* A, long long m, long long row0, long long col0, long long row_end,
                                         long long col_end) {
        const int lane = threadIdx.x % kWave, r = lane % 16, q = lane / 16;
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const long long col = col0 + 16 * ct + q + 4 * i, row = row0 + 16 * rt + r;
                    c22[ct][rt][i] = (col < col_end && row < row_end) ? A[col * m + row] : 0.0;
                }
    }
    __device__ __forceinline__ void multiply(const double* sl, int ls, const double* su, int us, int nd) {
        const int lane = threadIdx.x % kWave, r = lane % 16, q = lane / 16;
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t / 2][t % 2] = CHAIN ? c22[t / 2][t % 2] : d4v{0.0, 0.0, 0.0, 0.0};
        for (int k = 0; k < nd; k += 4) {
            double x[2], y[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                x[t] = su[(k + q) * us + 16 * t + r];
                y[t] = sl[(k + q) * ls + 16 * t + r];
            }
#pragma unroll
            for (int ct = 0; ct < 2; ++ct)
#pragma unroll
                for (int rt = 0; rt < 2; ++rt)
                    acc[ct][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[ct], y[rt], acc[ct][rt], 0, 0, 0);
        }
    }
    __device__ __forceinline__ void store(double* A, long long m, long long row0, long long col0, long long row_end,
                                          long long col_end) const {
        const int lane = threadIdx.x % kWave, r = lane % 16, q = lane / 16;
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const long long col = col0 + 16 * ct + q + 4 * i, row = row0 + 16 * rt + r;
                    if (col < col_end && row < row_end) A[col * m + row] = CHAIN ? acc[ct][rt][i] : c22[ct][rt][i] + acc[ct][rt][i];
                }
    }
};

// Back substitution inside rows lo .. hi - 1 (hi - lo <= ROWS) for rc <= RHS
// right-hand sides from column m + r0 of A on: the block's solution goes back to those
// columns and to x.  In diagonal blocks of kBackBlock rows from the bottom: a wave solves
// the diagonal block (lanes over its rows) for RHS / kSolveWaves right-hand sides at a
// time, then threads over rows update the rest of the block.  load_u: false if L.u holds
// the one diagonal block already.
constexpr int kBackBlock = 64;
constexpr int kBackRows = 512;
constexpr int kBackRhs = kSolveWaves;
template <int RHS, int ROWS>
struct BackLds {
    double u[kBackBlock][kBackBlock + 1];    // a diagonal block of U: [column][row]
    double y[RHS][ROWS];
};
template <int RHS, int ROWS>
__device__ inline void back_block(double* A, long long m, int lo, int hi, int r0, int rc, double* x, BackLds<RHS, ROWS>& L,
                                  bool load_u) {
    constexpr int PER = RHS / kSolveWaves;
    const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
    for (int e = t; e < rc * ROWS; e += kSolveThreads) {
        const int c = e / ROWS, i = e % ROWS;
        if (lo + i < hi) L.y[c][i] = A[(m + r0 + c) * m + lo + i];
    }
    for (int ie = hi; ie > lo; ie -= kBackBlock) {
        const int ib = max(lo, ie - kBackBlock), bs = ie - ib;
        if (load_u)
            for (int e = t; e < kBackBlock * kBackBlock; e += kSolveThreads) {
                const int c = e / kBackBlock, r = e % kBackBlock;
                if (c < bs && r <= c) L.u[c][r] = A[(ib + c) * m + ib + r];
            }
        __syncthreads();
        if (wave < rc) {
            double y0[PER], xv[PER];
#pragma unroll
            for (int p = 0; p < PER; ++p)
                xv[p] = y0[p] = lane < bs && wave + p * kSolveWaves < rc ? L.y[wave + p * kSolveWaves][ib - lo + lane] : 0.0;
            const double ud = lane < bs ? L.u[lane][lane] : 1.0, uinv = 1.0 / ud;
            bool divide = !__all(plain_exponent((unsigned)(__double_as_longlong(ud) >> 32) & 0x7fffffffu));
            if (!divide) {
                // y / u from the reciprocal with one correction step
                for (int i = bs - 1; i >= 0; --i) {
                    const double u = lane_value(ud, i), v = lane_value(uinv, i);
                    const double ui = L.u[i][lane];
#pragma unroll
                    for (int p = 0; p < PER; ++p) {
                        const double yi = lane_value(xv[p], i);
                        double xi = yi * v;
                        xi = __builtin_fma(__builtin_fma(-xi, u, yi), v, xi);
                        xv[p] = lane == i ? xi : (lane < i ? __builtin_fma(-ui, xi, xv[p]) : xv[p]);
                    }
                }
                // the correction of an infinite quotient is NaN: the block is taken again
                bool finite = true;
#pragma unroll
                for (int p = 0; p < PER; ++p) finite = finite && __builtin_isfinite(xv[p]);
                divide = !__all(finite);
            }
            if (divide) {
#pragma unroll
                for (int p = 0; p < PER; ++p) {
                    xv[p] = y0[p];
                    for (int i = bs - 1; i >= 0; --i) {
                        const double xi = lane_value(xv[p], i) / lane_value(ud, i);
                        const double ui = L.u[i][lane];
                        xv[p] = lane == i ? xi : (lane < i ? __builtin_fma(-ui, xi, xv[p]) : xv[p]);
                    }
                }
            }
#pragma unroll
            for (int p = 0; p < PER; ++p) {
                const int c = wave + p * kSolveWaves;
                if (lane < bs && c < rc) {
                    L.y[c][ib - lo + lane] = xv[p];
                    A[(m + r0 + c) * m + ib + lane] = xv[p];
                    x[(long long)(r0 + c) * m + ib + lane] = xv[p];
                }
            }
        }
        __syncthreads();
        const int rows = ib - lo;
        for (int e = t; e < rows * rc; e += kSolveThreads) {
            const int c = e / rows, i = e - c * rows;
            const double* U = A + (long long)ib * m + lo + i;
            double acc = 0.0;
            int j = 0;
            for (; j + 16 <= bs; j += 16) {
                double v[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) v[k] = U[(long long)(j + k) * m];
#pragma unroll
                for (int k = 0; k < 16; ++k) acc = __builtin_fma(v[k], L.y[c][ib - lo + j + k], acc);
            }
            for (; j < bs; ++j) acc = __builtin_fma(U[(long long)j * m], L.y[c][ib - lo + j], acc);
            L.y[c][i] -= acc;
        }
        __syncthreads();
    }
}

constexpr int kOuterNB = 32;               // columns per outer panel
// Systems of at least this many unknowns, or with more right-hand sides than
// one_group_rhs allows, take the multi-work-group path (one work-group /
// several, us): 176 296 / 301, 192 330 / 317, 256 496 / 437, 320 724 / 577, 383 995 / 712.
constexpr int kMultiMin = 192;
constexpr int kOneRows = kMultiMin + 48;   // LDS row stride of L21 in the one-work-group path: the rows and a tile's
                                           // remainder, 16 mod 32 (no conflicts)
constexpr int kOneCols = 128;              // columns of U12 staged at a time there
constexpr int kOneColStride = kOneCols + 16;

// Right-hand sides up to which one work-group is ahead.  It takes them 16 at a time in the
// back substitution, the others spread them over the chip but take some 40 us per outer
// panel (one work-group / several, us): 33 unknowns with 64 of them 79 / 86; 48 with 32 84 / 86,
// 40 92 / 89; 64 with 16 90 / 92, 24 100 / 93; 65 with 32 126 / 138, 48 141 / 142; 80 with 24
// 144 / 140; 100 with 24 186 / 188, 32 193 / 191; 128 with 16 198 / 202, 24 226 / 203.
inline int one_group_rhs(int m) { return m <= 48 ? 64 : m <= 64 ? 16 : m <= 80 ? 32 : 16; }

// LDS of the one-work-group elimination.
struct OneLds {
    double l[kOuterNB][kOneRows];            // -L21 and -L11 by columns (rows of the panel)
    double u[kOuterNB][kOneColStride];       // U12
    PivotLds<kOuterNB> p;
    int src[kOuterNB], dst[kOuterNB], moved;
};

// Factorise one panel there: U11 to A, the multipliers to L.l, the exchanges to L.src and L.dst.
template <int RPT>
__device__ __forceinline__ void one_panel(double* A, long long m, int k0, int mr, int nb, int waves, OneLds& L) {
    constexpr int NB = kOuterNB;
    PanelRows<NB, RPT> R;
    load_rows<NB, RPT>(R, A, m, k0, mr, nb, waves);
    factor_rows<NB, RPT>(R, nb, waves, L.p);
    if (L.p.sing) return;                    // positions hold nothing of use then
    put_rows(R, L.p, nb, [&](int r, int c, double v) {
        L.l[c][r] = -v;
        if (r < nb) A[(k0 + c) * m + k0 + r] = v;
    });
    compose_moves(L.p, nb, L.src, L.dst, &L.moved);
}

// The whole solve in one work-group (kTinyMax < m < kMultiMin), the matrix in the caller's
// workspace (L2).  Bound by the panels' column chains (about 1 us per column).
__global__ void __launch_bounds__(kSolveThreads) master_solve_kernel(SolveArgs a) {
    constexpr int NB = kOuterNB;
    struct Tile {
        double v[kBackBlock][kBackBlock + 1];
    };
    __shared__ union Lds {
        OneLds e;
        Tile t;
        BackLds<kBackRhs, kMultiMin> b;
        BackLds<2 * kBackRhs, kMultiMin> b2;
    } S;
    const int t = threadIdx.x, wave = t / kWave;
    const int m = a.m, nr = a.n_rhs, ld = m + nr;
    double* A = a.work;

    // assemble [K | C~] by columns through LDS tiles
    for (int c0 = 0; c0 < ld; c0 += kBackBlock)
        for (int r0 = 0; r0 < m; r0 += kBackBlock) {
            for (int e = t; e < kBackBlock * kBackBlock; e += kSolveThreads) {
                // rows of K are contiguous; a right-hand side is contiguous over r
                const int r = e / kBackBlock, c = e % kBackBlock;
                if (r0 + r < m && c0 + c < ld) S.t.v[c][r] = assembled(a, r0 + r, c0 + c);
            }
            __syncthreads();
            for (int e = t; e < kBackBlock * kBackBlock; e += kSolveThreads) {
                const int c = e / kBackBlock, r = e % kBackBlock;
                if (r0 + r < m && c0 + c < ld) A[(long long)(c0 + c) * m + r0 + r] = S.t.v[c][r];
            }
            __syncthreads();
        }
    if (t == 0) S.e.p.sing = S.e.moved = 0;
    __syncthreads();

    bool singular = false;
    for (int k0 = 0; k0 < m; k0 += NB) {
        const int nb = min(NB, m - k0), mr = m - k0;
        {
            // at most 128 rows: two per lane of one wave, no barriers
            if (mr <= 2 * kWave)
                one_panel<2>(A, m, k0, mr, nb, 1, S.e);
            else
                one_panel<1>(A, m, k0, mr, nb, (mr + kWave - 1) / kWave, S.e);
        }
        __syncthreads();
        singular = S.e.p.sing != 0;
        if (singular) break;
        const bool moved = S.e.moved != 0;
        for (int c0 = k0 + nb; c0 < ld; c0 += kOneCols) {
            const int w = min(kOneCols, ld - c0);
            // the exchanges, the top block into S.e.u: a wave takes 8 x 8 entries at a time, so
            // that an access touches 8 columns (a thread per column touched 64: 31000 clocks
            // per panel at 118 unknowns, 16000 like this)
            const int r8 = t % 8, c16 = t / kWave * 16 + t % kWave / 8;
            double v[8], d[8];
            int to[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int i = 8 * g + r8;
                const int from = i < nb ? S.e.src[i] : 0;
                to[g] = moved && i < nb ? S.e.dst[i] : -1;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const double* Ac = A + (long long)(c0 + min(c16 + 8 * h, w - 1)) * m + k0;
                    v[2 * g + h] = Ac[from];
                    d[2 * g + h] = Ac[i < nb ? i : 0];
                }
            }
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int c = c16 + 8 * h;
                    S.e.u[8 * g + r8][c] = 8 * g + r8 < nb && c < w ? v[2 * g + h] : 0.0;
                    // every row of this column is read, by this wave, before any is written
                    if (to[g] >= 0 && c < w) A[(long long)(c0 + c) * m + k0 + to[g]] = d[2 * g + h];
                }
            __syncthreads();
            if (t < w) {
                double u[NB];
#pragma unroll
                for (int i = 0; i < NB; ++i) u[i] = S.e.u[i][t];
                solve_lower<NB>(&S.e.l[0][0], kOneRows, 1.0, u);
#pragma unroll
                for (int i = 0; i < NB; ++i) S.e.u[i][t] = u[i];
            }
            __syncthreads();
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int c = c16 + 8 * h;
                    if (8 * g + r8 < nb && c < w) A[(long long)(c0 + c) * m + k0 + 8 * g + r8] = S.e.u[8 * g + r8][c];
                }
            const int tr = (mr - nb + 31) / 32, tc = (w + 31) / 32;
            for (int e = wave; e < tr * tc; e += kSolveWaves) {
                const int ir = e % tr, ic = e / tr;
                UpdateTile<true> T;
                T.load(A, m, k0 + nb + 32 * ir, c0 + 32 * ic, m, c0 + w);
                T.multiply(&S.e.l[0][nb + 32 * ir], kOneRows, &S.e.u[0][32 * ic], kOneColStride, NB);
                T.store(A, m, k0 + nb + 32 * ir, c0 + 32 * ic, m, c0 + w);
            }
            __syncthreads();
        }
        if (t == 0) S.e.moved = 0;           // the next panel's barriers order this before its moves
    }

    if (singular) {
        for (long long e = t; e < (long long)nr * m; e += kSolveThreads) a.x[e] = __builtin_nan("");
        return;
    }
    __syncthreads();
    if (nr <= kBackRhs) {
        back_block(A, m, 0, m, 0, nr, a.x, S.b, true);
        return;
    }
    // two right-hand sides per wave take little longer than one (33 unknowns and 32 of them
    // 67 us per call, 75 with one): a step waits for its chain
    for (int r0 = 0; r0 < nr; r0 += 2 * kBackRhs) {
        __syncthreads();
        back_block(A, m, 0, m, r0, min(2 * kBackRhs, nr - r0), a.x, S.b2, r0 == 0 || m > kBackBlock);
    }
}

// Up to kTinyMax unknowns the matrix is one panel: the first wave of every work-group
// factorises it, straight from K, and each thread solves one right-hand side in registers.
// No workspace.  Bound by the launch and the columns' chains (0.7 us each): 1 / 16 / 32
// unknowns 8 / 15 / 30 us per call with up to 128 right-hand sides, 8 / 18 / 38 us with 4000.
// The one-work-group kernel, made for larger systems, took 15 / 28 / 40 us with one and 1212 /
// 2296 / 3327 us with 4000, which it solves eight at a time.
constexpr int kTinyMax = kOuterNB;
static_assert(kTinyMax >= kOuterNB, "the several work-groups keep a flag in column 0 beside the last outer panel");
constexpr int kTinyThreads = 256;
template <int NB>
__global__ void __launch_bounds__(kTinyThreads) master_solve_tiny_kernel(SolveArgs a) {
    __shared__ PivotLds<NB> P;
    __shared__ double lu[NB][NB];                // L below the diagonal and U, by columns
    __shared__ int src[NB], dst[NB], moved;
    const int t = threadIdx.x, m = a.m;
    PanelRows<NB, 1> R;
    R.stride = kWave;
    R.pos = t;
    const bool in = t < m;
    R.step[0] = in ? -1 : NB;
#pragma unroll
    for (int c = 0; c < NB; ++c) R.a[0][c] = in && c < m ? assembled(a, t, c) : 0.0;
    if (t == 0) P.sing = moved = 0;
    __syncthreads();
    factor_rows<NB, 1>(R, m, 1, P);
    const int q = blockIdx.x * kTinyThreads + t;
    double* x = a.x + (long long)q * m;
    if (P.sing) {                                // positions hold nothing of use then
        if (q < a.n_rhs)
            for (int i = 0; i < m; ++i) x[i] = __builtin_nan("");
        return;
    }
    put_rows(R, P, m, [&](int r, int c, double v) { lu[c][r] = v; });
    compose_moves(P, m, src, dst, &moved);
    __syncthreads();
    if (q >= a.n_rhs) return;
    const double* y = a.rhs + (long long)q * m;
    double u[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) u[i] = y[src[min(i, m - 1)]];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        if (i >= m) continue;
#pragma unroll
        for (int j = i + 1; j < NB; ++j) u[j] = __builtin_fma(-lu[i][j], u[i], u[j]);
    }
#pragma unroll
    for (int i = NB - 1; i >= 0; --i) {
        if (i >= m) continue;
        u[i] /= lu[i][i];
#pragma unroll
        for (int j = 0; j < i; ++j) u[j] = __builtin_fma(-lu[i][j], u[i], u[j]);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i)
        if (i < m) x[i] = u[i];
}

// ---------------------------------------------------------------------------
// Multi-work-group path (m > kTinyMax).
constexpr int kSingularSlot = kOuterNB;    // x[kSingularSlot]: an outer panel met a zero pivot
constexpr int kSwapCols = 64;              // columns per work-group of the swap + TRSM kernel
constexpr int kSwapThreads = 256;
static_assert(kWave % kOuterNB == 0, "a column's touched rows are read by one wave");
constexpr int kUpdTile = 64;               // the update kernel's tile: 4 waves of 32 x 32
constexpr int kUpdThreads = 256;
constexpr int kWaitRows = 128;             // rows of a tile of the waiting update
constexpr int kUpdStride = kUpdTile + 16;  // LDS stride of its operands (16 mod 32: no conflicts)
// Work-groups go to the XCDs in turn, so every eighth one of a launch lands beside
// work-group 0, the panel's.  With the panel's columns written from there the panel
// kernel loads 4000 x 8 entries in 10000 clocks; from all XCDs 25000.
constexpr int kXcds = 8;
constexpr int kAboveRows = 64;             // rows per work-group of solve_back_above_kernel
static_assert(kOuterNB <= kWave, "the swap kernel's mapping keeps two touched rows per lane of one wave");
// Systems of fewer unknowns add the products of an update one by one (UpdateTile), as the
// one-work-group path does, so that equal rows cancel exactly and give NaN.  Panels of
// one row per thread reach kSolveThreads rows; from 400 on the summed form keeps one
// rounding of A22 per panel.
constexpr int kChainBelow = 400;
static_assert(kChainBelow <= kSolveThreads, "their panels are 32 columns with one row per thread");
static_assert(kTinyMax >= kSingularSlot, "x must hold the pivots and the flag");
static_assert(kMultiMin <= kBackRows && kMultiMin <= kSolveThreads, "one row per thread and one back block below it");

struct OuterArgs {
    double* A;                   // the augmented matrix by columns: m + n_rhs columns of m
    double* x;                   // pivots of the outer panel in x[0 .. kOuterNB), the flag in x[kSingularSlot]
    long long ld;                // columns
    int m, k0, nbo;              // outer panel: columns k0 .. k0 + nbo - 1
    int kk, nb;                  // panel and update kernels: columns kk .. kk + nb - 1 of it
    long long c0, c1;            // update kernel: columns c0 .. c1 - 1
    int spread;                  // update kernel: one of `spread` work-groups has a tile
    int w0, row_tiles;           // panel kernel: its first tile of the waiting update, and that update's row tiles
    long long wc0;               // first column of the waiting update (panel k0 - kOuterNB, columns wc0 .. ld - 1)
};

// A22 -= L21 U12 for one tile of ROWS x kUpdTile entries from (rb, cb) on (columns below
// c1), L21 and U12 from panel columns kk .. kk + nb - 1, one 32 x 32 part per wave at a time.
template <int ROWS>
struct UpdateLds {
    double l[kOuterNB * (ROWS + 16)];        // -L21: [k][row]
    double u[kOuterNB * kUpdStride];         // U12: [k][column]
};
template <bool CHAIN, int ROWS>
__device__ __forceinline__ void update_tile(double* A, long long m, int kk, int nb, long long rb, long long cb,
                                            long long c1, int threads, UpdateLds<ROWS>& S) {
    constexpr int ls = ROWS + 16;
    const int t = threadIdx.x, nd = (nb + 3) / 4 * 4;
    for (int e = t; e < ROWS * nd; e += threads) {
        const int k = e / ROWS, r = e % ROWS;
        S.l[k * ls + r] = (k < nb && rb + r < m) ? -A[(kk + k) * m + rb + r] : 0.0;
    }
    for (int e = t; e < kUpdTile * nd; e += threads) {
        const int cc = e / nd, k = e - cc * nd;
        S.u[k * kUpdStride + cc] = (k < nb && cb + cc < c1) ? A[(cb + cc) * m + kk + k] : 0.0;
    }
    __syncthreads();
    for (int part = t / kWave; part < ROWS / 16; part += threads / kWave) {
        const int wr = 32 * (part % (ROWS / 32)), wc = 32 * (part / (ROWS / 32));
        if (rb + wr >= m || cb + wc >= c1) continue;
        UpdateTile<CHAIN> T;
        T.load(A, m, rb + wr, cb + wc, m, c1);
        T.multiply(S.l + wr, ls, S.u + wc, kUpdStride, nd);
        T.store(A, m, rb + wr, cb + wc, m, c1);
    }
}

// 32 x 32 tiles of [K | C~] through LDS, from rows of K to columns of the workspace.
constexpr int kAsmTile = 32;
__global__ void __launch_bounds__(256) solve_assemble_kernel(SolveArgs a) {
    __shared__ double v[kAsmTile][kAsmTile + 1];
    const int r0 = blockIdx.y * kAsmTile, c0 = blockIdx.x * kAsmTile;
    const int lo = threadIdx.x % kAsmTile, up = threadIdx.x / kAsmTile;
    const int ld = a.m + a.n_rhs;
#pragma unroll
    for (int q = 0; q < kAsmTile; q += 8)
        if (r0 + up + q < a.m && c0 + lo < ld) v[up + q][lo] = assembled(a, r0 + up + q, c0 + lo);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kAsmTile; q += 8)
        if (r0 + lo < a.m && c0 + up + q < ld) a.work[(long long)(c0 + up + q) * a.m + r0 + lo] = v[lo][up + q];
}

// One work-group factorises columns kk .. kk + nb - 1 (rows kk .. m - 1) of the
// outer panel in registers and applies the exchanges to the outer panel's
// other columns, with U12 for those on the right.  Bound by one compute unit's
// reach: of 60000 .. 65000 clocks for 8 columns of 3000 .. 4000 rows the column
// chains take 30000, the loads 10000 (see kXcds) and the stores 6000.  The other
// work-groups do the waiting update of the columns beyond, which took 65 us per outer
// panel by itself at 4000 rows and adds 3 us to each of four launches here: 4000
// unknowns 18.5 -> 17.0 ms, 9000 100 -> 84 ms; with the columns written from one XCD and
// one barrier per column 15.5 and 82.
template <int NB, int RPT, bool CHAIN = false, int T = kSolveThreads>
__global__ void __launch_bounds__(T) solve_panel_kernel(OuterArgs a) {
    struct Panel {
        PivotLds<NB> p;
        double l[NB][NB];                    // L11 by columns
        int src[NB], dst[NB], moved;
    };
    __shared__ union Lds {
        Panel f;
        UpdateLds<kWaitRows> u;
    } S;
    const int t = threadIdx.x;
    const int m = a.m, kk = a.kk, nb = a.nb, mr = m - kk;
    double* A = a.A;
    // the first panel clears the flag (not the assembly: x may be the right-hand side)
    if (kk == 0) {
        if (t == 0) a.x[kSingularSlot] = 0.0;
    } else if (a.x[kSingularSlot] != 0.0) {
        return;                              // an earlier panel was singular
    }
    if constexpr (T <= kSolveThreads) {
        if (blockIdx.x > 0) {
            const int w = a.w0 + (int)blockIdx.x - 1;
            update_tile<CHAIN>(A, m, a.k0 - kOuterNB, kOuterNB, a.k0 + (long long)(w % a.row_tiles) * kWaitRows,
                        a.wc0 + (long long)(w / a.row_tiles) * kUpdTile, a.ld, blockDim.x, S.u);
            return;
        }
    }
    PivotLds<NB>& P = S.f.p;
    double (&s_l)[NB][NB] = S.f.l;
    int (&s_src)[NB] = S.f.src;
    int (&s_dst)[NB] = S.f.dst;
    int& s_moved = S.f.moved;
    if (t == 0) P.sing = s_moved = 0;
    __syncthreads();
    const int waves = min((int)blockDim.x, mr + kWave - 1) / kWave;
    PanelRows<NB, RPT> R;
    load_rows<NB, RPT>(R, A, m, kk, mr, nb, waves);
    factor_rows<NB, RPT>(R, nb, waves, P);
    if (P.sing) {                            // positions hold nothing of use then
        if (t == 0) a.x[kSingularSlot] = 1.0;
        return;
    }
    put_rows(R, P, nb, [&](int r, int c, double v) {
        A[(long long)(kk + c) * m + kk + r] = v;
        if (r < NB) s_l[c][r] = v;
    });
    if constexpr (NB < kOuterNB) compose_moves(P, nb, s_src, s_dst, &s_moved);
    __syncthreads();
    if (t < nb) a.x[kk - a.k0 + t] = (double)(kk + P.piv[t]);
    if constexpr (NB < kOuterNB) {
        const int nleft = kk - a.k0, nother = nleft + (a.k0 + a.nbo - kk - nb);
        if (t < nother) {
            const int c = t < nleft ? a.k0 + t : kk + nb + (t - nleft);
            double u[NB];
            move_and_solve<NB>(A + (long long)c * m + kk, nb, s_moved != 0, s_src, s_dst, &s_l[0][0], NB, -1.0,
                               t >= nleft, u);
        }
    }
}

// Right of the outer panel, kSwapCols columns per work-group: the nbo row
// exchanges of the panel composed into one permutation of the rows they touch
// (the top block k0 .. k0+nbo-1 and at most nbo rows below it), applied by
// reading every source row before writing any, then U12 = L11^-1 A12 for the
// top block, one thread per column.  The top block passes through LDS both ways, so
// that memory is read and written along columns (a thread per column there
// touched 64 cache lines per access: 13.7 us per launch at 4000 unknowns, now 10.6).
__global__ void __launch_bounds__(kSwapThreads) solve_swap_trsm_kernel(OuterArgs a) {
    __shared__ double s_tile[kSwapCols][kOuterNB + 1];
    __shared__ double s_l[kOuterNB][kOuterNB];   // L11 by columns
    __shared__ int s_row[2 * kWave];             // touched rows: the top block first (two per lane)
    __shared__ int s_src[2 * kWave];             // the row whose old values land in s_row[i]
    const int t = threadIdx.x;
    const int k0 = a.k0, nbo = a.nbo;
    const long long m = a.m;
    const long long c0 = (long long)k0 + nbo;
    const double flag = a.x[kSingularSlot];
    // after the last panel: the flag moves into an entry of L that is no longer read
    if (c0 == m && blockIdx.x == 0 && t == 0) a.A[m - 1] = flag;
    if (flag != 0.0) return;
    for (int e = t; e < kOuterNB * kOuterNB; e += kSwapThreads) {
        const int c = e / kOuterNB, r = e % kOuterNB;
        s_l[c][r] = (c < nbo && r < nbo) ? a.A[(k0 + c) * m + k0 + r] : 0.0;
    }
    __shared__ int s_n;                          // touched rows (0: no row moves)
    if (t < kWave) {
        // one wave: lane i keeps touched rows i and i + 64 in registers; a ballot
        // finds where the pivot row sits
        const int l = t;
        int n = nbo;
        bool moved = false;
        int row0 = l < nbo ? k0 + l : -1, src0 = row0;
        int row1 = -1, src1 = -1;
        const int piv = l < nbo ? (int)a.x[l] : 0;       // all pivots in one load
        for (int j = 0; j < nbo; ++j) {
            const int p = __builtin_amdgcn_readlane(piv, j);
            if (p == k0 + j) continue;
            moved = true;
            const unsigned long long h0 = __ballot(row0 == p), h1 = __ballot(row1 == p);
            int ip;
            if (h0) {
                ip = __ffsll((long long)h0) - 1;
            } else if (h1) {
                ip = kWave + __ffsll((long long)h1) - 1;
            } else {
                ip = n++;
                if (l == ip - kWave) row1 = src1 = p;     // p > k0 + nbo - 1 here, so ip >= nbo
                if (ip < kWave && l == ip) row0 = src0 = p;
            }
            // swap the sources of positions j (< nbo <= 64) and ip
            const int sj = __shfl(src0, j);
            const int sip = ip < kWave ? __shfl(src0, ip) : __shfl(src1, ip - kWave);
            if (l == j) src0 = sip;
            if (ip < kWave) {
                if (l == ip) src0 = sj;
            } else if (l == ip - kWave) {
                src1 = sj;
            }
        }
        s_row[l] = row0;
        s_src[l] = src0;
        s_row[kWave + l] = row1;
        s_src[kWave + l] = src1;
        if (l == 0) s_n = moved ? n : 0;
    }
    __syncthreads();
    const int n = s_n;
    const long long cb = c0 + (long long)blockIdx.x * kSwapCols;
    const int w = (int)(a.ld - cb < kSwapCols ? a.ld - cb : kSwapCols);
    // lanes over the top block's rows, two columns per wave and pass
    constexpr int kPer = kSwapCols * kOuterNB / kSwapThreads;
    const int i = t % kOuterNB, g = t / kOuterNB;
    const bool top = i < nbo;
    double v[kPer], d[kPer];
    const int from = !top ? k0 : n ? s_src[i] : k0 + i;
    const bool down = nbo + i < n;
    const int dfrom = down ? s_src[nbo + i] : k0, dto = down ? s_row[nbo + i] : k0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int c = g + q * (kSwapThreads / kOuterNB);
        const double* Ac = a.A + (cb + min(c, w - 1)) * m;
        v[q] = Ac[from];
        if (n) d[q] = Ac[dfrom];
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int c = g + q * (kSwapThreads / kOuterNB);
        s_tile[c][i] = v[q];
        // each column's rows are all read (by lanes of this same wave) before this writes any
        if (down && c < w) a.A[(cb + c) * m + dto] = d[q];
    }
    __syncthreads();
    if (t < kSwapCols) {
        double u[kOuterNB];
#pragma unroll
        for (int r = 0; r < kOuterNB; ++r) u[r] = s_tile[t][r];
        solve_lower<kOuterNB>(&s_l[0][0], kOuterNB, -1.0, u);
#pragma unroll
        for (int r = 0; r < kOuterNB; ++r) s_tile[t][r] = u[r];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int c = g + q * (kSwapThreads / kOuterNB);
        if (top && c < w) a.A[(cb + c) * m + k0 + i] = s_tile[c][i];
    }
}

// A22 -= L21 U12 over rows kk+nb .. m-1 and columns c0 .. c1-1, depth nb:
// kUpdTile x kUpdTile entries per work-group, one 32 x 32 quarter per wave.
// Only the columns that are needed next (the others wait, see solve_panel_kernel): bound
// by its chain of loads, 5 .. 11 us per launch at 4000 unknowns.
template <bool CHAIN>
__global__ void __launch_bounds__(kUpdThreads) solve_update_kernel(OuterArgs a) {
    __shared__ UpdateLds<kUpdTile> S;
    if (a.x[kSingularSlot] != 0.0) return;
    // the next panel's columns: all tiles on the panel kernel's XCD, whose L2 then holds them
    if (blockIdx.x % a.spread) return;
    const long long rb = (long long)a.kk + a.nb + (long long)(blockIdx.x / a.spread) * kUpdTile;
    const long long cb = a.c0 + (long long)blockIdx.y * kUpdTile;
    update_tile<CHAIN>(a.A, a.m, a.kk, a.nb, rb, cb, a.c1, kUpdThreads, S);
}

struct BackArgs {
    double* A;
    double* x;                   // [n_rhs][m]
    int m, n_rhs, lo, hi;        // rows lo .. hi - 1 of this block
};

// kBackRhs right-hand sides per work-group.
__global__ void __launch_bounds__(kSolveThreads) solve_back_block_kernel(BackArgs a) {
    __shared__ BackLds<kBackRhs, kBackRows> L;
    const int r0 = blockIdx.x * kBackRhs, rc = min(kBackRhs, a.n_rhs - r0);
    if (a.A[a.m - 1] != 0.0) {                // singular
        for (int c = 0; c < rc; ++c)
            for (int i = a.lo + threadIdx.x; i < a.hi; i += kSolveThreads)
                a.x[(long long)(r0 + c) * a.m + i] = __builtin_nan("");
        return;
    }
    back_block(a.A, a.m, a.lo, a.hi, r0, rc, a.x, L, true);
}

// Rows r < lo of right-hand side blockIdx.y: y[r] -= sum over the block's columns
// of U[r][c] x[c]; kAboveRows rows per work-group, its waves take every fourth column.
__global__ void __launch_bounds__(256) solve_back_above_kernel(BackArgs a) {
    __shared__ double s_x[kBackRows];
    __shared__ double s_p[4][kAboveRows];
    const long long m = a.m;
    const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
    double* y = a.A + (m + blockIdx.y) * m;
    for (int i = t; i < a.hi - a.lo; i += 256) s_x[i] = y[a.lo + i];
    __syncthreads();
    const int r = blockIdx.x * kAboveRows + lane;
    double acc = 0.0;
    if (r < a.lo) {
        const double* U = a.A + (long long)a.lo * m + r;
#pragma unroll 8
        for (int c = wave; c < a.hi - a.lo; c += 4) acc = __builtin_fma(U[c * m], s_x[c], acc);
    }
    s_p[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && r < a.lo) y[r] -= (s_p[0][lane] + s_p[1][lane]) + (s_p[2][lane] + s_p[3][lane]);
}

}  // namespace

hipError_t launch_bin_spectra(const couple_ctx* ctx, int n_spec, const double* cl, int cl_stride,
                              const int* bin_edges_host, int n_bins, double* out, hipStream_t s) {
    BinSpecArgs a;
    a.cl = cl;
    a.cl_stride = cl_stride;
    a.out = out;
    a.edges_dev = ctx->edges_dev;
    a.inline_edges = n_bins <= kInlineBins ? 1 : 0;
    for (int i = 0; i <= kInlineBins; ++i) a.edges_in[i] = (a.inline_edges && i <= n_bins) ? bin_edges_host[i] : 0;
    a.n_spec = n_spec;
    a.n_bins = n_bins;
    const int total = n_spec * n_bins;
    hipLaunchKernelGGL(bin_spectra_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

// Workspace of couple_master_solve_noalloc: the [m][m + n_rhs] system lives in
// this file-scope device array instead of a caller or library allocation.
// Every GPU the library runs on holds its own copy until the process ends.
// Host code never passes the array's name to a kernel: it uses the device
// address that hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) double scratch[kNoallocSolveDoubles];

static std::mutex g_scratch_mutex;
static double* g_scratch_ptr[kMaxDevices] = {};

hipError_t noalloc_scratch(int device, double** ptr) {
    *ptr = nullptr;
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[device]) {
        // called with `device` current: the symbol resolves to that GPU's copy
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[device] = static_cast<double*>(p);
    }
    *ptr = g_scratch_ptr[device];
    return hipSuccess;
}

hipError_t launch_master_solve(int pol, int n, const double* K, int n_rhs, const double* rhs, double* work,
                               double* x, hipStream_t s) {
    SolveArgs a;
    a.K = K;
    a.rhs = rhs;
    a.work = work;
    a.x = x;
    a.n = n;
    a.m = pol ? 2 * n : n;
    a.n_rhs = n_rhs;
    a.pol = pol;
    if (a.m + n_rhs > kSolveMaxCols) return hipErrorInvalidValue;
    if (a.m <= kTinyMax) {
        const dim3 grid((unsigned)((n_rhs + kTinyThreads - 1) / kTinyThreads)), block(kTinyThreads);
        if (a.m <= 8)
            hipLaunchKernelGGL(master_solve_tiny_kernel<8>, grid, block, 0, s, a);
        else if (a.m <= 16)
            hipLaunchKernelGGL(master_solve_tiny_kernel<16>, grid, block, 0, s, a);
        else
            hipLaunchKernelGGL(master_solve_tiny_kernel<32>, grid, block, 0, s, a);
        return hipGetLastError();
    }
    if (a.m < kMultiMin && n_rhs <= one_group_rhs(a.m)) {
        hipLaunchKernelGGL(master_solve_kernel, dim3(1), dim3(kSolveThreads), 0, s, a);
        return hipGetLastError();
    }
    const int m = a.m;
    const long long ld = (long long)m + n_rhs;
    hipLaunchKernelGGL(solve_assemble_kernel,
                       dim3((unsigned)((ld + kAsmTile - 1) / kAsmTile), (unsigned)((m + kAsmTile - 1) / kAsmTile)),
                       dim3(256), 0, s, a);
    OuterArgs o;
    o.A = work;
    o.x = x;
    o.ld = ld;
    o.m = m;
    // columns of the widest panel whose rows fit in registers (64 doubles per thread)
    auto panel_width = [](int rows) {
        return rows <= 2 * kSolveThreads ? 32 : rows <= 4 * kSolveThreads ? 16 : rows <= 8 * kSolveThreads ? 8
               : rows <= 16 * kSolveThreads ? 4 : 2;
    };
    const bool chain = m < kChainBelow;
    auto update = [&](long long c0, long long c1) {
        const long long rows = m - (o.kk + o.nb);
        if (rows <= 0 || c1 <= c0) return;
        o.c0 = c0;
        o.spread = c1 - c0 <= kOuterNB ? kXcds : 1;
        o.c1 = c1;
        const dim3 grid((unsigned)((rows + kUpdTile - 1) / kUpdTile * o.spread), (unsigned)((c1 - c0 + kUpdTile - 1) / kUpdTile));
        if (chain)
            hipLaunchKernelGGL(solve_update_kernel<true>, grid, dim3(kUpdThreads), 0, s, o);
        else
            hipLaunchKernelGGL(solve_update_kernel<false>, grid, dim3(kUpdThreads), 0, s, o);
    };
    for (int k0 = 0; k0 < m; k0 += kOuterNB) {
        o.k0 = k0;
        o.nbo = std::min(kOuterNB, m - k0);
        const int ce = k0 + o.nbo;
        // chosen by the outer panel's first column
        const int nb = panel_width(m - k0);
        // the update that the previous outer panel left waiting, spread over this one's launches
        o.wc0 = ce;
        o.row_tiles = (m - k0 + kWaitRows - 1) / kWaitRows;
        const long long waiting = k0 && nb > 2 ? o.row_tiles * ((ld - ce + kUpdTile - 1) / kUpdTile) : 0;
        const int launches = (o.nbo + nb - 1) / nb;
        for (int kk = k0, i = 0; kk < ce; kk += nb, ++i) {
            o.kk = kk;
            o.nb = std::min(nb, ce - kk);
            o.w0 = (int)(waiting * i / launches);
            const dim3 grid(1 + (unsigned)(waiting * (i + 1) / launches - o.w0));
            const int mr = m - kk;
            if (chain)
                hipLaunchKernelGGL((solve_panel_kernel<32, 1, true>), grid, dim3((unsigned)((mr + kWave - 1) / kWave * kWave)), 0, s, o);
            else if (nb == 32 && mr <= kSolveThreads)
                hipLaunchKernelGGL((solve_panel_kernel<32, 1>), grid, dim3((unsigned)((mr + kWave - 1) / kWave * kWave)), 0, s, o);
            else if (nb == 32)
                hipLaunchKernelGGL((solve_panel_kernel<32, 2>), grid, dim3(kSolveThreads), 0, s, o);
            else if (nb == 16)
                hipLaunchKernelGGL((solve_panel_kernel<16, 4>), grid, dim3(kSolveThreads), 0, s, o);
            else if (nb == 8)
                hipLaunchKernelGGL((solve_panel_kernel<8, 8>), grid, dim3(kSolveThreads), 0, s, o);
            else if (nb == 4)
                hipLaunchKernelGGL((solve_panel_kernel<4, 16>), grid, dim3(kSolveThreads), 0, s, o);
            else
                hipLaunchKernelGGL((solve_panel_kernel<2, 16, false, kTallThreads>), grid, dim3(kTallThreads), 0, s, o);
            update(kk + o.nb, ce);               // the outer panel's later columns
        }
        o.kk = k0;
        o.nb = o.nbo;
        const unsigned col_groups = (unsigned)((ld - ce + kSwapCols - 1) / kSwapCols);   // >= 1: right-hand sides
        hipLaunchKernelGGL(solve_swap_trsm_kernel, dim3(col_groups), dim3(kSwapThreads), 0, s, o);
        // the next outer panel's columns now, the others beside its factorisation (not in the
        // panel kernel for two columns: its 1024 threads leave too few registers)
        update(ce, ce < m && panel_width(m - ce) > 2 ? std::min(ce + kOuterNB, m) : ld);
    }
    BackArgs b;
    b.A = work;
    b.x = x;
    b.m = m;
    b.n_rhs = n_rhs;
    for (b.hi = m; b.hi > 0; b.hi = b.lo) {
        b.lo = std::max(0, b.hi - kBackRows);
        hipLaunchKernelGGL(solve_back_block_kernel, dim3((unsigned)((n_rhs + kBackRhs - 1) / kBackRhs)), dim3(kSolveThreads),
                           0, s, b);
        if (b.lo > 0)
            hipLaunchKernelGGL(solve_back_above_kernel, dim3((unsigned)((b.lo + kAboveRows - 1) / kAboveRows), (unsigned)n_rhs),
                               dim3(256), 0, s, b);
    }
    return hipGetLastError();
}

}  // namespace couple
