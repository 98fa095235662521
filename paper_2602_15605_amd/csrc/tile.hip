// The float64 l3 reduction over a whole triangle as a matrix product.
//
// With s = l1 + l2 and d = l2 - l1 the squared (0 0 0) symbol factorises: the
// halved triangle combinations of eq. trianglecombos are p1, p2 = (l3 +- d)/2 and
// p, p3 = (s +- l3)/2, so by eq. 000_sq_main
//
//     (l1 l2 l3; 0 0 0)^2 = [g((l3-d)/2) g((l3+d)/2)] [g((s-l3)/2) h((s+l3)/2)],
//
// the first factor (with the window, U_X) a function of (l3, d) and the second
// (P) one of (l3, s).  For even L the three share their parity, so with s = 2 S +
// par, d = 2 D + par, l3 = 2 L + par every sum over l3 = d .. s is one over L = D
// .. S, and Xi_TT(S, D) = sum_L P(L, S) U(L, D) is a product of two matrices:
// tile_tt_kernel takes it on the float64 matrix cores, one multiply-add per term.
//
// The (-2 2 0) polynomial of strip.hip factorises the same way up to a constant:
//
//     N' = f e + G,  f = c - (s+1)^2 + 1 + a,  e = c - d^2 + 2 - a,
//
// all integers, f of (l3, s), e of (l3, d) and the rest G of (s, d); the tile's
// integer a keeps G exact (n_shift).  So N' is one fused multiply-add per term,
// rounded once.  tile_pol_kernel gives each thread a patch of s and d values, so
// that P, U and f, e serve several terms each:
// N', P N' and P N'^2 and one multiply-add per spectrum, 6 operations per term
// (TT + TE + EE) where a diagonal strip takes 8.  Odd L (EB) is the same with
// (s+1, d+1): P f1 U (c + mu)^2, 4 operations instead of 7.
//
// Per element the terms are those of the multi-mask strips in the same order (l3
// ascending, each sum one chain of fused multiply-adds; the matrix cores'
// float64 product is that chain too), so both give the same bits; but for EB's
// product, which the one-mask strips take in another order, strip_fp64_kernel's too.
//
// A work-group owns a tile of TS x TD (s, d) values of one parity and walks L in
// chunks; P and U of a chunk are staged in LDS.  Terms outside an element's own
// range are exact zeros (U = 0 below D and outside the band, g = 0 above S).  That
// holds for finite U only: window values that are infinite, NaN or so large that U
// could overflow (wild) are staged as 0, and a tile that met one adds their terms to
// its elements at the end, each to those whose sums hold it (add_wild).  Looking for
// them costs nothing that can be measured (TT at lmax 500 19.0 us, EE at 2700 597 us; as a
// second form of the steps it spilled registers), EE in 2 x 2 patches excepted (lmax 2000
// 285 us, 277 without).
#include <algorithm>

#include "couple_internal.hpp"

namespace couple {
namespace {

typedef double d4v __attribute__((ext_vector_type(4)));

constexpr int kTileThreads = 256;
constexpr int kTileChunk = 32;               // L values staged at a time

struct TileArgs {
    const double* g;     // g(p), 0 .. lmax_max, a zero on both sides
    const double* h;     // 1/((2p+1) g(p)), 0 .. 2 lmax_max, a zero on both sides
    const double* wp;    // scaled windows, 3 x wp_stride
    const double* cl;    // c_l
    double* xi;          // packed triangles, xi_stride apart
    long long xi_stride;
    int wp_stride;
    int g_len, h_len;    // lmax_max + 1, 2 lmax_max + 1
    int lmax;
    int l3_lo, l3_hi;
    int m_top;           // largest level
};

// One tile: parity, first S and D, and the L range (empty: no tile).
struct TileWhere {
    int par, S0, D0, L_lo, L_hi;
};

// Tiles of a level m = (TS/TD) I - J (I, J the tile's place along S and D) in one
// parity: those with l2 = S + D + par <= lmax somewhere, i.e. TS I + TD J + par <= reach
// (reach = lmax; for EB, where (s, d) stand for (l1 + l2 + 1, l2 - l1 + 1), lmax + 1).
// J runs from level_first in steps of TS/TD.
template <int TS, int TD>
__host__ __device__ inline int level_tiles(int reach, int m, int par) {
    constexpr int rho = TS / TD;
    static_assert(rho * TD == TS && (rho == 1 || rho == 2), "one or two D tiles per S tile");
    const int first = rho == 2 ? (m & 1) : 0;
    const int room = reach - par - TD * (m + 2 * first);      // TS I + TD J = TD (m + 2 J)
    return room < 0 ? 0 : room / (2 * rho * TD) + 1;
}

// Window values from 2^960 on, infinities and NaN stay out of the staged products (below
// that U stays below 2^1024: g <= 1, and EB's factor is below 2^31).
__device__ __forceinline__ bool wild(double w) { return !(fabs(w) < 0x1p960); }

// Work-group -> tile.  Tiles are numbered by level, the highest first: a tile runs
// about TD m + TS steps, so the longest start first, and without gaps: work-groups
// go to the eight XCDs in turn whatever they find to do, and a grid with empty
// places loaded them unevenly.
template <int TS, int TD>
__device__ inline bool tile_of(const TileArgs& a, int reach, TileWhere* w) {
    constexpr int rho = TS / TD;
    int i = blockIdx.x, m = a.m_top, n0 = 0;
    for (; m >= 1 - rho; --m) {
        n0 = level_tiles<TS, TD>(reach, m, 0);
        const int n = n0 + level_tiles<TS, TD>(reach, m, 1);
        if (i < n) break;
        i -= n;
    }
    if (m < 1 - rho) return false;
    const int par = i >= n0 ? 1 : 0;
    const int J = rho * (i - (par ? n0 : 0)) + (rho == 2 ? (m & 1) : 0);
    const int I = (m + J) / rho;
    const int S0 = TS * I, D0 = TD * J;
    w->par = par;
    w->S0 = S0;
    w->D0 = D0;
    w->L_lo = max(D0, (a.l3_lo - par + 1) >> 1);
    // no element reaches above L = S; those with S > lmax are not stored
    w->L_hi = min(min(S0 + TS - 1, a.lmax), (a.l3_hi - par) >> 1);
    return true;
}

// The table windows of one chunk (L = L0 .. L0 + KC - 1) in LDS, from which its P
// and U are formed: a few entries per thread where P and U have dozens.  They
// are loaded into registers a chunk ahead (fetch), so that the loads run under the
// steps of the chunk before.
//   P(L, S) = g(S - L) h(S + L + par) = g1[S - S0 - k + KC - 1] h1[S - S0 + k],
//   U_X(L, D) = W'_X(2 L + par) g(L - D) g(L + D + par)
//             = w[x][k] g2[k - (D - D0) + TD - 1] g3[D - D0 + k],   k = L - L0.
template <int TS, int TD, int NX, int KC>
struct TileWindows {
    static constexpr int n1 = TS + KC, n2 = TD + KC;
    static constexpr int kAll = 2 * n1 + 2 * n2 + NX * KC;
    static constexpr int kPer = (kAll + kTileThreads - 1) / kTileThreads;
    double v[kPer * kTileThreads];
    int met_wild;                // one of this tile's window values was
    __device__ double g1(int i) const { return v[i]; }
    __device__ double h1(int i) const { return v[n1 + i]; }
    __device__ double g2(int i) const { return v[2 * n1 + i]; }
    __device__ double g3(int i) const { return v[2 * n1 + n2 + i]; }
    __device__ double w(int x, int k) const { return v[2 * n1 + 2 * n2 + x * KC + k]; }
    // This thread's entries: where the next chunk's lie.  Indexes below 0 or from len
    // on give 0 (outside the tables; windows: beyond L_hi).
    struct Reader {
        const double* base[kPer];
        int at[kPer], step[kPer], len[kPer];
        double reg[kPer];
        __device__ __forceinline__ void start(const TileArgs& a, const TileWhere& t, const int (&window)[3]) {
#pragma unroll
            for (int n = 0; n < kPer; ++n) {
                const int e = (int)threadIdx.x + n * kTileThreads;
                base[n] = a.g;
                len[n] = a.g_len;
                step[n] = KC;
                if (e < n1) {
                    at[n] = t.S0 - t.L_lo - (KC - 1) + e;
                    step[n] = -KC;
                } else if (e < 2 * n1) {
                    base[n] = a.h;
                    len[n] = a.h_len;
                    at[n] = t.S0 + t.L_lo + t.par + (e - n1);
                } else if (e < 2 * n1 + n2) {
                    at[n] = t.L_lo - t.D0 - (TD - 1) + (e - 2 * n1);
                } else if (e < 2 * n1 + 2 * n2) {
                    at[n] = t.L_lo + t.D0 + t.par + (e - 2 * n1 - n2);
                } else {
                    const int i = e - (2 * n1 + 2 * n2), x = min(i / KC, NX - 1);
                    base[n] = a.wp + (long long)window[x] * a.wp_stride;
                    len[n] = 2 * t.L_hi + t.par + 1;
                    at[n] = 2 * (t.L_lo + i % KC) + t.par;
                    step[n] = 2 * KC;
                }
            }
        }
        __device__ __forceinline__ void fetch() {
#pragma unroll
            for (int n = 0; n < kPer; ++n) {
                const bool in = (unsigned)at[n] < (unsigned)len[n];
                const double r = base[n][in ? at[n] : 0];
                reg[n] = in ? r : 0.0;
                at[n] += step[n];
            }
        }
    };
    // met: this thread's wave has met a wild value
    __device__ __forceinline__ void put(const Reader& r, bool& met) {
#pragma unroll
        for (int n = 0; n < kPer; ++n) {
            double w = r.reg[n];
            if ((n + 1) * kTileThreads > 2 * n1 + 2 * n2 && __builtin_expect(__any(wild(w)), 0)) {      // windows come last
                w = wild(w) ? 0.0 : w;
                met = true;
            }
            v[threadIdx.x + n * kTileThreads] = w;
        }
    }
    // After the stores: whether the work-group met one (met_wild was cleared by thread 0
    // before the first put, whose barriers order it).
    __device__ __forceinline__ bool any_wild(bool met) {
        if (met) met_wild = 1;
        __syncthreads();
        return met_wild != 0;
    }
};

// The terms of the wild window values, added to the stored sums of element (S, D) by the
// thread that stored them: l3 over the element's own range.
template <int MODE>
__device__ inline void add_wild(const TileArgs& a, int par, int S, int D) {
    constexpr bool EB = MODE == kStripEB;
    const int d = 2 * D + par - (EB ? 1 : 0), l1 = S - D, l2 = l1 + d;
    if (d < 0 || l1 < 0 || l2 > a.lmax) return;
    double* x = a.xi + diag_offset(a.lmax, d) + l1;
    const double sc = MODE == kStripTT ? 1.0 : 0.5 * a.cl[l1] * a.cl[l2];
    const long long sh = n_shift(l1 + l2, d);
    // EB: s = l1 + l2 + 1 here, and odd L end at l3 = s - 2
    const int top = min(S - (EB ? 1 : 0), (a.l3_hi - par) >> 1);
    for (int L = max(D, (a.l3_lo - par + 1) >> 1); L <= top; ++L) {
        const int l3 = 2 * L + par;
        const double* w = a.wp + l3;
        const double tt = w[0], te = w[a.wp_stride], ee = w[2LL * a.wp_stride];
        const bool on_tt = MODE != kStripEB && MODE != kStripEE && wild(tt), on_te = MODE == kStripPol && wild(te),
                   on_ee = MODE != kStripTT && wild(ee);
        if (!on_tt && !on_te && !on_ee) continue;
        const double P = a.g[S - L] * a.h[S + L + par], gg = a.g[L - D] * a.g[L + D + par];
        if (on_tt) x[0] += tt * gg * P;
        const long long s = l1 + l2, c = (long long)l3 * (l3 + 1);
        if (EB) {
            const double f1 = (double)((s + 1) * (s + 2) - c), f2 = (double)(c - (long long)d * (d + 1));
            const double f3 = (double)(c + 2LL * (l1 + 2) * (l2 + 2) - (s + 2) * (s + 3));
            x[3 * a.xi_stride] += (sc * sc) * (ee * gg * f2 * (P * f1 * f3 * f3));
            continue;
        }
        const double N = __builtin_fma((double)(c - (s + 1) * (s + 1) + 1 + sh), (double)(c - (long long)d * d + 2 - sh),
                                       (double)n_rest(s, d, sh));
        if (on_te) x[a.xi_stride] += sc * (te * gg * (P * N));
        if (on_ee) x[2 * a.xi_stride] += (sc * sc) * (ee * gg * (P * N * N));
    }
}

// ---------------------------------------------------------------------------
// TT on the float64 matrix cores.  A wave owns NS x ND MFMA tiles of 16 x 16
// (D along the MFMA's rows, S along its columns, so that a store's 16 lanes are
// 16 consecutive l1 of one diagonal: 128 bytes), a work-group 2 x 2 waves.
// What bounds it: the matrix cores (one v_mfma_f64_16x16x4 per 1024 terms), 73 %
// busy at lmax = 10^4: 6.3 ms for 1.67e11 terms (14.8 ms with the strips, which form
// each P once per term).  A higher wave priority for one of a SIMD's two waves, so
// that one stages while the other multiplies, changed nothing.
template <int NS, int ND>
__global__ void __launch_bounds__(kTileThreads) tile_tt_kernel(TileArgs a) {
    constexpr int KC = kTileChunk;
    constexpr int TS = 32 * NS, TD = 32 * ND;
    constexpr int PS = TS + 16, US = TD + 16;    // 16 mod 32 doubles: the operand reads are free of conflicts
    using Win = TileWindows<TS, TD, 1, KC>;
    __shared__ Win W;
    __shared__ double s_p[KC * PS];
    __shared__ double s_u[KC * US];
    TileWhere w;
    if (!tile_of<TS, TD>(a, a.lmax, &w)) return;
    const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
    const int r = lane % 16, q = lane / 16;
    const int ws = (wave % 2) * 16 * NS, wd = (wave / 2) * 16 * ND;
    d4v acc[ND][NS];
#pragma unroll
    for (int i = 0; i < ND; ++i)
#pragma unroll
        for (int j = 0; j < NS; ++j) acc[i][j] = d4v{0.0, 0.0, 0.0, 0.0};
    constexpr int window[3] = {0, 0, 0};
    if (t == 0) W.met_wild = 0;
    bool met = false;
    typename Win::Reader R;
    R.start(a, w, window);
    R.fetch();
    for (int L0 = w.L_lo; L0 <= w.L_hi; L0 += KC) {
        W.put(R, met);
        __syncthreads();
        R.fetch();
#pragma unroll
        for (int i = 0; i < KC * TS / kTileThreads; ++i) {
            const int e = t + i * kTileThreads, k = e / TS, S = e % TS;
            s_p[k * PS + S] = W.g1(S - k + KC - 1) * W.h1(S + k);
        }
#pragma unroll
        for (int i = 0; i < KC * TD / kTileThreads; ++i) {
            const int e = t + i * kTileThreads, k = e / TD, D = e % TD;
            const double u = W.w(0, k) * (W.g2(k - D + TD - 1) * W.g3(D + k));
            s_u[k * US + D] = L0 + k >= w.D0 + D ? u : 0.0;
        }
        __syncthreads();
        const int kn = min(KC, w.L_hi - L0 + 1);
        for (int k = 0; k < kn; k += 4) {
            double u[ND], p[NS];
#pragma unroll
            for (int i = 0; i < ND; ++i) u[i] = s_u[(k + q) * US + wd + 16 * i + r];
#pragma unroll
            for (int j = 0; j < NS; ++j) p[j] = s_p[(k + q) * PS + ws + 16 * j + r];
#pragma unroll
            for (int i = 0; i < ND; ++i)
#pragma unroll
                for (int j = 0; j < NS; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(u[i], p[j], acc[i][j], 0, 0, 0);
        }
    }
    // accumulator register v of lane (r, q): D = q + 4 v, S = r of the 16 x 16 tile
#pragma unroll
    for (int i = 0; i < ND; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int D = w.D0 + wd + 16 * i + q + 4 * v, d = 2 * D + w.par;
            if (d > a.lmax) continue;
            double* xd = a.xi + diag_offset(a.lmax, d);
#pragma unroll
            for (int j = 0; j < NS; ++j) {
                const int l1 = w.S0 + ws + 16 * j + r - D;
                if (l1 >= 0 && l1 + d <= a.lmax) xd[l1] = acc[i][j][v];
            }
        }
    if (__builtin_expect(W.any_wild(met), 0))
#pragma unroll 1
        for (int e = 0; e < ND * 4 * NS; ++e)
            add_wild<kStripTT>(a, w.par, w.S0 + ws + 16 * (e % NS) + r, w.D0 + wd + 16 * (e / (4 * NS)) + q + 4 * (e / NS % 4));
}

// ---------------------------------------------------------------------------
// The polarised and odd-L sums on the vector unit.  Thread (ts, td) of 16 x 16
// owns RS values of S and RD of D, in pairs 2 ts, 2 ts + 1 (+ 32), so that its
// LDS reads are 16-byte ones free of conflicts.
// What bounds it: the float64 vector unit, 4.2 .. 4.6 clocks per instruction of a
// wave where 4 is the least.  4 x 4 patches execute 105 float64 instructions per
// step and 16 terms for TT + TE + EE (the strips 8 per term and 6 % more terms), and
// the staging about 8 more: lmax = 6000 8.5 ms (10.6 with the strips), EE alone at
// 10^4 25.2 ms (38.6; n_shift saves an addition per term there), EB at 5000 3.1 ms (5.0).
template <int MODE, int RS, int RD>
__global__ void __launch_bounds__(kTileThreads, RS * RD >= 16 ? 2 : 3) tile_pol_kernel(TileArgs a) {
    constexpr bool EB = MODE == kStripEB;
    constexpr bool TTS = MODE == kStripPol || MODE == kStripPolEE;
    constexpr bool TE = MODE == kStripPol;
    constexpr int NX = (TTS ? 1 : 0) + (TE ? 1 : 0) + 1;     // window factors staged: TT, TE, then EE's (or EB's)
    constexpr int XE = NX - 1;
    // steps staged at a time: LDS for two work-groups or more
    constexpr int KC = RS * RD == 4 && NX == 2 ? 2 * kTileChunk : NX * RS * RD > 32 ? kTileChunk / 2 : kTileChunk;
    constexpr int TS = 16 * RS, TD = 16 * RD;
    using Win = TileWindows<TS, TD, NX, KC>;
    __shared__ Win W;
    __shared__ __align__(16) double s_p[KC][TS];
    __shared__ __align__(16) double s_u[NX][KC][TD];
    TileWhere w;
    if (!tile_of<TS, TD>(a, a.lmax + (EB ? 1 : 0), &w)) return;
    const int t = threadIdx.x, ts = t % 16, td = t / 16;
    const int par = w.par;

    double tt[RS][RD], te[RS][RD], ee[RS][RD], G[RS][RD], f[RS], e[RD];
    const long long shift = EB ? 0 : n_shift(2LL * w.S0 + TS + par, 2LL * w.D0 + TD + par);   // from the tile's middle
    const long long l3s = 2LL * w.L_lo + par;
    double cc = (double)(l3s * (l3s + 1)), dc = (double)(4 * l3s + 6);   // c(l3) and its step to l3 + 2
#pragma unroll
    for (int i = 0; i < RS; ++i) {
        const long long s = 2LL * (w.S0 + 2 * ts + (i & 1) + 32 * (i >> 1)) + par;
        f[i] = cc - (double)((s + 1) * (s + 1) - 1 - shift);
#pragma unroll
        for (int j = 0; j < RD; ++j) {
            const long long d = 2LL * (w.D0 + 2 * td + (j & 1) + 32 * (j >> 1)) + par;
            if (i == 0) e[j] = cc - (double)(d * d - 2 + shift);
            if (EB) {
                // mu = 2 (l1+2)(l2+2) - tau (tau+1), tau = s + 1, with l1 + l2 = s - 1, l2 - l1 = d - 1
                const long long l1 = (s - d) / 2, l2 = l1 + d - 1;
                G[i][j] = (double)(2 * (l1 + 2) * (l2 + 2) - (s + 1) * (s + 2));
            } else {
                G[i][j] = (double)n_rest(s, d, shift);
            }
            tt[i][j] = te[i][j] = ee[i][j] = 0.0;
        }
    }

    // the windows in the order they are staged
    constexpr int window[3] = {TTS ? 0 : 2, TE ? 1 : 2, 2};
    if (t == 0) W.met_wild = 0;
    bool met = false;
    typename Win::Reader R;
    R.start(a, w, window);
    R.fetch();
    for (int L0 = w.L_lo; L0 <= w.L_hi; L0 += KC) {
        W.put(R, met);
        __syncthreads();
        R.fetch();
#pragma unroll
        for (int i = 0; i < KC * TS / kTileThreads; ++i) {
            const int x = t + i * kTileThreads, k = x / TS, S = x % TS;
            double p = W.g1(S - k + KC - 1) * W.h1(S + k);
            if (EB) {
                const long long s = 2LL * (w.S0 + S) + par, l3 = 2LL * (L0 + k) + par;
                p *= (double)(s * (s + 1) - l3 * (l3 + 1));
            }
            s_p[k][S] = p;
        }
#pragma unroll
        for (int i = 0; i < KC * TD / kTileThreads; ++i) {
            const int x = t + i * kTileThreads, k = x / TD, D = x % TD;
            const bool on = L0 + k >= w.D0 + D;
            const double gg = W.g2(k - D + TD - 1) * W.g3(D + k);
#pragma unroll
            for (int y = 0; y < NX; ++y) {
                double u = W.w(y, k) * gg;
                if (EB) {
                    const long long d = 2LL * (w.D0 + D) + par, l3 = 2LL * (L0 + k) + par;
                    u *= (double)(l3 * (l3 + 1) - d * (d - 1));
                }
                s_u[y][k][D] = on ? u : 0.0;
            }
        }
        __syncthreads();
        const int kn = min(KC, w.L_hi - L0 + 1);
#pragma unroll 2
        for (int k = 0; k < kn; ++k) {
            double p[RS], u[NX][RD];
#pragma unroll
            for (int i = 0; i < RS; i += 2) {
                const double2 v = *reinterpret_cast<const double2*>(&s_p[k][2 * ts + 16 * i]);
                p[i] = v.x;
                p[i + 1] = v.y;
            }
#pragma unroll
            for (int x = 0; x < NX; ++x)
#pragma unroll
                for (int j = 0; j < RD; j += 2) {
                    const double2 v = *reinterpret_cast<const double2*>(&s_u[x][k][2 * td + 16 * j]);
                    u[x][j] = v.x;
                    u[x][j + 1] = v.y;
                }
#pragma unroll
            for (int i = 0; i < RS; ++i)
#pragma unroll
                for (int j = 0; j < RD; ++j) {
                    if (EB) {
                        // P (sig(sig+1) - c) (c + mu)^2, the first product staged
                        const double f3 = cc + G[i][j];
                        ee[i][j] = __builtin_fma(u[XE][j], (p[i] * f3) * f3, ee[i][j]);
                        continue;
                    }
                    const double N = __builtin_fma(f[i], e[j], G[i][j]);
                    const double y = p[i] * N;
                    if (TTS) tt[i][j] = __builtin_fma(u[0][j], p[i], tt[i][j]);
                    if (TE) te[i][j] = __builtin_fma(u[1][j], y, te[i][j]);
                    ee[i][j] = __builtin_fma(u[XE][j], y * N, ee[i][j]);
                }
            // c(l3 + 2) = c(l3) + 4 l3 + 6: exact integers
            if (EB) {
                cc += dc;
            } else {
#pragma unroll
                for (int i = 0; i < RS; ++i) f[i] += dc;
#pragma unroll
                for (int j = 0; j < RD; ++j) e[j] += dc;
            }
            dc += 8.0;
        }
    }

#pragma unroll
    for (int j = 0; j < RD; ++j) {
        const int D = w.D0 + 2 * td + (j & 1) + 32 * (j >> 1);
        const int d = 2 * D + par - (EB ? 1 : 0);
        if (d < 0 || d > a.lmax) continue;
        double* xd = a.xi + diag_offset(a.lmax, d);
#pragma unroll
        for (int i = 0; i < RS; ++i) {
            const int l1 = w.S0 + 2 * ts + (i & 1) + 32 * (i >> 1) - D;
            if (l1 < 0 || l1 + d > a.lmax) continue;
            const double sc = 0.5 * a.cl[l1] * a.cl[l1 + d];
            if (EB) {
                xd[3 * a.xi_stride + l1] = (sc * sc) * ee[i][j];
                continue;
            }
            if (TTS) xd[l1] = tt[i][j];
            if (TE) xd[a.xi_stride + l1] = sc * te[i][j];
            xd[2 * a.xi_stride + l1] = (sc * sc) * ee[i][j];
        }
    }
    if (__builtin_expect(W.any_wild(met), 0))
#pragma unroll 1
        for (int x = 0; x < RS * RD; ++x) {
            const int i = x % RS, j = x / RS;
            add_wild<MODE>(a, par, w.S0 + 2 * ts + (i & 1) + 32 * (i >> 1), w.D0 + 2 * td + (j & 1) + 32 * (j >> 1));
        }
}

// Grid of the tiles TS x TD (level_tiles), and the highest level.
template <int TS, int TD>
dim3 tile_grid(TileArgs& a, int reach) {
    constexpr int rho = TS / TD;
    a.m_top = rho * (reach / TS);
    unsigned n = 0;
    for (int m = a.m_top; m >= 1 - rho; --m) n += level_tiles<TS, TD>(reach, m, 0) + level_tiles<TS, TD>(reach, m, 1);
    return dim3(n);
}

template <int MODE, int RS, int RD>
hipError_t launch_pol(TileArgs a, hipStream_t s) {
    const dim3 grid = tile_grid<16 * RS, 16 * RD>(a, a.lmax + (MODE == kStripEB ? 1 : 0));
    hipLaunchKernelGGL((tile_pol_kernel<MODE, RS, RD>), grid, dim3(kTileThreads), 0, s, a);
    return hipGetLastError();
}

template <int RS, int RD>
hipError_t launch_pol_mode(const TileArgs& a, int mode, hipStream_t s) {
    switch (mode) {
    case kStripEB: return launch_pol<kStripEB, RS, RD>(a, s);
    case kStripPol: return launch_pol<kStripPol, RS, RD>(a, s);
    case kStripPolEE: return launch_pol<kStripPolEE, RS, RD>(a, s);
    case kStripEE: return launch_pol<kStripEE, RS, RD>(a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_tile_fp64(const couple_ctx* ctx, int lmax, int mode, int l3_lo, int l3_hi, hipStream_t s) {
    TileArgs a;
    a.g = ctx->g_pad + kTablePad;
    a.h = ctx->h_pad + kTablePad;
    a.wp = ctx->wp;
    a.cl = ctx->cl;
    a.xi = ctx->xi;
    a.xi_stride = tri_size(lmax);
    a.wp_stride = 2 * ctx->lmax_max + 1;
    a.g_len = ctx->lmax_max + 1;
    a.h_len = 2 * ctx->lmax_max + 1;
    a.lmax = lmax;
    a.l3_lo = l3_lo;
    a.l3_hi = l3_hi;
    a.m_top = 0;
    if (mode == kStripTT) {
        if (lmax >= kTileTTBig) {
            const dim3 grid = tile_grid<128, 64>(a, lmax);
            hipLaunchKernelGGL((tile_tt_kernel<4, 2>), grid, dim3(kTileThreads), 0, s, a);
        } else if (lmax >= kTileTTMid) {
            const dim3 grid = tile_grid<64, 64>(a, lmax);
            hipLaunchKernelGGL((tile_tt_kernel<2, 2>), grid, dim3(kTileThreads), 0, s, a);
        } else {
            const dim3 grid = tile_grid<32, 32>(a, lmax);
            hipLaunchKernelGGL((tile_tt_kernel<1, 1>), grid, dim3(kTileThreads), 0, s, a);
        }
        return hipGetLastError();
    }
    if (lmax >= kTilePolBig) return launch_pol_mode<4, 4>(a, mode, s);
    if (lmax >= kTilePolMid) return launch_pol_mode<4, 2>(a, mode, s);
    return launch_pol_mode<2, 2>(a, mode, s);
}

}  // namespace couple
