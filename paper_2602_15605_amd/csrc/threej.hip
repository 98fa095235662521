// Rows of Wigner 3j symbols (l1 l2 l3; -m m 0), m = 0, 1, 2, over every
// l3 = |l1 - l2| .. l1 + l2, from the g(p) tables in closed form.
//
// (0 0 0): eq. 000_sq_main, X^2 = g(P-l1) g(P-l2) g(P-l3) / ((2P+1) g(P)),
//   P = L/2, sign (-1)^P, zero for odd L (L = l1 + l2 + l3).
// (-1 1 0) = (l3 l1 l2; 0 -1 1) (cyclic), the J_(-1,1) family of App. B:
//   odd L  (eq. joneodd with (j1, j2, j3) = (l3, l1, l2)):
//     -1/2 [(L+2)(L-2 l3+1)(L-2 l1+1)(L-2 l2) / (a b)]^{1/2} (l1, l2+1, l3; 0 0 0);
//   even L: eq. joneeven's two (0 0 0) terms of opposite sign collapse, by the
//     (0 0 0) ratio of eq. g_rec, to the single product
//     -(l1 l2 l3; 0 0 0) (a + b - c) / (2 sqrt(a b)),
//   with a = l1(l1+1), b = l2(l2+1), c = l3(l3+1); zero for l1 or l2 < 1.
// (-2 2 0): App. B.3 (eq. 022_linear_closedform) for even L,
//     X N' c_l1 c_l2 / 2,  N' = c (c - 2(a+b-1)) + a(a-2) + b(b-2);
//   odd L (eq. 022_rearranged with eqs. joneodd, joneevensimp at j3 + 1):
//     -Y' (c + mu) (c_l1 c_l2 / 2) [(sig(sig+1) - c)(c - d(d+1))]^{1/2},
//     Y' = (l1, l2+1, l3; 0 0 0), sig = l1 + l2 + 1, tau = sig + 1,
//     mu = 2 (l1+2)(l2+2) - tau(tau+1), d = l2 - l1;
//   zero for l1 or l2 < 2.
// Every integer factor is exact (or, for N', one rounding of an exact value); the
// other roundings are the table values, the products and one square root, so there is
// no cancellation.
//
// The family kernels below extend this to (l1 l2 l3; m1 m2 m3) with small
// magnetic numbers, (1 1 -2) and (2 2 -4) among them.
//
// One work-group per (l1, l2) pair and piece of its row (256 threads, short rows 64), threads over
// l3.  The pairs are read from device memory, so the kernel itself checks them: a pair
// outside [0, lmax_max] gives a row of NaN and reads no table.
#include <algorithm>
#include <type_traits>

#include "couple_internal.hpp"

namespace couple {
namespace {

// Threads per work-group: 64 for rows of at most kThreejShort entries.  A row's setup runs
// in every wave, and with four waves for 21 entries it was most of the time (20000 rows at
// lmax 10, 256 / 64 threads: m = 0 15 / 9 us, m = 1 30 / 12, (2 2 -4) 48 / 16; at lmax 200
// 17.5 / 13.6, 38 / 19, 63 / 26); at 801 entries 2000 rows of (2 -1 -1) take 9.9 / 13.3 us.
constexpr int kThreejShort = 512;
// Symbols that a thread computes before it stores any (m = 0 and the general family: one;
// two took 13.9 against 13.5 us for 5000 rows of m = 0 at lmax 1000 and 18.5 against 17.6 us
// for 2000 of (2 -1 -1)).
constexpr int kThreejBatch = 2;
// Entries of a row per block.  One block per row left the longest rows running alone at
// the end (on average half the waves that fit): with the kernels below 2000 rows at lmax
// 6000 took 64 us (m = 1) and 75 us ((2 2 -4)), with these pieces 37 and 54 us (1024
// entries: 52 and 79 us, the row's setup weighs more; 8192: 58 and 65 us).  Plain stores:
// past the caches (nontemporal) the same rows took 56 and 64 us.
constexpr int kThreejPiece = 2048;
// Results beyond the memory-side cache take longer pieces: first pieces of all rows are
// written before second ones, and memory likes long runs (entries 2048 / 4096 / 8192, 20000
// rows at lmax 2000: m = 1 153 / 137 / 137 us, (2 -1 -1) 219 / 185 / 185; 10000 at lmax 4000:
// 147 / 139 / 145 and 212 / 210 / 191).
constexpr double kThreejPastBytes = 256e6;
constexpr int kThreejPastPiece = 4096, kFamilyPastPiece = 8192;

inline bool past_cache(int n_pairs, long long stride) { return 8.0 * n_pairs * (double)stride > kThreejPastBytes; }
inline dim3 piece_grid(int n_pairs, long long stride, int piece) {
    return dim3((unsigned)n_pairs, (unsigned)std::min((stride + piece - 1) / piece, 1024LL));
}

struct ThreejArgs {
    const double* g;             // g(p), p = 0 .. lmax_max
    const double* h;             // 1/((2p+1) g(p)), p = 0 .. 2 lmax_max
    const double* cl;            // c_l, l = 0 .. lmax_max
    const int* l1;
    const int* l2;
    double* out;                 // [n_pairs][stride]
    long long stride;
    int lmax_max;
    int m;
};

// Zeros in entries i .. end - 1 of a row, 16 bytes per store.
template <int T>
__device__ inline void put_zeros(double* row, long long i, long long end) {
    typedef double d2v __attribute__((ext_vector_type(2)));
    if (i < end && (reinterpret_cast<uintptr_t>(row + i) & 15)) {
        if (threadIdx.x == 0) row[i] = 0.0;
        ++i;
    }
    const long long pairs = end > i ? (end - i) / 2 : 0;
    d2v* out = reinterpret_cast<d2v*>(row + i);
    for (long long q = threadIdx.x; q < pairs; q += T)
        out[q] = d2v{0.0, 0.0};
    if (threadIdx.x == 0 && i + 2 * pairs < end) row[end - 1] = 0.0;
}

// Runs `entries(lo, hi)` for the pieces of this block's row that hold some of its n
// symbols, and writes NaN (a degree out of range) or zeros elsewhere.  Pieces start at
// even entries.
template <int T, int PIECE, class Entries>
__device__ inline void each_piece(double* row, long long n, long long stride, bool nan, Entries entries) {
    for (long long lo = (long long)blockIdx.y * PIECE; lo < stride; lo += (long long)gridDim.y * PIECE) {
        const long long end = min(lo + PIECE, stride), hi = min(n, end);
        if (nan) {
            for (long long i = lo + threadIdx.x; i < end; i += T) row[i] = __builtin_nan("");
            continue;
        }
        put_zeros<T>(row, max(lo, hi), end);
        if (lo < hi) entries((int)lo, (int)hi);
    }
}

// The factor shared by a whole row of degrees >= m: m = 1: -1 / (2 sqrt(a b)); m = 2: c_l1 c_l2 / 2.
__device__ inline double row_factor(const ThreejArgs& a, long long l1, long long l2) {
    if (a.m == 1) return -0.5 / sqrt((double)(l1 * (l1 + 1)) * (double)(l2 * (l2 + 1)));
    return 0.5 * a.cl[l1] * a.cl[l2];
}

// For m = 1, 2 each thread computes kThreejBatch symbols of its row before it stores any,
// so their table reads are in flight together.  For m = 0 the symbols of odd
// L vanish; a row starts at L = 2 max(l1, l2), so its even entries are the
// even-L ones, and each thread takes a pair of entries: it evaluates the even
// one and writes a zero beside it.
//
// m = 1, 2: a thread's entries lie an even number apart, so all of them have one
// parity of L and it forms that parity's factor only.  Both parities need one
// (0 0 0) value, (l1 l2 l3) for even L and (l1, l2+1, l3) for odd L, whose total is
// then even; with p1, p2, p3 and P its halved combinations the factors are
//   m = 1 even: (a + b - c);   odd: the root of (L+2)(L-2 l3+1)(L-2 l1+1)(L-2 l2);
//   m = 2 even: N' (n_shift and n_rest of the row: one fused multiply-add);
//         odd: -(c + mu) times the root of (sig(sig+1) - c)(c - d(d+1)),
// the roots taken together with the (0 0 0) value's.  Every integer below is
// exact in float64.  What bounds it: about 120 instructions per symbol, most of
// them the root; with 64-bit integers, both parities' factors and two roots per
// symbol 2000 rows at lmax 6000 took 57 us, now 37 us (115 MB of results and 77 MB of
// zeros: 5.2 TB/s); 200 rows at lmax 16000 67 us, now 16 us.
template <int T, int PIECE>
__global__ void __launch_bounds__(T) threej_rows_kernel(ThreejArgs a) {
    const long long p = blockIdx.x;
    const int l1 = a.l1[p], l2 = a.l2[p];
    double* row = a.out + p * a.stride;
    const bool nan = l1 < 0 || l2 < 0 || l1 > a.lmax_max || l2 > a.lmax_max;
    const int jmin = l1 > l2 ? l1 - l2 : l2 - l1;
    if (nan || min(l1, l2) < a.m) {           // a selection rule |m| <= l fails: zeros
        each_piece<T, PIECE>(row, 0, a.stride, nan, [](int, int) {});
        return;
    }
    const int n = l1 + l2 - jmin + 1;
    if (a.m == 0) {
        each_piece<T, PIECE>(row, n, a.stride, false, [&](int lo, int hi) {
            for (int i = lo + 2 * threadIdx.x; i < hi; i += 2 * T) {
                const int P = (l1 + l2 + jmin + i) / 2;
                const double r = sqrt(a.g[P - l1] * a.g[P - l2] * a.g[P - jmin - i] * a.h[P]);
                row[i] = (P & 1) ? -r : r;
                if (i + 1 < hi) row[i + 1] = 0.0;
            }
        });
        return;
    }
    const double rowf = row_factor(a, l1, l2);
    const int odd = (l1 + l2 + jmin + (int)threadIdx.x) & 1;
    const double A = (double)l1 * (l1 + 1), B = (double)l2 * (l2 + 1);
    // m = 2, even L: N' = (c - es)(c - ed) + rest; odd L: sig(sig+1), mu, d(d+1)
    const long long s = (long long)l1 + l2, d = jmin, sh = n_shift(s, d);
    const double es = (double)((s + 1) * (s + 1) - 1 - sh), ed = (double)(d * d - 2 + sh), rest = (double)n_rest(s, d, sh);
    const long long dd = (long long)l2 - l1;
    const double s1 = (double)((s + 1) * (s + 2)), d1 = (double)(dd * (dd + 1));
    const double mu = (double)(2LL * (l1 + 2) * (l2 + 2) - (s + 2) * (s + 3));
    each_piece<T, PIECE>(row, n, a.stride, false, [&](int lo, int hi) {
        for (int i0 = lo + threadIdx.x; i0 < hi; i0 += T * kThreejBatch) {
            double v[kThreejBatch];
#pragma unroll
            for (int q = 0; q < kThreejBatch; ++q) {
                // entries past the piece repeat its last one of this parity, unstored
                const int i = min(i0 + q * T, hi - 1 - ((hi - 1 - i0) & 1));
                const int l3 = jmin + i, L = l1 + l2 + l3;
                // (l1, l2 + odd, l3; 0 0 0)^2: odd L has |l1 - l2 - 1| <= l3 < l1 + l2
                const int P = (L + odd) / 2;
                double x = a.g[P - l1] * a.g[P - l2 - odd] * a.g[P - l3] * a.h[P];
                const double c = (double)l3 * (l3 + 1);
                double f;
                if (a.m == 1) {
                    f = odd ? 1.0 : A + B - c;
                    if (odd) x *= ((double)(L + 2) * (double)(L - 2 * l3 + 1)) * ((double)(L - 2 * l1 + 1) * (double)(L - 2 * l2));
                } else {
                    f = odd ? -(c + mu) : __builtin_fma(c - es, c - ed, rest);
                    if (odd) x *= (s1 - c) * (c - d1);
                }
                const double r = sqrt(x);
                v[q] = ((P & 1) ? -r : r) * f * rowf;
            }
#pragma unroll
            for (int q = 0; q < kThreejBatch; ++q) {
                const int i = i0 + q * T;
                if (i < hi) row[i] = v[q];
            }
        }
    });
}

// Rows of m = 0 of these many entries that go past the memory-side cache: one block per
// row, symbols and zeros in one pass, and no more than six work-groups per compute unit.
// How the rows fall into memory decides here, not the instructions (eight work-groups per
// compute unit take up to a fifth longer): threej_rows_kernel / this one take 75 / 67 us for
// 30000 rows at lmax 800, 70 / 64 for 25000 at 900, 61 / 58 for 20000 at 1000, 77 / 72 at 1200,
// but 75 / 85 for 40000 at 600 and 136 / 140 for 20000 at 2000.
constexpr int kZeroRowsFrom = 1400, kZeroRowsTo = 2600;
constexpr int kZeroRowsLds = 26500;              // six work-groups per compute unit
__global__ void __launch_bounds__(256) threej_zero_rows_kernel(ThreejArgs a) {
    constexpr int kBatch = 4;
    const long long p = blockIdx.x, l1 = a.l1[p], l2 = a.l2[p];
    double* row = a.out + p * a.stride;
    if (l1 < 0 || l2 < 0 || l1 > a.lmax_max || l2 > a.lmax_max) {
        for (long long i = threadIdx.x; i < a.stride; i += 256) row[i] = __builtin_nan("");
        return;
    }
    const long long jmin = l1 > l2 ? l1 - l2 : l2 - l1, n = l1 + l2 - jmin + 1;
    auto x000 = [&](long long l3) {
        const long long L = l1 + l2 + l3;
        if ((L & 1) || l3 < jmin || l3 > l1 + l2) return 0.0;
        const long long P = L / 2;
        const double r = sqrt(a.g[P - l1] * a.g[P - l2] * a.g[P - l3] * a.h[P]);
        return (P & 1) ? -r : r;
    };
    for (long long q0 = threadIdx.x; 2 * q0 < a.stride; q0 += 256 * kBatch) {
        double v[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
            const long long i = 2 * (q0 + 256 * q);
            v[q] = i < n ? x000(jmin + i) : 0.0;
        }
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
            const long long i = 2 * (q0 + 256 * q);
            if (i < a.stride) row[i] = v[q];
            if (i + 1 < a.stride) row[i + 1] = 0.0;
        }
    }
}

// ---------------------------------------------------------------------------
// Rows of (l1 l2 l3; m1 m2 m3), m3 = -m1 - m2, for small magnetic numbers: the
// (1 1 -2) and (2 2 -4) families of the Conclusion and their relatives.
//
// Every triple with zero sum has two entries of one sign (or zero) and one of
// the other.  A cyclic permutation of the columns (no sign) puts the odd one
// last and, when the first two are <= 0, the m-flip (a factor (-1)^L) makes
// them >= 0.  The host does this once per call (same for every element); what
// is left is F_ab(x, y, z) = (x y z; a b -a-b) with 0 <= a, b <= 2, where
// (x, y, z) is the rotated (l1, l2, l3).
//
// On the lines a = 0 and b = 0 F_ab is an App. B symbol: (0 -1 1) and
// (0 -2 2) up to a permutation and an m-flip.  The lowering relation of E57
// Sec. 3.7,
//   sqrt((x+a)(x-a+1)) F_{a-1,b} + sqrt((y+b)(y-b+1)) F_{a,b-1}
//     + sqrt((z+a+b)(z-a-b+1)) F_ab = 0,
// fills the quadrant from them.  Taken numerically that relation cancels where
// z << x ~ y (its two large terms nearly cancel; about 2e-6 relative for
// (2 2 -4) near l = 6000), so the chain is collapsed symbolically to one
// closed form per family and parity:
//   even L:  F_ab = X N_ab(A, B, C) / (2 D_ab),   X = (x y z; 0 0 0),
//   odd L:   F_ab = W N_ab(A, B, C) / (2 D_ab),
//            W = (-1)^P [8 p1 p2 p3 (L+2) g(p1) g(p2) g(p3) h(P)]^{1/2},
//            P = (L+1)/2, p_i = P - l_i; W equals
//            (x, y, z+1; 0 0 0) [(L+2)(L+1-2x)(L+1-2y)(L-2z)]^{1/2}, the odd-L
//            form of App. B, written symmetrically;
//   D_ab^2 = prod_{k<a} (A - k(k+1)) prod_{k<b} (B - k(k+1)) prod_{k<a+b} (C - k(k+1)),
//   A = x(x+1), B = y(y+1), C = z(z+1),
// with the integer polynomials N_ab of family_numerator.  N_ab is evaluated
// exactly in 128-bit integers (below 2^118 for l <= 16384; A, B, C and s, t
// are even, so the halvings are exact), so the roundings are its conversion,
// the table product, D_ab and two square roots: no cancellation anywhere.

struct FamilyArgs {
    const double* g;
    const double* h;
    const int* l1;
    const int* l2;
    double* out;                 // [n_pairs][stride]
    long long stride;
    int lmax_max;
    int rot;                     // (x, y, z) = (l1, l2, l3) rotated left by rot
    int flip;                    // 1: times (-1)^L
};

// Sign and magnitude, then the two 64-bit words of |v|: the high word
// rounds only above 2^53 (|v| >= 2^117), the low word's rounding (at most
// 2^11) is far below the last place of a result >= 2^64 and exact below it,
// and the sum rounds once.  (Converting a negative v by words would leave
// its low word near 2^64, where that rounding is not negligible.)
__device__ inline double i128_to_double(__int128 v) {
    const bool neg = v < 0;
    const unsigned __int128 m = neg ? (unsigned __int128)(-v) : (unsigned __int128)v;
    const double r = (double)(unsigned long long)(m >> 64) * 18446744073709551616.0 + (double)(unsigned long long)m;
    return neg ? -r : r;
}

// N_ab(A, B, C) for L even (odd = 0) and odd (odd = 1); s = A - B, t = A + B.
template <int AB>
__device__ inline __int128 family_numerator(int odd, __int128 A, __int128 B, __int128 C) {
    const __int128 s = A - B, t = A + B;
    switch (AB) {
    case 0:  // (0 0 0)
        return odd ? 0 : 2;
    case 1:  // (0 1 -1)
        return odd ? (__int128)1 : s - C;
    case 2:  // (0 2 -2)
        return odd ? s - C + 2 : C * C - C * (t + s + 2) + s * s + 2 * s;
    case 3:  // (1 0 -1)
        return odd ? (__int128)-1 : -(s + C);
    case 4:  // (1 1 -2)
        return odd ? -s : C * t - s * s;
    case 5:  // (1 2 -3)
        return odd ? C * A - s * s - 3 * s - t
                   : -C * C * A + C * ((s * s + 3 * s * t) / 2 + s + 3 * t) - s * s * s - 3 * s * s - s * t;
    case 6:  // (2 0 -2)
        return odd ? s + C - 2 : C * C - C * (t - s + 2) + s * s - 2 * s;
    case 7:  // (2 1 -3)
        return odd ? -C * B + s * s - 3 * s + t
                   : -C * C * B + C * ((s * s - 3 * s * t) / 2 - s + 3 * t) + s * s * s - 3 * s * s + s * t;
    default:  // (2 2 -4)
        return odd ? s * (C * (2 - t) + s * s + 4 * t - 12)
                   : C * C * ((s * s + t * t) / 2 - 2 * t) + C * (-2 * s * s * t + s * s - 3 * t * t + 12 * t) +
                         s * s * (s * s + 4 * t - 12);
    }
}

template <int AB>
__device__ inline double family_symbol(const FamilyArgs& f, long long l1, long long l2, long long l3) {
    constexpr int a = AB / 3, b = AB % 3;
    const long long x = f.rot == 0 ? l1 : (f.rot == 1 ? l2 : l3);
    const long long y = f.rot == 0 ? l2 : (f.rot == 1 ? l3 : l1);
    const long long z = f.rot == 0 ? l3 : (f.rot == 1 ? l1 : l2);
    if (x < a || y < b || z < a + b) return 0.0;
    const long long L = l1 + l2 + l3;
    const int odd = (int)(L & 1);
    const long long P = (L + 1) / 2;
    const long long p1 = P - l1, p2 = P - l2, p3 = P - l3;
    const long long A = x * (x + 1), B = y * (y + 1), C = z * (z + 1);
    double base = f.g[p1] * f.g[p2] * f.g[p3] * f.h[P];
    if (odd) base *= (double)(8 * p1 * p2 * p3) * (double)(L + 2);
    double d2 = 1.0;
#pragma unroll
    for (int k = 0; k < a; ++k) d2 *= (double)(A - k * (k + 1));
#pragma unroll
    for (int k = 0; k < b; ++k) d2 *= (double)(B - k * (k + 1));
#pragma unroll
    for (int k = 0; k < a + b; ++k) d2 *= (double)(C - k * (k + 1));
    const double n = i128_to_double(family_numerator<AB>(odd, A, B, C));
    double v = sqrt(base) * n / (2.0 * sqrt(d2));
    if (P & 1) v = -v;
    if (f.flip && odd) v = -v;
    return v;
}

// The general kernel: rows whose l3 is not the column z.
template <int AB, int T, int PIECE>
__global__ void __launch_bounds__(T) threej_family_kernel(FamilyArgs f) {
    const long long p = blockIdx.x;
    const int l1 = f.l1[p], l2 = f.l2[p];
    double* row = f.out + p * f.stride;
    const bool nan = l1 < 0 || l2 < 0 || l1 > f.lmax_max || l2 > f.lmax_max;
    const long long jmin = l1 > l2 ? l1 - l2 : l2 - l1;
    each_piece<T, PIECE>(row, nan ? 0 : (long long)l1 + l2 - jmin + 1, f.stride, nan, [&](int lo, int hi) {
        for (int i = lo + threadIdx.x; i < hi; i += T) {
            const double v = i < hi ? family_symbol<AB>(f, l1, l2, jmin + i) : 0.0;
            if (i < hi) row[i] = v;
        }
    });
}

// v c modulo 2^128, from four 32-bit products.
__device__ inline unsigned __int128 mul_u32(unsigned __int128 v, unsigned c) {
    const unsigned long long a0 = (unsigned long long)(unsigned)v * c;
    const unsigned long long a1 = (unsigned long long)(unsigned)(v >> 32) * c + (a0 >> 32);
    const unsigned long long a2 = (unsigned long long)(unsigned)(v >> 64) * c + (a1 >> 32);
    const unsigned a3 = (unsigned)(v >> 96) * c + (unsigned)(a2 >> 32);
    return (unsigned __int128)(a1 << 32 | (unsigned)a0) | (unsigned __int128)((unsigned long long)a3 << 32 | (unsigned)a2) << 64;
}

// Rows with l3 = z (rot = 0: (1 1 -2), (2 2 -4) and their m-flips among them).
// Along such a row A and B are fixed and N_ab is a quadratic in C, so its three
// coefficients are formed once per row and a symbol takes two 128 x 32-bit
// products, exact as before (|N| < 2^118, every partial sum below 2^127 and
// wrapping harmless in any case).  A thread's entries lie an even number apart, so
// all of them have one parity of L and it evaluates that parity's polynomial only;
// the two roots become one, of the table product over D^2.
// What bounds it: about 150 instructions per symbol.  2000 rows of (2 2 -4) at lmax 6000
// take 54 us, with the full 128-bit polynomials of both parities and two roots per
// symbol 131 us; (1 1 -2) 43 us, before 78 us.
template <int AB, int T, int PIECE>
__global__ void __launch_bounds__(T) threej_family_row_kernel(FamilyArgs f) {
    constexpr int a = AB / 3, b = AB % 3;
    const long long p = blockIdx.x;
    const int l1 = f.l1[p], l2 = f.l2[p];
    double* row = f.out + p * f.stride;
    const bool nan = l1 < 0 || l2 < 0 || l1 > f.lmax_max || l2 > f.lmax_max;
    if (nan || l1 < a || l2 < b) {
        each_piece<T, PIECE>(row, 0, f.stride, nan, [](int, int) {});
        return;
    }
    const int jmin = l1 > l2 ? l1 - l2 : l2 - l1, n = l1 + l2 - jmin + 1;
    const long long A = (long long)l1 * (l1 + 1), B = (long long)l2 * (l2 + 1);
    const int odd = (l1 + l2 + jmin + (int)threadIdx.x) & 1;
    // N(C) = (c2 C + c1) C + c0 from N(0), N(1) and N(-1) (the sums are even)
    __int128 c0, c1, c2;
    {
        const __int128 e0 = family_numerator<AB>(0, A, B, 0), ep = family_numerator<AB>(0, A, B, 1),
                       em = family_numerator<AB>(0, A, B, -1);
        const __int128 o0 = family_numerator<AB>(1, A, B, 0), op = family_numerator<AB>(1, A, B, 1),
                       om = family_numerator<AB>(1, A, B, -1);
        c0 = odd ? o0 : e0;
        c1 = odd ? (op - om) / 2 : (ep - em) / 2;
        c2 = (odd ? (op + om) / 2 : (ep + em) / 2) - c0;
    }
    double dab = 1.0;
#pragma unroll
    for (int k = 0; k < a; ++k) dab *= (double)(A - k * (k + 1));
#pragma unroll
    for (int k = 0; k < b; ++k) dab *= (double)(B - k * (k + 1));
    each_piece<T, PIECE>(row, n, f.stride, false, [&](int lo, int hi) {
        for (int i0 = lo + threadIdx.x; i0 < hi; i0 += T * kThreejBatch) {
            double v[kThreejBatch];
#pragma unroll
            for (int q = 0; q < kThreejBatch; ++q) {
                const int i = min(i0 + q * T, hi - 1 - ((hi - 1 - i0) & 1));
                const int l3 = jmin + i, L = l1 + l2 + l3, P = (L + 1) / 2;
                const int p1 = P - l1, p2 = P - l2, p3 = P - l3;
                const int C = l3 * (l3 + 1);
                double base = f.g[p1] * f.g[p2] * f.g[p3] * f.h[P];
                if (odd) base *= (8.0 * (double)p1 * (double)p2 * (double)p3) * (double)(L + 2);
                double d2 = dab;
#pragma unroll
                for (int k = 0; k < a + b; ++k) d2 *= (double)(C - k * (k + 1));
                const unsigned __int128 N =
                    mul_u32(mul_u32((unsigned __int128)c2, (unsigned)C) + (unsigned __int128)c1, (unsigned)C) + (unsigned __int128)c0;
                const double r = 0.5 * sqrt(base / d2) * i128_to_double((__int128)N);
                const bool minus = ((P & 1) != 0) != (f.flip && odd);
                v[q] = l3 < a + b ? 0.0 : (minus ? -r : r);
            }
#pragma unroll
            for (int q = 0; q < kThreejBatch; ++q) {
                const int i = i0 + q * T;
                if (i < hi) row[i] = v[q];
            }
        }
    });
}

}  // namespace

hipError_t launch_threej_family(const couple_ctx* ctx, int rot, int flip, int a, int b, int n_pairs, const int* l1,
                                const int* l2, double* out, long long stride, hipStream_t s) {
    FamilyArgs f;
    f.g = ctx->g_pad + kTablePad;
    f.h = ctx->h_pad + kTablePad;
    f.l1 = l1;
    f.l2 = l2;
    f.out = out;
    f.stride = stride;
    f.lmax_max = ctx->lmax_max;
    f.rot = rot;
    f.flip = flip;
    auto launch_form = [&](auto ab, auto threads, auto piece) {
        constexpr int AB = decltype(ab)::value, T = decltype(threads)::value, PIECE = decltype(piece)::value;
        const dim3 grid = piece_grid(n_pairs, stride, PIECE);
        if (rot == 0)
            hipLaunchKernelGGL((threej_family_row_kernel<AB, T, PIECE>), grid, dim3(T), 0, s, f);
        else
            hipLaunchKernelGGL((threej_family_kernel<AB, T, PIECE>), grid, dim3(T), 0, s, f);
    };
    auto launch = [&](auto ab) {
        if (stride <= kThreejShort)
            launch_form(ab, std::integral_constant<int, 64>(), std::integral_constant<int, kThreejPiece>());
        else if (past_cache(n_pairs, stride))
            launch_form(ab, std::integral_constant<int, 256>(), std::integral_constant<int, kFamilyPastPiece>());
        else
            launch_form(ab, std::integral_constant<int, 256>(), std::integral_constant<int, kThreejPiece>());
    };
    switch (3 * a + b) {
    case 0: launch(std::integral_constant<int, 0>()); break;
    case 1: launch(std::integral_constant<int, 1>()); break;
    case 2: launch(std::integral_constant<int, 2>()); break;
    case 3: launch(std::integral_constant<int, 3>()); break;
    case 4: launch(std::integral_constant<int, 4>()); break;
    case 5: launch(std::integral_constant<int, 5>()); break;
    case 6: launch(std::integral_constant<int, 6>()); break;
    case 7: launch(std::integral_constant<int, 7>()); break;
    case 8: launch(std::integral_constant<int, 8>()); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_threej_rows(const couple_ctx* ctx, int m, int n_pairs, const int* l1, const int* l2, double* out,
                              long long stride, hipStream_t s) {
    ThreejArgs a;
    a.g = ctx->g_pad + kTablePad;
    a.h = ctx->h_pad + kTablePad;
    a.cl = ctx->cl;
    a.l1 = l1;
    a.l2 = l2;
    a.out = out;
    a.stride = stride;
    a.lmax_max = ctx->lmax_max;
    a.m = m;
    const bool past = past_cache(n_pairs, stride);
    if (m == 0 && past && stride >= kZeroRowsFrom && stride <= kZeroRowsTo)
        hipLaunchKernelGGL(threej_zero_rows_kernel, dim3((unsigned)n_pairs), dim3(256), kZeroRowsLds, s, a);
    else if (stride <= kThreejShort)
        hipLaunchKernelGGL((threej_rows_kernel<64, kThreejPiece>), piece_grid(n_pairs, stride, kThreejPiece), dim3(64), 0, s, a);
    else if (past)
        hipLaunchKernelGGL((threej_rows_kernel<256, kThreejPastPiece>), piece_grid(n_pairs, stride, kThreejPastPiece), dim3(256), 0,
                           s, a);
    else
        hipLaunchKernelGGL((threej_rows_kernel<256, kThreejPiece>), piece_grid(n_pairs, stride, kThreejPiece), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace couple
