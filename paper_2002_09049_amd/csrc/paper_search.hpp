// The search of the paper's grid for the best scale (see fit_paper.hip), one
// workgroup of kT threads per residual.  The including file gives what joins
// the threads: threadIdx, block_reduce with MinOp (reduce.hpp) and block_best.
#pragma once

#include <math.h>

namespace mpq {

namespace {

struct Best {
    double e;
    long long g;
};

__device__ __forceinline__ Best better(Best x, Best y)
{
    return (y.e < x.e || (y.e == x.e && y.g < x.g)) ? y : x;
}

template <int kT>
__device__ Best block_best(Best v, double *se, long long *sg);

// E(a) from the sorted magnitudes s and their prefix sums S; also A, B.  A
// magnitude exactly at a (k + 1/2) has the code of the even neighbour (Eq.
// (2)'s ties to even): past level k when k + 1 is even.  The searches of kB
// levels run side by side (a search alone waits for LDS at every step), and
// the terms are added in the order of the levels.
// c: the last kB levels' counts (all levels' when M <= kB).
template <int kB>
__device__ __forceinline__ double paper_error(const double *s, const double *S, int d, int dpad, int M, double R,
                                              double a, double &A, double &B, int (&c)[kB])
{
    double sa = 0.0, sb = 0.0;
    for (int k0 = 0; k0 < M; k0 += kB) {
        double thr[kB];
#pragma unroll
        for (int z = 0; z < kB; ++z) {
            thr[z] = k0 + z < M ? a * ((double)(k0 + z) + 0.5) : INFINITY;
            c[z] = 0;
        }
        // c = the number of s above thr (odd levels: or at it); the pads, -1,
        // are below every threshold
        auto above = [&](int z, int at) { return (z & 1) ? s[at] >= thr[z] : s[at] > thr[z]; };
        for (int step = dpad >> 1; step > 0; step >>= 1) {
#pragma unroll
            for (int z = 0; z < kB; ++z) c[z] += above(z, c[z] + step - 1) ? step : 0;
        }
#pragma unroll
        for (int z = 0; z < kB; ++z) c[z] = min(c[z] + (above(z, c[z]) ? 1 : 0), d);
        double v[kB];
#pragma unroll
        for (int z = 0; z < kB; ++z) v[z] = S[c[z]];
#pragma unroll
        for (int z = 0; z < kB; ++z) {
            sa += v[z];
            sb += (double)(2 * (k0 + z) + 1) * (double)c[z];
        }
    }
    A = sa;
    B = sb;
    return (R - 2.0 * a * sa) + a * a * sb;
}

// whether every level's count at a is c's (M <= kB): a lies in the same piece
template <int kB>
__device__ __forceinline__ bool same_piece(const double *s, int d, int M, double a, const int (&c)[kB])
{
    bool same = true;
#pragma unroll
    for (int z = 0; z < kB; ++z) {
        if (z >= M) break;
        const double thr = a * ((double)z + 0.5);
        const double last = s[max(c[z] - 1, 0)], next = s[min(c[z], d - 1)];
        same = same && (c[z] == 0 || ((z & 1) ? last >= thr : last > thr)) &&
               (c[z] == d || !((z & 1) ? next >= thr : next > thr));
    }
    return same;
}

constexpr int kMarks = 4;   // marks per thread

// The best point of the grid g gamma, g = 1 .. count, for the sorted
// magnitudes s (descending, pads -1 up to dpad, a power of two) and their
// prefix sums S.  First E, A and B at kMarks kT marks (grid points, evenly
// spaced in log a from s_max / (8 M) to 2 s_max, where every code is zero)
// bound E between the marks: A and B do not grow with a, so between marks lo
// and hi E' = -2 A + 2 a B lies in [-2 A_lo + 2 lo B_hi, -2 A_hi + 2 hi B_lo],
// and E above the two lines with these slopes through the marks.  Intervals
// whose bound exceeds the least E of a mark hold no argmin (the bound's slack
// is second order in their width: about 2 R (0.5%)^2 here); what is left is a
// short range of a, and only the breakpoints in it and the piece that holds
// its lower end are searched (the pieces in it are each tried from the
// breakpoint on their left; one that reaches below the range, or down to 0,
// has none there).  The marks themselves are candidates.
template <int kT, int kB>
__device__ Best paper_search_n(const double *s, const double *S, int d, int dpad, int M, double R, double gamma,
                             long long count, double *s_red, long long *s_redg)
{
    const int t = threadIdx.x;
    const double smax = s[0], margin = 1e-10 * R;
    // mark i, i = 0 .. kMarks kT (the last one past 2 s_max)
    constexpr int kN = kMarks * kT;
    const float span = log2f(16.0f * (float)M) / (float)kN;
    auto mark = [&](int i) {
        const double raw = i == kN ? 2.0 * smax + 1.5 * gamma
                                   : smax / (8.0 * (double)M) * (double)exp2f(span * (float)i);
        const long long g = (long long)fmin(floor(raw / gamma), 4e18);
        return min(max(g, 1ll), count);
    };
    double a[kMarks + 1], A[kMarks + 1], Bq[kMarks + 1], E[kMarks + 1];
    long long g_last = 0;
    Best best{INFINITY, 0x7fffffffffffffffLL};
    if (count >= 1) {
#pragma unroll 1
        for (int z = 0; z <= kMarks; ++z) {
            const long long g = mark(t * kMarks + z);
            const double az = (double)g * gamma;
            double Az, Bz;
            int c[kB];
            const double Ez = paper_error<kB>(s, S, d, dpad, M, R, az, Az, Bz, c);
            best = better(best, Best{Ez, g});
#pragma unroll
            for (int y = 0; y <= kMarks; ++y) {
                if (y == z) {
                    a[y] = az;
                    A[y] = Az;
                    Bq[y] = Bz;
                    E[y] = Ez;
                }
            }
            g_last = g;
        }
    }
    const double U = block_reduce<kT>(best.e, MinOp(), s_red);
    // the range of a left: [alo, ahi]
    double alo = INFINITY, ahi = 0.0;
    auto interval = [&](double lo, double Alo, double Blo, double Elo, double hi, double Ahi, double Bhi,
                        double Ehi) {
        const double m1 = -2.0 * Alo + 2.0 * lo * Bhi, m2 = -2.0 * Ahi + 2.0 * hi * Blo, w = hi - lo;
        double lb;
        if (m1 >= 0.0) {
            lb = Elo;
        } else if (m2 <= 0.0) {
            lb = Ehi;
        } else {
            const double x = (Ehi - m2 * w - Elo) / (m1 - m2);
            lb = Elo + m1 * fmin(fmax(x, 0.0), w);
        }
        if (!(lb > U + margin)) {
            alo = fmin(alo, lo);
            ahi = fmax(ahi, hi);
        }
    };
    if (count >= 1) {
        if (t == 0)
            interval(0.0, (double)M * S[d], (double)M * (double)M * (double)d, R, a[0], A[0], Bq[0], E[0]);
#pragma unroll
        for (int z = 0; z < kMarks; ++z) interval(a[z], A[z], Bq[z], E[z], a[z + 1], A[z + 1], Bq[z + 1], E[z + 1]);
        // past the last mark every code is zero, E = R (or no grid point is left)
        if (t == kT - 1 && g_last < count && !(R > U + margin)) ahi = INFINITY;
        if (ahi == INFINITY) alo = fmin(alo, a[kMarks]);
    }
    alo = block_reduce<kT>(alo, MinOp(), s_red);
    ahi = -block_reduce<kT>(-ahi, MinOp(), s_red);
    if (!(alo <= ahi)) return block_best<kT>(best, s_red, s_redg);   // uniform: no grid point
    auto try_g = [&](long long g) {
        if (g < 1 || g > count) return;
        double Ag, Bg;
        int c[kB];
        const double Eg = paper_error<kB>(s, S, d, dpad, M, R, (double)g * gamma, Ag, Bg, c);
        best = better(best, Best{Eg, g});
    };
    // The grid points next to the vertex of a piece (A, B; counts c): its
    // quadratic has its minimum R - A^2 / B there, a lower bound for every
    // grid point of the piece: skipped when it already exceeds the least error
    // found (with a margin for rounding).  Where the vertex lies outside its
    // piece (nearly always) the points belong to other pieces, which try them
    // themselves.
    auto try_vertex = [&](double Ag, double Bg, const int (&c)[kB]) {
        if (Bg > 0.0 && R - Ag * Ag / Bg <= fmin(best.e, U) + 1e-12 * R) {
            const long long gv = (long long)fmin(floor((Ag / Bg) / gamma), 4e18);
            for (long long g = gv; g <= gv + 1; ++g) {
                if (M > kB) {
                    try_g(g);
                } else if (g >= 1 && g <= count && same_piece<kB>(s, d, M, (double)g * gamma, c)) {
                    const double x = (double)g * gamma;
                    best = better(best, Best{(R - 2.0 * x * Ag) + x * x * Bg, g});
                }
            }
        }
    };
    // |E'| <= 2 max(A, a B) in the range: what E may fall over two grid steps
    const double fall = 4.0 * gamma * fmax((double)M * S[d], (ahi + 4.0 * gamma) * (double)M * (double)M * (double)d);
    // The breakpoints s_j / (k + 1/2) with a grid point next to them in the
    // range (margins for the products' roundings): for each level a run of j.
    // A level's runs are dealt to the threads from where the last one's ended.
    const double blo = (alo - 3.0 * gamma) * (1.0 - 1e-12), bhi = (ahi + 3.0 * gamma) * (1.0 + 1e-12);
    auto above = [&](double x) {   // #{ j : s_j > x }
        if (!(x > 0.0)) return d;
        int c = 0;
        for (int step = dpad >> 1; step > 0; step >>= 1) c += s[c + step - 1] > x ? step : 0;
        c += s[c] > x ? 1 : 0;
        return min(c, d);
    };
    int shift = 0;
    for (int kl = 0; kl < M; ++kl) {
        const double h = (double)kl + 0.5;
        const int j0 = above(bhi * h), j1 = above(blo * h);
        for (int j = j0 + (t + kT - shift) % kT; j < j1; j += kT) {
            const double b = s[j] / h;
            if (!(b > 0.0)) continue;
            long long g0 = (long long)fmin(floor(b / gamma), 4e18);
            // The first grid point above the breakpoint, g0 + 1, is the first
            // of the piece that begins there; the ones at or below it are at
            // most `fall` less.  Breakpoints often fall on the grid (gamma is
            // a fraction of a gap), and floor may lose one to a rounding: then
            // the level's own comparison still has g0 + 1 on the left.  Past
            // 2^49 grid points even the next one may round onto the
            // breakpoint: the piece is then entered a little right of it.
            auto left = [&](long long g) {
                const double thr = (double)g * gamma * h;
                return (kl & 1) ? s[j] >= thr : s[j] > thr;
            };
            if (left(g0 + 1)) ++g0;
            double E1 = -INFINITY;
            if (g0 + 1 <= count) {
                const bool on = left(g0 + 1);
                double Ag, Bg;
                int c[kB];
                E1 = paper_error<kB>(s, S, d, dpad, M, R, on ? b * (1.0 + 0x1p-49) : (double)(g0 + 1) * gamma, Ag, Bg, c);
                if (!on) best = better(best, Best{E1, g0 + 1});
                try_vertex(Ag, Bg, c);
            }
            if (!(E1 - fall > fmin(best.e, U) + margin)) {
                for (long long g = g0 - 1; g <= g0; ++g) {
                    if (g < 1 || g > count) continue;
                    double Ag, Bg;
                    int c[kB];
                    const double Eg = paper_error<kB>(s, S, d, dpad, M, R, (double)g * gamma, Ag, Bg, c);
                    best = better(best, Best{Eg, g});
                    try_vertex(Ag, Bg, c);
                }
            }
        }
        shift = (shift + max(j1 - j0, 0)) % kT;
    }
    // The piece that begins below the range and reaches into it; of a range
    // from 0 (the best scale may saturate every weight, left of all
    // breakpoints) the one that holds the first grid point.
    if (t == shift) {
        double Ag, Bg;
        int c[kB];
        const double Eg = paper_error<kB>(s, S, d, dpad, M, R, fmax(alo, gamma), Ag, Bg, c);
        if (!(alo > 0.0)) best = better(best, Best{Eg, 1});
        try_vertex(Ag, Bg, c);
    }
    return block_best<kT>(best, s_red, s_redg);
}

template <int kT>
__device__ __forceinline__ Best paper_search(const double *s, const double *S, int d, int dpad, int M, double R,
                                             double gamma, long long count, double *s_red, long long *s_redg)
{
    return M <= 4 ? paper_search_n<kT, 4>(s, S, d, dpad, M, R, gamma, count, s_red, s_redg)
                  : paper_search_n<kT, 8>(s, S, d, dpad, M, R, gamma, count, s_red, s_redg);
}

}  // namespace

}  // namespace mpq
