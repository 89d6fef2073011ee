// The histogram search of the greedy multipoint fit (Algorithm 1, Sec. 3.2,
// with the stopping rule of Algorithm 2, Sec. 3.3): an exact O(d M + G)
// evaluation of the candidate errors of Eq. (9).
//
// For a candidate scale a and x = |r_j|, the code magnitude of element j is
// the number of levels k in [0, M) whose boundary (k + 1/2) a lies below x
// (Eq. (2); an exact half-way point gives the same error either way).  The
// candidates ascend, so for each (j, k) the ones that lift element j past
// level k are a prefix g < n_jk, n_jk = #{ g : (k + 1/2) a_g < x_j }.  With
// A(g) = sum_j x_j |q_j(g)| and B(g) = sum_j q_j(g)^2,
//     E(g) = ||r||^2 - 2 a_g A(g) + a_g^2 B(g),
// and A, B are suffix sums of histograms over n_jk.  LDS atomics on integers
// (x in fixed point, a count above it in the same 64-bit word) make the
// histograms independent of the order of the elements.
//
// Every E(g) carries an error bound; a candidate whose interval reaches the
// smallest E's is a finalist, and when there is more than one, the finalists
// are evaluated directly (fp64, Eq. (9) written out) and the smallest error
// wins, ties to the smallest g.  The bound makes room for two shortcuts:
//
//  - Boundaries are located in units of the default grid's spacing, without
//    a look at the candidates' own fp32 roundings.  An element on the wrong
//    side of a boundary that lies within t of it costs 2 a |x - (k + 1/2) a|
//    <= 2 a t x, at most once per element, and sum x <= sqrt(d) ||r||.
//  - (modes other than lattice) Candidates that cannot win are left out: the
//    largest element alone costs max(0, m - M a_g)^2, so with the error E_top
//    of the largest candidate every c_g < 1 - sqrt(E_top) / m loses to it.
//    Short channels and wide codes lose most of their candidates this way
//    (at 8 bits nine in ten), and with them most level boundaries.
//
// Modes:
//  lattice  default grid, long channels.  With u = m / (2 G M) every boundary
//           (k + 1/2) a_g lies within relative 2^-23 of L u, L = (2k+1)(g+1),
//           so an element goes to the one bucket floor(x / u) and A(g), B(g)
//           are sums over k of suffix sums at L: one atomic per element, and
//           a pass over (2M-1) G buckets per step.
//  linear   default grid, M <= 7: one atomic per (element, level) into G bins.
//  wide     default grid, M >= 15: the same from the element's code at the
//           largest candidate upwards, and two words per bin (the counts of
//           up to 127 levels do not fit beside x).
//  grid     a caller's grid: as wide, the bin found from a table of the grid
//           over 1/1024ths and exact comparisons.
//
// One workgroup of T threads per channel, the fp64 residual in registers for
// the whole fit (EPT elements per thread), so a step reads nothing from HBM.
// What bounds the kernel is VALU issue (the SIMDs' VALU is 84% busy on the
// linear mode's channels of 256 weights and 76% on those of 512, 50% on the
// lattice mode's) and, with few wavefronts in flight, the latency of a step's
// serial phases.  By the instructions of ResNet-50's launches (3.1 points a
// channel) an element costs about 40 a step in the lattice mode and 85 in the
// linear one at 7 levels, a wavefront about 500 and 350 more
// (reductions, scan, candidates), so a channel takes as few wavefronts as its
// registers allow: one up to 1280 elements, without barriers.  Measured alone
// against the kernel that this one replaced (64 to 1024 threads of up to nine
// elements, exact comparisons at every boundary, a bucket per lattice point;
// 4 bits, 256 candidates, about 2 to 4 points a channel):
//   7168 x 64    37 -> 26 us     7808 x 512   169 -> 79 us
//   4032 x 1024 150 -> 83 us     1536 x 2304  113 -> 53 us
//   1536 x 4608 173 -> 78 us     4096 x 25088 (3 bits, 512) 1916 -> 1122 us
//   1000 x 2048 at 8 bits 422 -> 61 us
#pragma once

#include <math.h>
#include <stdio.h>

#include "internal.hpp"
#include "mpq.h"
#include "reduce.hpp"

namespace mpq {

enum HistMode { kHistLattice = 0, kHistLinear = 1, kHistWide = 2, kHistGrid = 3 };

constexpr int kHistTable = 1024;       // grid mode: entries of the count table
constexpr int kHistDump = 32;          // lattice mode: words that take the elements below every boundary
constexpr int kMaxFinalists = 32;      // listed; more than that are found by a scan

namespace hist {

// fixed-point words of the lattice buckets: x below bit 48, the count above
constexpr int kLatShift = 48;

// a workgroup's barrier; the LDS accesses of a single wavefront are in order
template <int T>
__device__ __forceinline__ void sync()
{
    if constexpr (T > kWave) __syncthreads();
    else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// A value every lane holds alike, moved to scalar registers.
__device__ __forceinline__ double uni(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ float uni(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// 1 / x to within an ulp or so (x normal), for uses that allow for that.
__device__ __forceinline__ double recip(double x)
{
    double y = __builtin_amdgcn_rcp(x);   // 2^-26 or better
    y = fma(fma(-x, y, 1.0), y, y);
    return fma(fma(-x, y, 1.0), y, y);
}

// fl64(r / a), ia = recip(a): q0 = r ia is within 2 ulp of the quotient, so
// r - q0 a is exact (a has 24 bits) and one correction leaves q0 plus a term
// with relative error 2^-51.  The quotient of a 53-bit and a 24-bit number
// lies at least 2^-25 ulp from every midpoint of doubles (a midpoint times a
// needs more than 53 bits unless a is a power of two, when the quotient is
// exact), so that rounds as the division does.
__device__ __forceinline__ double quotient(double r, double a, double ia)
{
    const double q0 = r * ia;
    return fma(fma(-q0, a, r), ia, q0);
}

// The best candidate (e, g) seen, its lower bound lb, and the least lower
// bound of the others.
struct Lead {
    double e, lb, rest;
    int g;
};

__device__ __forceinline__ void lead_add(Lead &L, double e, double lb, int g)
{
    const bool win = e < L.e || (e == L.e && g < L.g);
    L.rest = fmin(L.rest, win ? L.lb : lb);
    L.e = win ? e : L.e;
    L.lb = win ? lb : L.lb;
    L.g = win ? g : L.g;
}

}  // namespace hist

// Lattice mode's geometry for T threads: n distinct boundary points in chunks
// of `per` per thread, the top chunk first; `pad` words lie below the first
// point.  An odd chunk keeps the lanes of a wavefront on distinct LDS banks.
struct LatticeShape {
    int n, per, pad;
};
__host__ __device__ inline LatticeShape lattice_shape(int T, int points)
{
    LatticeShape s;
    s.n = points;
    s.per = ((s.n + T - 1) / T) | 1;
    s.pad = s.per * T - s.n;
    return s;
}

// Dynamic LDS (bytes) of a workgroup of T threads.
// points: the lattice's distinct boundary points.
__host__ __device__ inline size_t hist_lds(int mode, int T, int M, int G, int points)
{
    if (mode == kHistLattice)
        return 8 * (size_t)(kHistDump + lattice_shape(T, points).per * T) + 2 * (size_t)((2 * M - 1) * G + 8);
    size_t b = 8 * (size_t)(G + 1 + (mode == kHistLinear ? 64 : 0));   // x sums (linear: with counts)
    if (mode != kHistLinear) b += 4 * (size_t)(G + 1);                // counts
    if (mode == kHistGrid) b += 8 * (size_t)(G + 1) + 2 * (kHistTable + 2);   // c_g, a_g, table
    return (b + 15) / 16 * 16;
}

// Wavefronts per SIMD the register budget aims at: the residual takes 2 EPT
// VGPRs and a step about 50 more; a workgroup of 1024 threads needs four.
template <int T, int EPT, int kMode>
constexpr int hist_waves_per_simd()
{
    return EPT <= 4 ? 6 : EPT <= 8 ? 5 : EPT <= 20 ? (kMode == kHistLattice ? 3 : 4) : EPT <= 36 ? 3 : 2;
}

std::string hist_name(int T, int EPT, int mode);

// kM: the levels M (a template argument in the lattice and linear modes, so
// that their loops over levels unroll without guards), or 0 for B.M.
template <int T, int EPT, int kMode, int kM>
__global__ void __launch_bounds__(T)
__attribute__((amdgpu_waves_per_eu(hist_waves_per_simd<T, EPT, kMode>())))
fit_hist_kernel(const HistBatch B)
{
    using namespace hist;
    typedef unsigned long long u64;
    constexpr int kWaves = T / kWave;
    // a thread's elements: groups of kC consecutive ones, element u = kC v + c
    // being j = kC (t + T v) + c
    constexpr int kC = EPT >= 4 ? 4 : 1;
    constexpr int kSlots = EPT / kC;
    static_assert(EPT % kC == 0, "whole groups");

    extern __shared__ __align__(16) char hsmem[];
    __shared__ double s_red[2][kWaves];      // per-wave maxima, two sets in turn
    __shared__ double s_part[kWaves > 1 ? 2 : 1][kWaves > 4 ? kWaves : 4][kWaves > 1 ? kWave : 1];   // partial sums
    __shared__ u64 s_scan[kWaves];
    __shared__ int s_pick[2];                // the chosen candidate, whether there are finalists
    __shared__ int s_nfin, s_fin[kMaxFinalists];

    const int li = last_at_most(B.n_layers, (int)blockIdx.x, [&](int i) { return B.L[i].c_begin; });
    const HistLayer &Ly = B.L[li];
    const int G = B.G, P = B.P, M = kM > 0 ? kM : B.M;
    const int64_t k = (int64_t)blockIdx.x - Ly.c_begin;
    int t = threadIdx.x, lane = t % kWave;
    const int wid = __builtin_amdgcn_readfirstlane(t / kWave);
    const int d = Ly.d;   // <= kHistMaxDim; offsets inside a channel fit 32 bits
    const double Md = uni((double)M), rM = uni(1.0 / Md);
    int8_t *qk = Ly.codes + k * (int64_t)P * d;
    const float *wk = Ly.W + k * (int64_t)d;

    const bool stepping = B.single != 0;   // a calibration step: at most one point
    const int s0 = B.start;                // resumes the channels that hold s0 points
    if (s0 >= 1 && Ly.counts[k] != s0) return;   // uniform

    // groups of four: one 16-byte load of W, one 32-bit word of codes
    const bool vec = kC == 4 && d % 4 == 0 && (uintptr_t)wk % 16 == 0 && (uintptr_t)qk % 4 == 0;

    double r[EPT];
    double beta = 0.0;
    // f(v, first element) for the slots that hold elements in some thread
    // (thread and length made opaque here: hoisted out of the step loop, the
    // slots' addresses and bounds would fill the registers)
    auto each_slot = [&](auto &&f) {
        int tt = t, dd = d;
        asm volatile("" : "+v"(tt));
        asm volatile("" : "+s"(dd));
#pragma unroll
        for (int v = 0; v < kSlots; ++v)
            if (kC * T * v < dd) f(v, kC * (tt + T * v), dd);   // uniform
    };
    // the residual after the first np stored points, with the fp64
    // operations of the running one in point order (0 past the channel)
    auto load_residual = [&](int np, double beta) {
#pragma unroll
        for (int u = 0; u < EPT; ++u) r[u] = 0.0;
        each_slot([&](int v, int j0, int d) {
            if (vec) {
                if (j0 < d) {
                    const float4 w4 = *(const float4 *)(wk + j0);
                    const float w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                    for (int c = 0; c < kC; ++c) r[v * kC + c] = (double)w[c % 4] - beta;
                }
            } else {
#pragma unroll
                for (int c = 0; c < kC; ++c)
                    if (j0 + c < d) r[v * kC + c] = (double)wk[j0 + c] - beta;
            }
        });
        for (int p = 0; p < np; ++p) {
            const double a = -(double)Ly.scales[k * P + p];
            const int8_t *row = qk + (int64_t)p * d;
            each_slot([&](int v, int j0, int d) {
                if (vec) {
                    if (j0 < d) {
                        const uint32_t q = *(const uint32_t *)(row + j0);
#pragma unroll
                        for (int c = 0; c < kC; ++c)
                            r[v * kC + c] = fma(a, (double)(int)(int8_t)(uint8_t)(q >> (8 * c)), r[v * kC + c]);
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < kC; ++c)
                        if (j0 + c < d) r[v * kC + c] = fma(a, (double)row[j0 + c], r[v * kC + c]);
                }
            });
        }
    };
    // the codes of a slot (bytes past the channel are not stored)
    auto store_codes = [&](int8_t *row, int j0, int d, uint32_t q) {
        if (vec) {
            if (j0 < d) *(uint32_t *)(row + j0) = q;
        } else {
#pragma unroll
            for (int c = 0; c < kC; ++c)
                if (j0 + c < d) row[j0 + c] = (int8_t)(uint8_t)(q >> (8 * c));
        }
    };
    // The sum of a channel's terms runs in an order that does not depend on
    // T (64, 128 or 256): the elements' groups of 64 lanes are dealt to four
    // partial sums in turn, each lane adds its four in order, then the lanes.
    // So a channel's fit is the same bit for bit whether one wavefront takes
    // it or four.  A thread holds the kPart of the four that its groups go to
    // (T = 512, longer channels: one per wavefront).
    constexpr int kPart = T >= 256 ? 1 : 256 / T;
    int rset = 0;   // two scratch sets in turn: one barrier per reduction
    auto put_parts = [&](const double (&p)[kPart]) {
        if constexpr (kWaves > 1) {
#pragma unroll
            for (int q = 0; q < kPart; ++q) s_part[rset][wid + q * kWaves][lane] = p[q];
        }
    };
    auto add_parts = [&](const double (&p)[kPart]) {   // after the barrier
        double x;
        if constexpr (kWaves > 1) {
            x = s_part[rset][0][lane];
#pragma unroll
            for (int q = 1; q < kPart * kWaves; ++q) x += s_part[rset][q][lane];
        } else {
            x = p[0];
#pragma unroll
            for (int q = 1; q < kPart; ++q) x += p[q];
        }
        return uni(wave_reduce(x, SumOp()));
    };
    auto total = [&](const double (&p)[kPart]) {
        put_parts(p);
        if constexpr (kWaves > 1) __syncthreads();
        const double x = add_parts(p);
        rset ^= 1;
        return x;
    };
    // the maximum of one value and such a sum, with one barrier
    auto max_total = [&](double &mx, const double (&p)[kPart]) {
        mx = wave_reduce(mx, MaxOp());
        put_parts(p);
        if constexpr (kWaves > 1) {
            if (lane == 0) s_red[rset][wid] = mx;
            __syncthreads();
            mx = s_red[rset][0];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) mx = MaxOp()(mx, s_red[rset][w]);
        }
        mx = uni(mx);
        const double x = add_parts(p);
        rset ^= 1;
        return x;
    };
    // two sums (in an order of their own: their users allow for the rounding)
    auto sum2 = [&](double &x, double &y) {
        x = wave_reduce(x, SumOp());
        y = wave_reduce(y, SumOp());
        if constexpr (kWaves > 1) {
            if (lane == 0) {
                s_part[rset][0][wid] = x;
                s_part[rset][1][wid] = y;
            }
            __syncthreads();
            x = s_part[rset][0][0];
            y = s_part[rset][1][0];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) {
                x += s_part[rset][0][w];
                y += s_part[rset][1][w];
            }
            rset ^= 1;
        }
        x = uni(x);
        y = uni(y);
    };

    // asymmetric codes (reading B2): the points fit w - beta, beta the fp32
    // midpoint of the channel's range; the stopping rule keeps ||w||^2
    double Ew = 0.0;
    const bool asym = Ly.offsets != nullptr;
    if (asym) {
        double mx = -INFINITY, mn = -INFINITY;
        for (int j = t; j < d; j += T) {
            mx = fmax(mx, (double)wk[j]);
            mn = fmax(mn, -(double)wk[j]);
        }
        const double none[kPart] = {};
        max_total(mx, none);
        max_total(mn, none);
        const float b = uni((float)((mx - mn) / 2.0));
        beta = (double)b;
        beta = uni(beta);
        if (t == 0) Ly.offsets[k] = b;
    }
    if (asym || (s0 >= 1 && !stepping)) {   // ||w||^2 when the first residual is not w
        load_residual(0, 0.0);
        double sw[kPart] = {};
#pragma unroll
        for (int u = 0; u < EPT; ++u) sw[u / kC % kPart] = fma(r[u], r[u], sw[u / kC % kPart]);
        Ew = total(sw);
    }
    load_residual(s0, beta);

    u64 *lat = (u64 *)hsmem;                                  // lattice: dump, pad, buckets
    u64 *ha = (u64 *)hsmem;                                   // [G + 1] sums at bin n; linear: and one of each lane's own
    uint32_t *hb = (uint32_t *)(ha + G + 1);                  // wide, grid: [G + 1] counts at bin n
    float *s_c = (float *)(hb + G + 1);                       // grid: [G] c_g
    float *s_a = s_c + G;                                     // grid: [G + 2] a_g, then +inf
    uint16_t *s_tab = (uint16_t *)(s_a + G + 2);              // grid: [kHistTable + 1]
    // a_g = fl32(m c_g / M), c_g the caller's multiplier or the default
    // fl32((g + 1) / G), the correctly rounded fp32 quotient (for G = 2^k
    // that is (g + 1) 2^-k).  m c_g is exact in fp64 (48 bits), and one
    // residual step rounds its quotient as a division would (a 48-bit number
    // over M <= 127 lies at least 2^-8 ulp from every midpoint of doubles).
    const bool pow2 = kMode != kHistGrid && (G & (G - 1)) == 0;
    const double rG = uni((double)__fdiv_rn(1.0f, (float)G));
    float m = 0.0f;
    double mG = 0.0;   // m / G for G = 2^k (exact)
    auto cand = [&](int g) {
        double x;
        if constexpr (kMode == kHistGrid) x = (double)m * (double)s_c[g];
        else x = pow2 ? (double)(g + 1) * mG : (double)m * (double)__fdiv_rn((float)(g + 1), (float)G);
        const double q = x * rM;
        return (float)fma(fma(-q, Md, x), rM, q);
    };
    // inclusive prefix sums of p[0 .. n - 1], a run of entries per thread
    auto prefix_sums = [&](uint16_t *p, int n) {
        sync<T>();
        const int per = (n + T - 1) / T;
        const int b0 = min(t * per, n), b1 = min(b0 + per, n);
        uint32_t tot = 0;
        for (int b = b0; b < b1; ++b) tot += p[b];
        uint32_t run = wave_prefix_sum(tot) - tot;
        if constexpr (kWaves > 1) {
            if (lane == kWave - 1) s_scan[wid] = run + tot;
            __syncthreads();
            for (int w = 0; w < wid; ++w) run += (uint32_t)s_scan[w];
        }
        for (int b = b0; b < b1; ++b) {
            run += p[b];
            p[b] = (uint16_t)run;
        }
        sync<T>();
    };
    if constexpr (kMode == kHistGrid) {
        // entry i: the multipliers below i / kHistTable less a margin for the
        // roundings of a query, counted at their first entry and summed up (a
        // binary search per entry took 5 us)
        for (int i = t; i < (kHistTable + 2) / 2; i += T) ((uint32_t *)s_tab)[i] = 0;
        sync<T>();
        for (int g = t; g < G; g += T) {
            const float c = B.grid[g];
            s_c[g] = c;
            int i = (int)(c * (float)kHistTable);
            while (i <= kHistTable && !(c < ((float)i - 0.001f) / (float)kHistTable)) ++i;   // at most three steps
            if (i <= kHistTable) atomicAdd((uint32_t *)s_tab + i / 2, 1u << (16 * (i % 2)));
        }
        prefix_sums(s_tab, kHistTable + 1);
    }
    const LatticeShape LS = lattice_shape(T, B.points);
    auto clear_lattice = [&]() {
        u64 *p = lat + kHistDump + t;
        const int n = LS.n + LS.pad;
        int b = 0;
#pragma unroll 1
        for (; b + 8 * T <= n; b += 8 * T) {
#pragma unroll
            for (int y = 0; y < 8; ++y) p[b + y * T] = 0;
        }
#pragma unroll 1
        for (; b + t < n; b += T) p[b] = 0;
    };
    // lattice: s_rank[b] = 8 times the number of boundary points
    // L = (2k+1)(g+1) up to b, the byte offset of bucket b's word past the
    // pad's last one.  Only the points need a word (1261 of 3328 at 4 bits
    // and 256 candidates), which shortens the scan of every step.
    uint16_t *s_rank = (uint16_t *)(lat + kHistDump + LS.per * T);
    const int last = (2 * M - 1) * G;
    if constexpr (kMode == kHistLattice) {
        for (int b = t; b <= last; b += T) s_rank[b] = 0;
        sync<T>();
        for (int g = t; g < G; g += T)
#pragma unroll
            for (int kk = 0; kk < kM; ++kk) s_rank[(2 * kk + 1) * (g + 1)] = 8;
        prefix_sums(s_rank, last + 1);
    }
    u64 full = 0;   // linear: the levels every candidate passes

    float apend = 0.0f;
    int n = 0;
    bool more = false;   // calibration step: the channel took its point and goes on
    // Algorithm 2's naive point (reading F1).  Calibration fit, first step:
    // the point is stored with its output error; the channel keeps it (and
    // takes no other) when that error meets the threshold.  Fresh fit:
    // gstate 1 takes the naive point at step 0, gstate 2 decides at step 1,
    // after it is applied, whether it stays or the fit restarts from w.
    bool kept = false;
    if (B.gate && stepping && s0 == 0) {
        const double thr = Ly.ref ? B.eps * (double)Ly.ref[k] : B.eps;
        kept = Ly.counts[k] == 1 && (double)Ly.xerr[k * P] <= thr;   // uniform
        if (kept) n = 1;
    }
    int gstate = (B.gate && !stepping && s0 == 0) ? 1 : 0;
    for (int i = s0; !kept; ++i) {
        // what a step derives from the thread's index is formed again in
        // each one: kept across the loop it would be spilled
        asm volatile("" : "+v"(t));
        lane = t % kWave;
        // ---- apply the pending point: codes of Eq. (10), the fp64 quotient
        // r / a rounded and clipped; residual of Eq. (7)
        double lmax = 0.0, lsum[kPart] = {};
        if (i > s0) {
            const double a = uni((double)apend), ia = uni(recip(a));
            int8_t *qrow = qk + (int64_t)(i - 1) * d;
            auto code_of = [&](double x) { return fmin(fmax(rint(quotient(x, a, ia)), -Md), Md); };
            // the scale of the update: the searched one, or (refit) the
            // least-squares scale of the codes, fl32(<r, q> / <q, q>)
            double aupd = a;
            if (B.refit && gstate != 2) {   // the naive point keeps its scale
                double rq[kPart] = {}, qq[kPart] = {};
                each_slot([&](int v, int, int) {
#pragma unroll
                    for (int c = 0; c < kC; ++c) {
                        const double q = code_of(r[v * kC + c]);
                        rq[v % kPart] = fma(r[v * kC + c], q, rq[v % kPart]);
                        qq[v % kPart] = fma(q, q, qq[v % kPart]);
                    }
                });
                const double srq = total(rq), sqq = total(qq);
                const float afit = uni((float)(srq / sqq));
                if (t == 0) Ly.scales[k * P + (i - 1)] = afit;
                aupd = uni((double)afit);
            }
            each_slot([&](int v, int j0, int d) {
                uint32_t q[4] = {};
#pragma unroll
                for (int c = 0; c < kC; ++c) {
                    const double cd = code_of(r[v * kC + c]);
                    q[c] = (uint32_t)(int)cd;
                    r[v * kC + c] = fma(-aupd, cd, r[v * kC + c]);
                }
                uint32_t qw = q[0];
                if constexpr (kC == 4)   // the low bytes
                    qw = __builtin_amdgcn_perm(q[1], q[0], 0x0c0c0400u) |
                         __builtin_amdgcn_perm(q[3], q[2], 0x04000c0cu);
                store_codes(qrow, j0, d, qw);
            });
        }
        if constexpr (kMode == kHistLattice && kWaves > 1) {   // the barrier below orders it
            clear_lattice();
        }
#pragma unroll
        for (int u = 0; u < EPT; ++u) {
            lmax = fmax(lmax, fabs(r[u]));
            lsum[u / kC % kPart] = fma(r[u], r[u], lsum[u / kC % kPart]);
        }
        const double R = max_total(lmax, lsum);
        m = uni((float)lmax);
        mG = uni((double)m * rG);

        // ---- stop / point count
        if (i == 0 && !asym) Ew = R;
        else if (i > s0 && Ly.err && t == 0) Ly.err[k * P + (i - 1)] = (float)R;
        if (stepping && i > s0) {   // one point per calibration step
            n = i;
            more = true;
            break;
        }
        bool stop = (i >= P) || (R == 0.0);
        if (!stop && i >= 1) {
            if (stepping) {
                // output error of the i points on the batch (the error pass
                // of the previous step) against the threshold
                const double thr = Ly.ref ? B.eps * (double)Ly.ref[k] : B.eps;
                stop = (double)Ly.xerr[k * P + (i - 1)] <= thr;
            } else {
                stop = R <= B.tol * Ew;
            }
        }
        if (gstate == 2) {   // step 1 of a gated fit: the naive point is applied
            gstate = 0;
            if (R <= B.tol * Ew) {   // Algorithm 2's test: the only point
                n = 1;
                break;
            }
            load_residual(0, beta);   // discarded: restart from w
            i = -1;
            continue;
        }
        if (stop) {
            n = i;
            break;
        }
        if (gstate == 1) {   // step 0 of a gated fit: the naive point first
            gstate = 0;
            const float aN = (float)((double)m / Md);   // the candidate c = 1
            if (aN != 0.0f) {
                gstate = 2;
                apend = aN;
                if (t == 0) Ly.scales[k * P] = aN;
                continue;
            }
        }

        // ---- histograms.  slackA bounds the error of A(g) from the fixed
        // point, miss the cost of misplaced elements over 2 a (see above),
        // both in units of x; sum x <= sqrt(d R).  A candidate below fp32's
        // normal range adds its absolute rounding, 2^-149, per level.  The
        // fp32 square roots are of values in [1, d] (R / m^2 and its like).
        const double inv_m = uni(recip((double)m));
        const double GM = (double)(G * M);
        const double sumx = (double)m * (double)(__builtin_amdgcn_sqrtf((float)((double)d * R * inv_m * inv_m)) * 1.000001f);
        const double sub = (double)d * Md * 0x1p-148;
        double slackA = 0.0, miss = 0.0;
        double unit = 0.0;                 // of the fixed-point sums
        double A0 = 0.0, B0 = 0.0;         // wide, grid: the levels every kept candidate passes
        int g_lo = 0, cs = kLatShift;
        if constexpr (kMode == kHistLattice) {
            // fixed point: x / u with F fraction bits, sums of M d values
            // below 2^48 (x / u <= 2 G M)
            const int lg = 64 - __clzll((u64)d * (u64)M * (uint32_t)(2 * G * M + 2));
            const int F = min(kLatShift - lg, 28);
            const double S = uni(ldexp(2.0 * GM * inv_m, F));
            unit = uni(recip(S));
            slackA = 0.51 * Md * (double)d * unit;
            miss = 0x1.04p-23 * sumx + (double)d * unit + sub;
            if constexpr (kWaves == 1) clear_lattice();
            // the word x 2^F / u + 2^48 is the low 52 bits of one fma; the
            // bucket floor(x / u) is cut out of it (twice, an offset into
            // s_rank).  Bucket 0 (nothing crossed, and the zeros past the
            // channel) goes to a dump word of the lane's own.
            const double bias = 0x1p52 + 0x1p48;
            char *base = (char *)(lat + kHistDump + LS.pad - 1);   // the p-th point's word at base + 8 p
            const uint32_t dump = (uint32_t)((char *)(lat + lane % kHistDump) - base);
            each_slot([&](int v, int, int) {
                uint32_t lo[kC], hi[kC], off[kC];
#pragma unroll
                for (int c = 0; c < kC; ++c) {
                    const u64 w = (u64)__double_as_longlong(fma(fabs(r[v * kC + c]), S, bias));
                    lo[c] = (uint32_t)w;
                    hi[c] = (uint32_t)(w >> 32) & 0xfffffu;
                    off[c] = min(__builtin_amdgcn_alignbit(hi[c], lo[c], (uint32_t)(F - 1)) & 0xfffeu, 2u * (uint32_t)last);
                }
#pragma unroll
                for (int c = 0; c < kC; ++c) off[c] = *(const uint16_t *)((const char *)s_rank + off[c]);
#pragma unroll
                for (int c = 0; c < kC; ++c) {
                    off[c] = off[c] == 0 ? dump : off[c];
                    atomicAdd((u64 *)(base + (int)off[c]), ((u64)hi[c] << 32) | lo[c]);
                }
            });
            sync<T>();
            // suffix sums over the points' words: thread t owns the t-th chunk from
            // the top
            u64 *top = lat + kHistDump + LS.pad + LS.n - t * LS.per - 1;
            u64 tot = 0;
            int z = 0;
            for (; z + 8 <= LS.per; z += 8) {
                u64 w[8];
#pragma unroll
                for (int y = 0; y < 8; ++y) w[y] = top[-z - y];
#pragma unroll
                for (int y = 0; y < 8; ++y) tot += w[y];
            }
#pragma unroll 1
            for (; z < LS.per; ++z) tot += top[-z];
            const u64 incl = wave_prefix_sum(tot);
            u64 run = incl - tot;
            if constexpr (kWaves > 1) {
                if (lane == kWave - 1) s_scan[wid] = incl;
                __syncthreads();
#pragma unroll
                for (int w = 0; w < kWaves - 1; ++w) run += w < wid ? s_scan[w] : 0ull;
            }
            z = 0;
            for (; z + 8 <= LS.per; z += 8) {
                u64 w[8];
#pragma unroll
                for (int y = 0; y < 8; ++y) w[y] = top[-z - y];
#pragma unroll
                for (int y = 0; y < 8; ++y) {
                    run += w[y];
                    top[-z - y] = run;
                }
            }
#pragma unroll 1
            for (; z < LS.per; ++z) {
                run += top[-z];
                top[-z] = run;
            }
            sync<T>();
        } else {
            // the codes at the largest candidate and its error, an upper
            // bound of the least
            const double a_top = uni((double)cand(G - 1)), ia = uni(a_top > 0.0 ? recip(a_top) : 0.0);
            for (int b = t; b < G + 1 + (kMode == kHistLinear ? kWave : 0); b += T) {
                ha[b] = 0;
                if constexpr (kMode != kHistLinear) hb[b] = 0;
            }
            if constexpr (kMode == kHistGrid) {
                for (int g = t; g < G; g += T) s_a[g] = cand(g);
                if (t == 0) s_a[G] = INFINITY;
            }
            auto top_code = [&](double x) { return fmin(rint(x * ia), Md); };
            // (linear: E_top is about d a_top^2 / 12, so past d = 6 M^2 less
            // than a third of the candidates could be left out)
            const bool prune = kMode != kHistLinear || d < 6 * M * M;
            if (prune) {
                each_slot([&](int v, int, int) {
#pragma unroll
                    for (int c = 0; c < kC; ++c) {
                        const double x = fabs(r[v * kC + c]), q = top_code(x);
                        A0 = fma(x, q, A0);
                        B0 = fma(q, q, B0);
                    }
                });
                sum2(A0, B0);   // its barrier publishes the cleared bins
            }
            if (kWaves == 1 || !prune) sync<T>();
            const double t2 = 2.0 * a_top * A0, t3 = a_top * a_top * B0;
            const double E_top = (R - t2) + t3 + 0x1p-40 * (R + t2 + t3);
            // c_g < cut loses to the top candidate (margins: 2^-23 of the
            // candidates' and the maximum's roundings); the top one stays
            const float root = __builtin_amdgcn_sqrtf((float)(E_top * inv_m * inv_m)) * 1.000001f;
            const float cut = prune && m >= 0x1p-100f && a_top > 0.0 ? (1.0f - root) - 0x1p-19f : 0.0f;
            if constexpr (kMode == kHistGrid) {
                int lo = 0, hi = G - 1;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (s_c[mid] < cut) lo = mid + 1;
                    else hi = mid;
                }
                g_lo = __builtin_amdgcn_readfirstlane(lo);
            } else {
                g_lo = __builtin_amdgcn_readfirstlane(min(max((int)(cut * (float)G) - 1, 0), G - 1));
            }
            // fixed point: sums of up to M d values x <= m (1 + 2^-24)
            const int ex = __builtin_amdgcn_readfirstlane(__builtin_amdgcn_frexp_exp((double)m));   // m < 2^ex
            const int lg = 64 - __clzll((u64)M * (u64)d);
            int sh = 51 - (ex + 1);
            if constexpr (kMode == kHistLinear) {
                // beside them the counts: sums of (2k+1) <= d M^2
                cs = min(63 - (64 - __clzll((u64)d * (u64)(M * M))), kLatShift);
                sh = cs - (ex + 1) - lg;
            } else {
                sh = min(sh, 62 - (ex + 1) - lg);
            }
            unit = uni(ldexp(1.0, -sh));
            slackA = 0.51 * Md * (double)d * unit + 0x1p-38 * A0;
            const double scale = uni(ldexp(1.0, sh));
            if constexpr (kMode == kHistLinear) {
                // n_jk = floor(x G M / (m (k + 1/2))): the low word of one fma
                // (rounded after the subtraction of 1/2; below 1/2 it reads
                // -1).  A level every candidate passes (n >= G: most elements'
                // low levels) goes to one of 64 bins from G on, by lane.
                miss = 0x1.04p-23 * sumx + sub;
                A0 = 0.0;
                B0 = 0.0;
                const double gm = uni(GM * inv_m);
                const int most = G + lane;
                each_slot([&](int v, int, int) {
#pragma unroll
                    for (int c = 0; c < kC; ++c) {
                        const double x = fabs(r[v * kC + c]);
                        const double y = x * gm;
                        const u64 w = (u64)__double_as_longlong(fma(x, scale, 0x1p52));
                        const uint32_t lo = (uint32_t)w, hi = (uint32_t)(w >> 32) & 0xfffffu;
#pragma unroll
                        for (int kk = 0; kk < kM; ++kk) {
                            const double t0 = fma(y, 1.0 / ((double)kk + 0.5), 0x1p52 - 0.5);
                            int nn = (int)(uint32_t)(u64)__double_as_longlong(t0);
                            if (nn > g_lo) {
                                nn = min(nn, most);
                                const uint32_t h = hi + ((uint32_t)(2 * kk + 1) << (cs - 32));
                                atomicAdd(&ha[nn], ((u64)h << 32) | lo);
                            }
                        }
                    }
                });
            } else {
                miss = (kMode == kHistWide ? 0x1p-21 : 0x1p-45) * sumx + sub;
                double ia2 = ia;   // grid: opaque (kept from above, the codes spilled 24 registers of 168 at EPT 36)
                if constexpr (kMode == kHistGrid) asm volatile("" : "+s"(ia2));
                const double ym = uni((kMode == kHistWide ? GM : (double)kHistTable * Md) * inv_m);
                each_slot([&](int v, int, int) {
#pragma unroll
                    for (int c = 0; c < kC; ++c) {
                        const double x = fabs(r[v * kC + c]);
                        const u64 X = (u64)__double_as_longlong(fma(x, scale, 0x1p52)) & ((1ull << 52) - 1);
                        int kk = (int)fmin(rint(x * ia2), Md);   // top_code: the levels below are in A0, B0
                        const float y = (float)(x * ym);
                        for (; kk < M; ++kk) {
                            const float h = (float)kk + 0.5f;
                            int nn;
                            if constexpr (kMode == kHistWide) {
                                // within relative 6 2^-24 (x, rcp's ulp, the
                                // product); at the boundary n = G or past it
                                // the level still counts for every candidate
                                nn = (int)(fminf(y * __builtin_amdgcn_rcpf(h), (float)G));
                            } else {
                                const int e = (int)fminf(y * __builtin_amdgcn_rcpf(h), (float)kHistTable);
                                nn = s_tab[e];
                                while (nn < G && fma((double)h, (double)s_a[nn], -x) < 0.0) ++nn;
                            }
                            if (nn <= g_lo) break;   // higher levels have higher boundaries
                            atomicAdd(&ha[nn], X);
                            atomicAdd(&hb[nn], (uint32_t)(2 * kk + 1));
                        }
                    }
                });
            }
            sync<T>();
        }

        // ---- candidate errors and lower bounds, argmin (for the lattice from
        // the suffix sums in LDS, candidate by candidate; otherwise lane l
        // owns the l-th chunk of the candidates kept, from the top).  The
        // fp64 operations err by 2^-50 (R + 2 a A + a^2 B) <= 2^-46 R for
        // every candidate with E <= R (a ||q|| <= 2 ||r|| there), and less
        // than that share of E for the others.
        const double c2 = uni(2.0 * (slackA + miss)), tiny = 0x1p-44 * R;
        const u64 low = (1ull << cs) - 1;
        auto fixed = [&](u64 A) {   // an integer below 2^52 as a double
            return __longlong_as_double((long long)(A | (0x433ull << 52))) - 0x1p52;
        };
        auto sweep = [&](auto &&f) {   // f(g, e, lower bound) over this thread's candidates
            if constexpr (kMode == kHistLattice) {
                const char *base = (const char *)(lat + kHistDump + LS.pad - 1);
#pragma unroll 1
                for (int g = t; g < G; g += kWave) {
                    u64 A = 0;
                    uint32_t Bc = 0;
#pragma unroll
                    for (int k0 = 0; k0 < kM; k0 += 8) {   // eight reads in flight
                        u64 w[8];
                        uint32_t off[8];
#pragma unroll
                        for (int z = 0; z < 8; ++z)
                            if (k0 + z < kM) off[z] = s_rank[(2 * (k0 + z) + 1) * (g + 1)];
#pragma unroll
                        for (int z = 0; z < 8; ++z)
                            if (k0 + z < kM) w[z] = *(const u64 *)(base + off[z]);
#pragma unroll
                        for (int z = 0; z < 8; ++z) {
                            if (k0 + z < kM) {
                                A += w[z];
                                Bc += (uint32_t)(2 * (k0 + z) + 1) * (uint32_t)(w[z] >> kLatShift);
                            }
                        }
                    }
                    const double a = (double)cand(g), aA = a * (fixed(A & low) * unit);
                    double e = fma(a * a, (double)Bc, fma(-2.0, aA, R));
                    if (a == 0.0) e = INFINITY;
                    f(g, e, fma(-a, c2, e));
                }
            } else {
                const int per = (G - g_lo + kWave - 1) / kWave;
                const int g1 = G - lane * per, g0 = max(g1 - per, g_lo);
                u64 la = 0;
                uint32_t lb = 0;
#pragma unroll 1
                for (int g = g0; g < g1; ++g) {
                    la += ha[g + 1];
                    if constexpr (kMode != kHistLinear) lb += hb[g + 1];
                }
                u64 A = wave_prefix_sum(la) - la;   // exclusive
                uint32_t Bq = 0;
                if constexpr (kMode != kHistLinear) Bq = wave_prefix_sum(lb) - lb;
                else A += full;
#pragma unroll 1
                for (int g = g1 - 1; g >= g0; --g) {
                    A += ha[g + 1];
                    double Ad, Bd;
                    if constexpr (kMode == kHistLinear) {
                        Ad = fixed(A & low) * unit;
                        Bd = (double)(uint32_t)(A >> cs);
                    } else {
                        Bq += hb[g + 1];
                        Ad = fma((double)A, unit, A0);
                        Bd = (double)Bq + B0;
                    }
                    const double a = (double)cand(g);
                    double e = fma(a * a, Bd, fma(-2.0, a * Ad, R));
                    if (a == 0.0) e = INFINITY;
                    f(g, e, fma(-a, c2, e));
                }
            }
        };
        int gstar = -1;
        bool other = false;   // uniform: a second candidate may be the best
        double thr = INFINITY;
        if (wid == 0) {   // one wavefront evaluates the candidates, the others wait
            if (t == 0) s_nfin = 0;
            if constexpr (kMode == kHistLinear) {   // the lanes' own bins
                const u64 mine = lane > 0 ? ha[G + lane] : 0;   // bin G is the last candidate's
                const u64 sum = wave_prefix_sum(mine);
                full = ((u64)(uint32_t)__builtin_amdgcn_readlane((int)(sum >> 32), 63) << 32) |
                       (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)sum, 63);
            }
            Lead L{INFINITY, INFINITY, INFINITY, 0x7fffffff};
            sweep([&](int g, double e, double lb) { lead_add(L, e, lb, g); });
            const double emin = wave_reduce(L.e, MinOp());
            // the smallest g among the lanes at the minimum
            int gm = L.e == emin ? L.g : 0x7fffffff;
            const u64 at = __builtin_amdgcn_ballot_w64(L.e == emin);
            gm = __builtin_popcountll(at) == 1 ? readlane(gm, (int)__builtin_ctzll(at)) : wave_reduce(gm, MinOp());
            gm = __builtin_amdgcn_readfirstlane(gm);
            // the other candidates' least lower bound
            const double rest = L.g == gm ? L.rest : fmin(L.rest, L.lb);
            gstar = emin == INFINITY ? -1 : gm;
            if (gstar >= 0) thr = fma((double)cand(gstar), c2, uni(emin)) + tiny;
            other = gstar >= 0 && __builtin_amdgcn_ballot_w64(rest <= thr) != 0;
        }
        // the finalists' list (rarely more than the best one)
        auto list_finalists = [&]() {
            sweep([&](int g, double, double e) {
                if (e <= thr) {
                    const int at = atomicAdd(&s_nfin, 1);
                    if (at < kMaxFinalists) s_fin[at] = g;
                }
            });
        };
        if (other && wid == 0) list_finalists();
        if constexpr (kWaves > 1) {
            if (t == 0) {
                s_pick[0] = gstar;
                s_pick[1] = other ? 1 : 0;
            }
            __syncthreads();
            gstar = s_pick[0];
            other = s_pick[1] != 0;
        } else if (other) {
            sync<T>();
        }
        if (other) {
            // direct fp64 evaluation (Eq. (9) written out); a list that
            // overflowed stands for every candidate kept
            const int nf = s_nfin;
            const bool all = nf > kMaxFinalists;
            ArgMin best{INFINITY, 0x7fffffff};
            for (int f = all ? g_lo : 0; f < (all ? G : nf); ++f) {
                const int g = all ? f : s_fin[f];
                const double a = uni((double)cand(g));
                if (a == 0.0) continue;
                const double ia = uni(recip(a));
                double part[kPart] = {};
                each_slot([&](int v, int, int) {
#pragma unroll
                    for (int c = 0; c < kC; ++c) {
                        const double x = r[v * kC + c], q = rint(quotient(x, a, ia));
                        const double e = fma(-a, fmin(fmax(q, -Md), Md), x);
                        part[v % kPart] = fma(e, e, part[v % kPart]);
                    }
                });
                const double E = total(part);
                if (E < best.e || (E == best.e && g < best.g)) best = ArgMin{E, g};
            }
            gstar = best.g;
        }
        if (gstar < 0) {   // every candidate scale is zero
            n = i;
            break;
        }
        apend = uni(cand(gstar));
        if (t == 0) Ly.scales[k * P + i] = apend;
    }

    // the channel's row of the output error's D, outside calibration steps:
    // the residual after its n points in fp32, zero past d up to the row's
    // nkb 32-k chunks (D holds tiles of 128 rows by 32 k, row-major inside)
    if (Ly.dres && !stepping) {
        const int nkb = (d + 31) / 32;
        float *drow = Ly.dres + (k / 128) * nkb * 4096 + (k % 128) * 32;
        if (t == 0) Ly.dmax[k] = __float_as_uint(m);   // of the residual after the last point
#pragma unroll
        for (int v = 0; v < kSlots; ++v) {
            const int j0 = kC * (t + T * v);
            if (j0 >= nkb * 32) continue;
            float *p = drow + (j0 / 32) * 4096 + j0 % 32;
            if constexpr (kC == 4)
                *(float4 *)p = make_float4((float)r[v * kC], (float)r[v * kC + kC / 4], (float)r[v * kC + kC / 2],
                                           (float)r[v * kC + kC - 1]);
            else
                *p = (float)r[v];
        }
    }
    if (t == 0) Ly.counts[k] = n;
    if (more) {
        if (t == 0) Ly.list[atomicAdd(Ly.nlist + s0, 1)] = (int32_t)k;
        return;
    }
    for (int q = n + t; q < P; q += T) {
        Ly.scales[k * P + q] = 0.0f;
        if (Ly.err) Ly.err[k * P + q] = 0.0f;
        if (Ly.xerr) Ly.xerr[k * P + q] = 0.0f;
    }
    // code rows n .. P - 1: one contiguous byte range, in 16-byte stores
    // between its unaligned head and tail
    int8_t *z0 = qk + (int64_t)n * d, *z1 = qk + (int64_t)P * d;
    int8_t *a0 = (int8_t *)(((uintptr_t)z0 + 15) & ~(uintptr_t)15);
    int8_t *a1 = (int8_t *)((uintptr_t)z1 & ~(uintptr_t)15);
    if (a0 >= a1) {
        for (int8_t *p = z0 + t; p < z1; p += T) *p = 0;
    } else {
        if (z0 + t < a0) z0[t] = 0;   // head < 16 <= T bytes
        if (a1 + t < z1) a1[t] = 0;   // tail < 16 bytes
        for (int64_t v = t; v < (a1 - a0) / 16; v += T) ((uint4 *)a0)[v] = make_uint4(0, 0, 0, 0);
    }
}

template <int T, int EPT, int kMode, int kM>
hipError_t launch_hist_t(const HistBatch &b, int64_t channels, hipStream_t s)
{
    if (kM > 0 && b.M != kM) return hipErrorInvalidValue;
    auto kern = fit_hist_kernel<T, EPT, kMode, kM>;
    const size_t lds = hist_lds(kMode, T, b.M, b.G, b.points);
    if (lds > 60000) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    LaunchTimer timer(s, hist_name(T, EPT, kMode).c_str());
    hipLaunchKernelGGL(kern, dim3((unsigned)channels), dim3(T), lds, s, b);
    return hipGetLastError();
}

}  // namespace mpq
