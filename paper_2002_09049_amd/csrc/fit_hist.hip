// Dispatch of the histogram search (fit_hist_kernel.hpp): which kernel
// variant fits channels of a length, and in which mode.
#include <stdio.h>

#include <bitset>

#include "fit_hist_kernel.hpp"

namespace mpq {

namespace {

// (threads, elements per thread, groups of four consecutive elements per
// thread) of each variant; variant v takes the channels longer than the
// capacity T * EPT of variant v - 1, up to its own.
struct Variant {
    int threads, ept;
    bool quad;
};
constexpr Variant kVariants[] = {{64, 1, false}, {64, 2, false}, {64, 4, true}, {64, 8, true},
                                 {64, 12, true}, {64, 20, true}, {128, 20, true}, {128, 36, true},
                                 {256, 36, true}, {512, 32, true}, {512, 52, true},
                                 {512, 64, true}};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);
static_assert(kVariants[kNumVariants - 1].threads * kVariants[kNumVariants - 1].ept >= kHistMaxDim,
              "the last variant covers the longest channels");

// The same channels by four wavefronts each, for calls whose channels would
// leave most SIMDs without one (hist_waves): shorter steps, the same results
// bit for bit.  Channels of more than kWideMinDim weights.
constexpr Variant kWide[] = {{256, 4, true}, {256, 8, true}, {256, 12, true}, {256, 20, true}};
constexpr int kNumWide = sizeof(kWide) / sizeof(kWide[0]);
constexpr int64_t kWideMinDim = 256;

// as the kernel takes it from the elements per thread
template <size_t kN>
constexpr bool quads_as_kernel(const Variant (&v)[kN])
{
    for (const Variant &x : v)
        if (x.quad != (x.ept >= 4) || (x.quad && x.ept % 4 != 0)) return false;
    return true;
}
static_assert(quads_as_kernel(kVariants) && quads_as_kernel(kWide), "groups of four");

// Lattice buckets of LDS at most (8 bytes each).
constexpr int kLatMaxBuckets = 7680;

}  // namespace

size_t fit_hist_lds(int G)
{
    return hist_lds(kHistGrid, 64, 127, G, 0);   // the mode that needs the most per candidate
}

bool fit_hist_supports(int64_t d) { return d >= 1 && d <= kHistMaxDim; }

// the short-channel variants (fit_small.hip), one per length 1 ..
// kSmallMaxDim, follow the histogram ones, and the wide ones follow those
constexpr int kSmallVariant = kNumVariants;
constexpr int kWideVariant = kSmallVariant + (int)kSmallMaxDim;

int hist_variant_count() { return kWideVariant + kNumWide; }

int hist_variant(int64_t d, bool wide)
{
    if (d >= 1 && d <= kSmallMaxDim) return kSmallVariant + (int)d - 1;
    if (wide && d > kWideMinDim)
        for (int v = 0; v < kNumWide; ++v)
            if (d <= (int64_t)kWide[v].threads * kWide[v].ept) return kWideVariant + v;
    int v = 0;
    while (v + 1 < kNumVariants && d > (int64_t)kVariants[v].threads * kVariants[v].ept) ++v;
    return v;
}

int hist_waves(int64_t d) { return d <= kSmallMaxDim ? 1 : kVariants[hist_variant(d, false)].threads / 64; }

namespace {

Variant variant_of(int v) { return v >= kWideVariant ? kWide[v - kWideVariant] : kVariants[v]; }

// Lattice mode where its pass over (2M-1) G buckets (about 10 instructions
// per bucket) costs less than the levels of the linear one (about 11 per
// element and level, up to seven), by the variant's longest channels.
int mode_of(int variant, int M, int G, bool default_grid)
{
    if (!default_grid) return kHistGrid;
    const int64_t n = (int64_t)(2 * M - 1) * G, cap = (int64_t)variant_of(variant).threads * variant_of(variant).ept;
    if (M <= 15 && n <= kLatMaxBuckets && cap >= 1024 && 2 * cap * (M < 7 ? M : 7) >= 3 * n) return kHistLattice;
    return M <= 7 ? kHistLinear : kHistWide;
}

// The distinct products (2k+1)(g+1), k < M, g < G.
int lattice_points(int M, int G)
{
    std::bitset<2 * kLatMaxBuckets> seen;
    for (int k = 0; k < M; ++k)
        for (int g = 1; g <= G; ++g) seen.set((size_t)(2 * k + 1) * g);
    return (int)seen.count();
}

}  // namespace

std::string hist_name(int T, int EPT, int mode)
{
    static const char *const names[] = {"lattice", "linear", "wide", "grid"};
    char name[64];
    snprintf(name, sizeof name, "fit_hist_kernel<%d,%d,%s>", T, EPT, names[mode]);
    return name;
}

std::string hist_kernel_name(int64_t d, int M, int G, bool default_grid)
{
    const int v = hist_variant(d, false);
    if (v >= kSmallVariant) return fit_small_name((int)d);
    return hist_name(kVariants[v].threads, kVariants[v].ept, mode_of(v, M, G, default_grid));
}

namespace {
__global__ void zero_i32_kernel(int32_t *p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}
}  // namespace

hipError_t launch_zero_i32(int32_t *p, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    if (n > (int64_t)256 * 0x7fffffff) return hipErrorInvalidValue;
    LaunchTimer timer(s, "zero_i32_kernel");
    hipLaunchKernelGGL(zero_i32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_fit_hist(const HistBatch &batch, int variant, int64_t channels, hipStream_t s)
{
    HistBatch b = batch;
    if (variant >= kSmallVariant && variant < kSmallVariant + kSmallMaxDim)
        return launch_fit_small(b, variant - kSmallVariant + 1, channels, s);
    if (variant < 0 || variant >= hist_variant_count()) return hipErrorInvalidValue;
    const int T = variant_of(variant).threads, ept = variant_of(variant).ept;
    switch (mode_of(variant, b.M, b.G, !b.grid)) {
    case kHistLattice:
        b.points = lattice_points(b.M, b.G);
        return b.M == 1   ? launch_hist_lattice1(b, T, ept, channels, s)
               : b.M == 3 ? launch_hist_lattice3(b, T, ept, channels, s)
               : b.M == 7 ? launch_hist_lattice7(b, T, ept, channels, s)
                          : launch_hist_lattice15(b, T, ept, channels, s);
    case kHistLinear:
        return b.M == 1   ? launch_hist_linear1(b, T, ept, channels, s)
               : b.M == 3 ? launch_hist_linear3(b, T, ept, channels, s)
                          : launch_hist_linear7(b, T, ept, channels, s);
    case kHistWide: return launch_hist_wide(b, T, ept, channels, s);
    default: return launch_hist_grid(b, T, ept, channels, s);
    }
}

}  // namespace mpq
