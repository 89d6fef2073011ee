// The paper grid's search (paper_search.hpp, the kernels' own source) on the
// CPU: a workgroup's kT threads one after the other, each run again from the
// start once the value of the next reduction over all of them is known.
#include <math.h>

#include <algorithm>
#include <vector>

#define __device__
#define __forceinline__ inline

namespace {

struct {
    int x;
} threadIdx;

using std::max;
using std::min;

}  // namespace

namespace mpq {

namespace {

struct MinOp {
    double operator()(double a, double b) const { return b < a ? b : a; }
};

constexpr int kT = 256;
std::vector<double> g_known;   // the results of the reductions so far
size_t g_at;                   // the reductions this thread has passed
struct Waits {
    double v;
};

template <int kThreads, class Op>
double block_reduce(double v, Op, double *)
{
    if (g_at == g_known.size()) throw Waits{v};
    return g_known[g_at++];
}

}  // namespace

}  // namespace mpq

#include "paper_search.hpp"

namespace mpq {

namespace {

template <int kThreads>
Best block_best(Best v, double *, long long *)   // joined by the caller
{
    return v;
}

}  // namespace

}  // namespace mpq

// The chosen grid point of residual r [d] on g gamma, g = 1 .. count; 0 when
// there is none.  Its error in *E.
extern "C" long long paper_search_host(const double *r, int d, int M, double gamma, long long count, double *E)
{
    using namespace mpq;
    int dpad = 1;
    while (dpad < d) dpad <<= 1;
    std::vector<double> s(dpad, -1.0), S(d + 1, 0.0);
    double R = 0.0;
    for (int j = 0; j < d; ++j) {
        s[j] = fabs(r[j]);
        R += r[j] * r[j];
    }
    std::sort(s.begin(), s.begin() + d, [](double a, double b) { return a > b; });
    for (int j = 0; j < d; ++j) S[j + 1] = S[j] + s[j];
    g_known.clear();
    for (;;) {
        Best best{INFINITY, 0x7fffffffffffffffLL};
        double v = INFINITY;
        bool waits = false;
        for (int t = 0; t < kT; ++t) {
            threadIdx.x = t;
            g_at = 0;
            try {
                best = better(best, paper_search<kT>(s.data(), S.data(), d, dpad, M, R, gamma, count, nullptr, nullptr));
            } catch (const Waits &w) {
                waits = true;
                v = MinOp()(v, w.v);
            }
        }
        if (!waits) {
            *E = best.e;
            return best.e == INFINITY ? 0 : best.g;
        }
        g_known.push_back(v);
    }
}
