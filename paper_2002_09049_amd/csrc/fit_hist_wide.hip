// The wide mode of the histogram search (fit_hist_kernel.hpp), for every
// variant of kVariants (fit_hist.hip) that takes it.
#include "fit_hist_kernel.hpp"

namespace mpq {

hipError_t launch_hist_wide(const HistBatch &b, int T, int ept, int64_t channels, hipStream_t s)
{
    if (T == 64 && ept == 1) return launch_hist_t<64, 1, kHistWide, 0>(b, channels, s);
    if (T == 64 && ept == 2) return launch_hist_t<64, 2, kHistWide, 0>(b, channels, s);
    if (T == 64 && ept == 4) return launch_hist_t<64, 4, kHistWide, 0>(b, channels, s);
    if (T == 64 && ept == 8) return launch_hist_t<64, 8, kHistWide, 0>(b, channels, s);
    if (T == 64 && ept == 12) return launch_hist_t<64, 12, kHistWide, 0>(b, channels, s);
    if (T == 64 && ept == 20) return launch_hist_t<64, 20, kHistWide, 0>(b, channels, s);
    if (T == 128 && ept == 20) return launch_hist_t<128, 20, kHistWide, 0>(b, channels, s);
    if (T == 128 && ept == 36) return launch_hist_t<128, 36, kHistWide, 0>(b, channels, s);
    if (T == 256 && ept == 36) return launch_hist_t<256, 36, kHistWide, 0>(b, channels, s);
    if (T == 512 && ept == 32) return launch_hist_t<512, 32, kHistWide, 0>(b, channels, s);
    if (T == 512 && ept == 52) return launch_hist_t<512, 52, kHistWide, 0>(b, channels, s);
    if (T == 512 && ept == 64) return launch_hist_t<512, 64, kHistWide, 0>(b, channels, s);
    if (T == 256 && ept == 4) return launch_hist_t<256, 4, kHistWide, 0>(b, channels, s);
    if (T == 256 && ept == 8) return launch_hist_t<256, 8, kHistWide, 0>(b, channels, s);
    if (T == 256 && ept == 12) return launch_hist_t<256, 12, kHistWide, 0>(b, channels, s);
    if (T == 256 && ept == 20) return launch_hist_t<256, 20, kHistWide, 0>(b, channels, s);
    return hipErrorInvalidValue;
}

}  // namespace mpq
