// Compile-time FFT plans of mesh sides without a file of their own: the default shape of each pass
// (default_pass), one kernel per operation.  The sides are dealt over four files to compile in parallel.

#include "fft_kernels.h"

namespace cola {

hipError_t fft_static_sides_1(const FftLaunch& L, int n) {
    switch (n) {
        case 18: return static_default<18>(L);
        case 48: return static_default<48>(L);
        case 96: return static_default<96>(L);
        case 162: return static_default<162>(L);
        case 432: return static_default<432>(L);
        case 864: return static_default<864>(L);
        case 1296: return static_default<1296>(L);
        default: return hipErrorNotSupported;
    }
}

}  // namespace cola
