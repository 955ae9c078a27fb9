// Compile-time FFT plans of mesh sides without a file of their own: the default shape of each pass
// (default_pass), one kernel per operation.  The sides are dealt over four files to compile in parallel.

#include "fft_kernels.h"

namespace cola {

hipError_t fft_static_sides_2(const FftLaunch& L, int n) {
    switch (n) {
        case 24: return static_default<24>(L);
        case 54: return static_default<54>(L);
        case 108: return static_default<108>(L);
        case 192: return static_default<192>(L);
        case 486: return static_default<486>(L);
        case 972: return static_default<972>(L);
        default: return hipErrorNotSupported;
    }
}

}  // namespace cola
