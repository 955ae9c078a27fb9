// Compile-time FFT plans of mesh sides without a file of their own: the default shape of each pass
// (default_pass), one kernel per operation.  The sides are dealt over four files to compile in parallel.

#include "fft_kernels.h"

namespace cola {

hipError_t fft_static_sides_0(const FftLaunch& L, int n) {
    switch (n) {
        case 16: return static_default<16>(L);
        case 36: return static_default<36>(L);
        case 72: return static_default<72>(L);
        case 144: return static_default<144>(L);
        case 324: return static_default<324>(L);
        case 648: return static_default<648>(L);
        case 1152: return static_default<1152>(L);
        default: return hipErrorNotSupported;
    }
}

}  // namespace cola
