// Compile-time FFT plans of mesh sides without a file of their own: the default shape of each pass
// (default_pass), one kernel per operation.  The sides are dealt over four files to compile in parallel.

#include "fft_kernels.h"

namespace cola {

hipError_t fft_static_sides_3(const FftLaunch& L, int n) {
    switch (n) {
        case 32: return static_default<32>(L);
        case 64: return static_default<64>(L);
        case 128: return static_default<128>(L);
        case 216: return static_default<216>(L);
        case 576: return static_default<576>(L);
        case 1024: return static_default<1024>(L);
        default: return hipErrorNotSupported;
    }
}

}  // namespace cola
