// rom_scan_lin_f32.hip -- FP32 row-scan sweeps of the linear kernel (both schemes) and diamond-difference
// ones with an isotropic source.
#include "rom_scan.h"

namespace rom {

#define ROM_SCAN_CASE(G_, C_, W_)                                                                   \
    if (G == G_ && C == C_ && W == W_) {                                                            \
        if (mom != 4) return launch_scan_t<float, G_, C_, W_, 0, true>(a, ntasks, inf, s);            \
        return dd ? launch_scan_t<float, G_, C_, W_, 1, true>(a, ntasks, inf, s)                      \
                  : launch_scan_t<float, G_, C_, W_, 1, false>(a, ntasks, inf, s);                    \
    }

hipError_t launch_scan_lin_f32(const ScanArgs& a, int ntasks, int W, int G, int C, int mom, bool dd, bool inf, hipStream_t s)
{
    ROM_SCAN_CASE(16, 4, 1)
    ROM_SCAN_CASE(16, 4, 4)
    ROM_SCAN_CASE(16, 8, 1)
    ROM_SCAN_CASE(16, 8, 4)
    ROM_SCAN_CASE(64, 2, 4)
    ROM_SCAN_CASE(64, 4, 4)
    ROM_SCAN_CASE(64, 8, 4)
    return hipErrorInvalidValue;
}

}  // namespace rom
