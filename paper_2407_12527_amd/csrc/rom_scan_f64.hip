// rom_scan_f64.hip -- FP64 single-ordinate instantiations of the row-scan sweep kernel (step scheme,
// isotropic source).
#include "rom_scan.h"

namespace rom {

#define ROM_SCAN_CASE(G_, C_, W_) \
    if (G == G_ && C == C_ && W == W_) return launch_scan_t<double, G_, C_, W_, 0, false>(a, ntasks, inf, s);

hipError_t launch_scan_f64(const ScanArgs& a, int ntasks, int W, int G, int C, bool inf, hipStream_t s)
{
    ROM_SCAN_CASE(64, 1, 4)
    ROM_SCAN_CASE(64, 2, 4)
    ROM_SCAN_CASE(64, 3, 4)
    ROM_SCAN_CASE(64, 4, 4)
    ROM_SCAN_CASE(64, 6, 4)
    ROM_SCAN_CASE(64, 8, 4)
    ROM_SCAN_CASE(64, 16, 4)
    ROM_SCAN_CASE(16, 4, 1)
    ROM_SCAN_CASE(16, 4, 4)
    ROM_SCAN_CASE(16, 8, 1)
    ROM_SCAN_CASE(16, 8, 4)
    return hipErrorInvalidValue;
}

}  // namespace rom
