// rom_scan_ang_f64.hip -- FP64 row-scan sweeps with per-ordinate sources (dense scattering kernels).
#include "rom_scan.h"

namespace rom {

#define ROM_SCAN_CASE(G_, C_) \
    if (G == G_ && C == C_) return launch_scan_t<double, G_, C_, 4, 2, false>(a, ntasks, inf, s);

hipError_t launch_scan_ang_f64(const ScanArgs& a, int ntasks, int G, int C, bool inf, hipStream_t s)
{
    ROM_SCAN_CASE(16, 4)
    ROM_SCAN_CASE(64, 1)
    ROM_SCAN_CASE(64, 2)
    ROM_SCAN_CASE(64, 3)
    ROM_SCAN_CASE(64, 4)
    ROM_SCAN_CASE(64, 6)
    ROM_SCAN_CASE(64, 8)
    return hipErrorInvalidValue;
}

}  // namespace rom
