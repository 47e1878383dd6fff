// rom_scan_f32.hip -- FP32 single-ordinate instantiations of the row-scan sweep kernel (step scheme,
// isotropic source).
#include "rom_scan.h"

namespace rom {

#define ROM_SCAN_CASE(G_, C_)                                                                  \
    if (G == G_ && C == C_)                                                                    \
        return inf ? launch_scan_t<float, G_, C_, kScanWaves, 0, false, true>(a, ntasks, s)    \
                   : launch_scan_t<float, G_, C_, kScanWaves, 0, false, false>(a, ntasks, s);

hipError_t launch_scan_f32(const ScanArgs& a, int ntasks, int G, int C, bool inf, hipStream_t s)
{
    ROM_SCAN_CASE(64, 1)
    ROM_SCAN_CASE(64, 2)
    ROM_SCAN_CASE(64, 3)
    ROM_SCAN_CASE(64, 4)
    ROM_SCAN_CASE(64, 5)
    ROM_SCAN_CASE(64, 6)
    ROM_SCAN_CASE(64, 8)
    ROM_SCAN_CASE(64, 12)
    ROM_SCAN_CASE(64, 16)
    ROM_SCAN_CASE(16, 4)
    return hipErrorInvalidValue;
}

}  // namespace rom
