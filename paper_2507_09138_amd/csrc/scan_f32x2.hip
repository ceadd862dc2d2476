// List-scan kernel instantiations for float32 rows that are split in LDS (all supported dimensions).
#include "scan_kernel.h"

namespace hr {
hipError_t launch_scan_f32x2(int d, const ScanArgs& a, int grid, size_t lds, hipStream_t s)
{
    return launch_scan_dtype<HR_F32X2>(d, a, grid, lds, s);
}
}  // namespace hr
