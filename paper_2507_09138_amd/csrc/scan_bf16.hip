// List-scan kernel instantiations for HR_BF16 storage (all supported dimensions).
#include "scan_kernel.h"

namespace hr {
hipError_t launch_scan_bf16(int d, const ScanArgs& a, int grid, size_t lds, hipStream_t s)
{
    return launch_scan_dtype<HR_BF16>(d, a, grid, lds, s);
}
hipError_t launch_seed_bf16(int d, const SeedArgs& a, const BucketArgs* group, hipStream_t s) { return launch_seed_dtype<HR_BF16>(d, a, group, s); }
}  // namespace hr
