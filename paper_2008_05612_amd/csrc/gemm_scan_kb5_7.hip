// Dense threshold scan, pure pair energies, chains of 5 .. 7 products (gemm_scan.h).
#include "gemm_scan.h"

namespace hpmap {

hipError_t launch_scan_kb5(const EnumJob &j, hipStream_t st)
{
    return launch_scan_kb<5, false>(j, st);
}
hipError_t launch_scan_kb6(const EnumJob &j, hipStream_t st)
{
    return launch_scan_kb<6, false>(j, st);
}
hipError_t launch_scan_kb7(const EnumJob &j, hipStream_t st)
{
    return launch_scan_kb<7, false>(j, st);
}

}  // namespace hpmap
