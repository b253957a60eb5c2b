// Dense threshold scan, two-letter tables, chains of 1 .. 3 products (gemm_scan.h).
#include "gemm_scan.h"

namespace hpmap {

hipError_t launch_scan_un1(const EnumJob &j, hipStream_t st)
{
    return launch_scan_kb<1, true>(j, st);
}
hipError_t launch_scan_un2(const EnumJob &j, hipStream_t st)
{
    return launch_scan_kb<2, true>(j, st);
}
hipError_t launch_scan_un3(const EnumJob &j, hipStream_t st)
{
    return launch_scan_kb<3, true>(j, st);
}

}  // namespace hpmap
