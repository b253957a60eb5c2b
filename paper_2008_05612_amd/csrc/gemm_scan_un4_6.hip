// Dense threshold scan, two-letter tables, chains of 4 .. 6 products (gemm_scan.h).
#include "gemm_scan.h"

namespace hpmap {

hipError_t launch_scan_un4(const EnumJob &j, hipStream_t st)
{
    return launch_scan_kb<4, true>(j, st);
}
hipError_t launch_scan_un5(const EnumJob &j, hipStream_t st)
{
    return launch_scan_kb<5, true>(j, st);
}
hipError_t launch_scan_un6(const EnumJob &j, hipStream_t st)
{
    return launch_scan_kb<6, true>(j, st);
}

}  // namespace hpmap
