// Dense threshold scan, pure pair energies, chains of 1 .. 4 products (gemm_scan.h).
#include "gemm_scan.h"

namespace hpmap {

hipError_t launch_scan_kb1(const EnumJob &j, hipStream_t st)
{
    return launch_scan_kb<1, false>(j, st);
}
hipError_t launch_scan_kb2(const EnumJob &j, hipStream_t st)
{
    return launch_scan_kb<2, false>(j, st);
}
hipError_t launch_scan_kb3(const EnumJob &j, hipStream_t st)
{
    return launch_scan_kb<3, false>(j, st);
}
hipError_t launch_scan_kb4(const EnumJob &j, hipStream_t st)
{
    return launch_scan_kb<4, false>(j, st);
}

}  // namespace hpmap
