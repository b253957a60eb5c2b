// Dense threshold scan, pure pair energies, chains of 8 .. 10 products (gemm_scan.h).
#include "gemm_scan.h"

namespace hpmap {

hipError_t launch_scan_kb8(const EnumJob &j, hipStream_t st)
{
    return launch_scan_kb<8, false>(j, st);
}
hipError_t launch_scan_kb9(const EnumJob &j, hipStream_t st)
{
    return launch_scan_kb<9, false>(j, st);
}
hipError_t launch_scan_kb10(const EnumJob &j, hipStream_t st)
{
    return launch_scan_kb<10, false>(j, st);
}

}  // namespace hpmap
