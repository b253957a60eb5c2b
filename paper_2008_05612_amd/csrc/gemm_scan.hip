// Dispatch of the dense threshold scan by chain length.  The kernels
// (gemm_scan.h) are instantiated in gemm_scan_kb*.hip and gemm_scan_un*.hip.
#include "hp_internal.h"
#include "kernels.h"

namespace hpmap {

#define HP_SCAN(name) hipError_t launch_scan_##name(const EnumJob &j, hipStream_t st);
HP_SCAN(kb1) HP_SCAN(kb2) HP_SCAN(kb3) HP_SCAN(kb4) HP_SCAN(kb5)
HP_SCAN(kb6) HP_SCAN(kb7) HP_SCAN(kb8) HP_SCAN(kb9) HP_SCAN(kb10)
HP_SCAN(un1) HP_SCAN(un2) HP_SCAN(un3) HP_SCAN(un4) HP_SCAN(un5) HP_SCAN(un6)
#undef HP_SCAN

hipError_t launch_scan(const EnumJob &j, hipStream_t st)
{
    using Launch = hipError_t (*)(const EnumJob &, hipStream_t);
    static const Launch pure[] = {nullptr, launch_scan_kb1, launch_scan_kb2, launch_scan_kb3,
                                  launch_scan_kb4, launch_scan_kb5, launch_scan_kb6, launch_scan_kb7,
                                  launch_scan_kb8, launch_scan_kb9, launch_scan_kb10};
    static const Launch un[] = {nullptr, launch_scan_un1, launch_scan_un2, launch_scan_un3,
                                launch_scan_un4, launch_scan_un5, launch_scan_un6};
    const int kb = j.scan_kb;
    if (kb < 1 || kb > (j.U ? 6 : 10))
        return hipErrorInvalidValue;
    return (j.U ? un : pure)[kb](j, st);
}

}  // namespace hpmap
