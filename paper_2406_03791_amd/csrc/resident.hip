// Choice of the resident decode kernel's instance (resident_impl.h, resident_inst.hip).
#include "engine.h"
#include "resident.h"

namespace rnnt {

typedef hipError_t (*ResidentLaunch)(const ResidentParams &, int, bool, hipStream_t, hipEvent_t);
#define RNNT_DECLARE(k, bf) \
    hipError_t launch_resident_##k##_##bf##_0(const ResidentParams &, int, bool, hipStream_t, hipEvent_t); \
    hipError_t launch_resident_##k##_##bf##_1(const ResidentParams &, int, bool, hipStream_t, hipEvent_t); \
    hipError_t launch_resident_##k##_##bf##_2(const ResidentParams &, int, bool, hipStream_t, hipEvent_t); \
    static const ResidentLaunch table_##k##_##bf[kResClasses] = {launch_resident_##k##_##bf##_0, launch_resident_##k##_##bf##_1, \
                                                                launch_resident_##k##_##bf##_2};
RNNT_DECLARE(1, 0)
RNNT_DECLARE(1, 1)
RNNT_DECLARE(2, 1)
RNNT_DECLARE(3, 0)
#undef RNNT_DECLARE

hipError_t launch_resident(const ResidentParams &p, int nmt, bool plain, hipStream_t stream, hipEvent_t end)
{
    // what the kernel's buffers are laid out for
    if (nmt < 1 || nmt > 2 || p.slots < 1 || p.slots > (nmt == 1 ? 2 : kResRows) ||
        p.pl.cls < 0 || p.pl.cls >= kResClasses || (p.B + p.pl.n_teams - 1) / p.pl.n_teams > kResList)
        return hipErrorInvalidValue;
    switch (p.pl.kind) {
    case kResident1: return (p.pl.bf ? table_1_1 : table_1_0)[p.pl.cls](p, nmt, plain, stream, end);
    case kResident2: return table_2_1[p.pl.cls](p, nmt, plain, stream, end);
    case kResident2Pair: return table_3_0[p.pl.cls](p, nmt, plain, stream, end);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace rnnt
