// One instantiation unit of the decode kernel with register-resident weights, compiled once per
//   -DRNNT_RES_KIND=1|2|3   ResidentKind
//   -DRNNT_RES_BF=0|1       bfloat16 mode
//   -DRNNT_RES_CLS=0|1|2    size class
// with its sample-tile variants.
#include "resident_impl.h"

#define RNNT_CAT_(a, b, c, d, e, f) a##b##c##d##e##f
#define RNNT_CAT(a, b, c, d, e, f) RNNT_CAT_(a, b, c, d, e, f)

namespace rnnt {
hipError_t RNNT_CAT(launch_resident_, RNNT_RES_KIND, _, RNNT_RES_BF, _, RNNT_RES_CLS)(const ResidentParams &p, int nmt, bool plain,
                                                                                      hipStream_t stream, hipEvent_t end)
{
    if (p.slots > 4) return launch_resident_one<RNNT_RES_KIND, RNNT_RES_BF != 0, RNNT_RES_CLS, 2, 8>(p, plain, stream, end);
    if (nmt == 2) return launch_resident_one<RNNT_RES_KIND, RNNT_RES_BF != 0, RNNT_RES_CLS, 2, 4>(p, plain, stream, end);
    if (p.slots == 1) return launch_resident_one<RNNT_RES_KIND, RNNT_RES_BF != 0, RNNT_RES_CLS, 1, 4, true>(p, plain, stream, end);
    return launch_resident_one<RNNT_RES_KIND, RNNT_RES_BF != 0, RNNT_RES_CLS, 1, 4>(p, plain, stream, end);
}
}  // namespace rnnt
