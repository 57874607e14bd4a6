// Host side of the resident decode kernel: which models fit it.  No device code and no HIP calls.
#pragma once
#include <algorithm>

#include "resident.h"
#include "solo.h"

namespace rnnt {

// The plan for a model, kind == kResidentNone when it does not fit: one or two LSTM layers of at
// most 640 units, a joint layer of at most 640, an output layer of at most 32 columns per
// work-group and a tail of one more.
inline ResidentPlan plan_resident(int H, int J, int L, int NOUT, bool bf, int n_cu)
{
    ResidentPlan pl{};
    if (L > 2 || n_cu % 32 != 0) return pl;
    const int n_xcd = n_cu / 32;
    const int kind = L == 1 ? kResident1 : (bf ? kResident2 : kResident2Pair);
    if (kind == kResident2Pair && res_chain_xcds(n_xcd) < 1) return pl;
    for (int cls = kResClasses - 1; cls >= 0; --cls) {
        const int ts = res_team(cls);
        const int units = (H + ts - 1) / ts, jg = (J / 4 + ts - 1) / ts;
        const int nout_m = std::min(NOUT, 32 * ts), n_tail = NOUT - nout_m;
        if (H > res_width(cls) || J > res_width(cls) || units > kResUnits || jg > 5 || n_tail > ts) continue;
        pl.kind = kind; pl.cls = cls; pl.bf = bf; pl.n_xcd = n_xcd;
        pl.n_teams = (kind == kResident2Pair ? res_chain_xcds(n_xcd) : n_xcd) * (32 / ts);
        pl.units = units; pl.jgroups = jg; pl.nout_m = nout_m; pl.n_tail = n_tail;
        // Models that a work-group decodes alone: hand-overs inside a team are most of their steps (solo.hip).
        pl.solo = solo_holds(H, J, L, NOUT, bf);
        if (pl.solo) pl.n_teams = n_cu;
        return pl;
    }
    return pl;
}

}  // namespace rnnt
