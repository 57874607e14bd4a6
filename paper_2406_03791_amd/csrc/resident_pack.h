// Host side of the resident decode kernel: which models fit it, and the memory of a call.  No device code and no HIP calls.
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

// The teams' exchange buffers for calls of up to B utterances.  Teams have eight rows only where every list has eight utterances (resident_rows), and their
// buffers are up to twice those of four: an engine of two layers of 640 in fp32 for one utterance keeps 11 MB of them, for 48 and more 20.
inline size_t exchange_bytes(const ResidentPlan &pl, int B)
{
    if (pl.solo) return 0;
    return (size_t)resident_buf(pl.kind, pl.bf != 0, pl.cls, B >= kResRows * pl.n_teams ? kResRows : 4).bytes * pl.n_teams;
}

// What a call of the entry point that allocates nothing is charged of RNNT_NOALLOC_SCRATCH_BYTES, for P and its workspace.  Which
// calls are refused is part of the interface, so this stays as it was when every kind had buffers of two recurrent
// vectors and one sum a unit, two-layer fp32 models five teams where they have six, and the smallest models teams as well.
inline size_t sized(size_t bytes) { return (bytes + 255) & ~(size_t)255; }
inline size_t charged_bytes(const ResidentPlan &pl, size_t p_bytes)
{
    const size_t w = res_width(pl.cls), ts = res_team(pl.cls);
    const size_t chain = kResSlots * (5 * 4 * w * 4 + kResSamples * (ts * 12 + kMaxDur * 4)), sums = 2 * kResSlots * ts * 5 * 64 * 4;
    const size_t teams = pl.solo ? pl.n_teams / res_team(pl.cls) : pl.kind == kResident2Pair ? pl.n_teams - pl.n_teams / 6 : pl.n_teams;
    return sized(p_bytes) + sized((chain + sums) * teams) + sized((size_t)pl.n_xcd * 32 * sizeof(unsigned)) +
           sized(teams * kStatStride * sizeof(long long)) + sized(sizeof(unsigned)) + sized(sizeof(int));
}
// Where it has them, every part 256-byte aligned.  Behind what is charged there is room for kScratchBeyond bytes more.
constexpr size_t kScratchBeyond = 20u << 20;
struct NoallocLayout { size_t P, xbuf, form, stats, abort_flag, status, bytes; };
inline NoallocLayout noalloc_layout(const ResidentPlan &pl, size_t p_bytes, int B)
{
    NoallocLayout l{};
    auto take = [&](size_t bytes) { const size_t at = l.bytes; l.bytes += sized(bytes); return at; };
    l.P = take(p_bytes);
    l.xbuf = take(exchange_bytes(pl, B));
    l.form = take((size_t)pl.n_xcd * 32 * sizeof(unsigned));
    l.stats = take((size_t)pl.n_teams * kStatStride * sizeof(long long));
    l.abort_flag = take(sizeof(unsigned));
    l.status = take(sizeof(int));
    return l;
}

}  // namespace rnnt
