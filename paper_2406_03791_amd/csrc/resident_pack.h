// Host side of the resident decode kernel: which models fit it, and the packed register images
// of its work-groups (the order is that of resident_impl.h).  No device code and no HIP calls.
#pragma once
#include <algorithm>
#include <cstdint>
#include <cstring>
#include <vector>

#include "pack.h"
#include "resident.h"

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
    if (kind == kResident2Pair && n_xcd < 2) return pl;
    for (int cls = kResClasses - 1; cls >= 0; --cls) {
        const int ts = res_team(cls);
        const int units = (H + ts - 1) / ts, jg = (J / 4 + ts - 1) / ts;
        const int nout_m = std::min(NOUT, 32 * ts), n_tail = NOUT - nout_m;
        if (H > res_width(cls) || J > res_width(cls) || units > kResUnits || jg > 5 || n_tail > ts) continue;
        pl.kind = kind; pl.cls = cls; pl.bf = bf; pl.n_xcd = n_xcd;
        pl.n_teams = (kind == kResident2Pair ? res_chain_xcds(n_xcd) : n_xcd) * (32 / ts);
        pl.units = units; pl.jgroups = jg; pl.nout_m = nout_m; pl.n_tail = n_tail;
        return pl;
    }
    return pl;
}

struct ResidentWeights {
    int H, J, L;
    const std::vector<std::vector<float>> *w_hh, *w_ih;
    const std::vector<float> *w_pred, *w_out;
};

namespace resident_detail {

// word e of piece k4 (columns 4 k4 ...) of a row of length K: one fp32 or two bf16
inline uint32_t piece_word(const float *row, int K, int k4, int e, bool bf)
{
    uint32_t u = 0;
    const int k = k4 * 4;
    if (bf) {
        if (k + 2 * e < K) u = bf16_bits(row[k + 2 * e]);
        if (k + 2 * e + 1 < K) u |= (uint32_t)bf16_bits(row[k + 2 * e + 1]) << 16;
    } else if (k + e < K) {
        std::memcpy(&u, row + k + e, 4);
    }
    return u;
}

// LSTM matrix: lane 4 b + gate.  Waves 0 .. 5: block b is unit b, pieces i + wave * (pieces per wave);
// waves 6, 7: block 4 s + u is unit 16 + u, every eighth piece from 4 (wave - 6) + s on.
inline void put_lstm(uint32_t *dst, const ResidentPlan &pl, const std::vector<float> &w, int H, int rank, int wave)
{
    const int n = res_lstm_pieces(pl.cls), pr = res_piece_regs(pl.bf), u0 = rank * pl.units, nu = std::max(0, std::min(pl.units, H - u0));
    for (int i = 0; i < n; ++i)
        for (int lane = 0; lane < 64; ++lane) {
            const int b = lane >> 2, u = wave < 6 ? b : 16 + (b & 3);
            const int k4 = wave < 6 ? wave * n + i : i * 8 + (wave - 6) * 4 + (b >> 2);
            if (u >= nu || k4 * 4 >= H) continue;
            for (int e = 0; e < pr; ++e)
                dst[(i * pr + e) * 64 + lane] = piece_word(w.data() + (size_t)((lane & 3) * H + u0 + u) * H, H, k4, e, pl.bf);
        }
}

}  // namespace resident_detail

inline std::vector<uint32_t> pack_resident_main(const ResidentPlan &pl, const ResidentWeights &rw)
{
    using namespace resident_detail;
    const bool bf = pl.bf != 0;
    const int nreg = res_main_regs(pl.kind, bf, pl.cls), ts = res_team(pl.cls), pr = res_piece_regs(bf);
    std::vector<uint32_t> out((size_t)ts * kResWaves * nreg * 64, 0u);
    for (int rank = 0; rank < ts; ++rank)
        for (int wave = 0; wave < kResWaves; ++wave) {
            uint32_t *dst = out.data() + (size_t)(rank * kResWaves + wave) * nreg * 64;
            auto next = [&](int regs) { uint32_t *p = dst; dst += (size_t)regs * 64; return p; };
            if (pl.kind != kResident2Pair)
                for (int l = 0; l < rw.L; ++l) put_lstm(next(res_lstm_regs(bf, pl.cls)), pl, (*rw.w_hh)[l], rw.H, rank, wave);
            if (rw.L > 1) put_lstm(next(res_lstm_regs(bf, pl.cls)), pl, (*rw.w_ih)[1], rw.H, rank, wave);
            // prediction-side projection, lane 4 b + column: block b is group b % 5 and slice 3 wave + b / 5, every 24th
            // piece of K (block 15: nothing)
            {
                uint32_t *d = next(res_pred_regs(bf, pl.cls));
                const int g0 = rank * pl.jgroups, njg = std::max(0, std::min(pl.jgroups, rw.J / 4 - g0));
                for (int i = 0; i < res_pred_pieces(pl.cls); ++i)
                    for (int lane = 0; lane < 60; ++lane) {
                        const int g = (lane >> 2) % 5, k4 = i * 24 + wave * 3 + (lane >> 2) / 5;
                        if (g >= njg || k4 * 4 >= rw.H) continue;
                        for (int e = 0; e < pr; ++e)
                            d[(i * pr + e) * 64 + lane] =
                                piece_word(rw.w_pred->data() + (size_t)((g0 + g) * 4 + (lane & 3)) * rw.H, rw.H, k4, e, bf);
                    }
            }
            // joint output: steps wave, wave + 8, ... of K for both column tiles
            {
                uint32_t *d = next(res_joint_regs(bf, pl.cls));
                for (int ii = 0; ii < res_joint_steps(pl.cls); ++ii)
                    for (int c = 0; c < 2; ++c)
                        for (int lane = 0; lane < 64; ++lane) {
                            const int col = (rank * 2 + c) * 16 + (lane & 15), k4 = (ii * 8 + wave) * 4 + (lane >> 4);
                            if (col >= pl.nout_m || k4 * 4 >= rw.J) continue;
                            for (int e = 0; e < pr; ++e)
                                d[((ii * 2 + c) * pr + e) * 64 + lane] = piece_word(rw.w_out->data() + (size_t)col * rw.J, rw.J, k4, e, bf);
                        }
            }
        }
    return out;
}

inline std::vector<uint32_t> pack_resident_helper(const ResidentPlan &pl, const ResidentWeights &rw)
{
    const int n = res_lstm_regs(pl.bf, pl.cls);
    std::vector<uint32_t> out((size_t)res_team(pl.cls) * kResWaves * 2 * n * 64, 0u);
    for (int rank = 0; rank < res_team(pl.cls); ++rank)
        for (int wave = 0; wave < kResWaves; ++wave)
            for (int l = 0; l < 2; ++l)
                resident_detail::put_lstm(out.data() + (size_t)((rank * kResWaves + wave) * 2 + l) * n * 64, pl, (*rw.w_hh)[l], rw.H,
                                          rank, wave);
    return out;
}

}  // namespace rnnt
