// Decode kernel with register-resident weights: parameters and the plan shared by the host side
// (engine.hip, which packs the weights) and the kernel (resident_impl.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "plan.h"

namespace rnnt {

constexpr int kResThreads = 512;          // eight waves, two per SIMD: 256 registers per lane
constexpr int kResWaves = 8;
constexpr int kResUnits = 20;             // LSTM units per work-group at most
constexpr int kResSlots = 4;              // exchange slots per vector, used in turn
constexpr int kResRows = 8;               // utterances a team decodes at the same time at most
constexpr int kResSamples = 32;           // (utterance, frame) pairs per joint step at most
constexpr int kResList = 128;             // utterances a team takes per launch at most

// Size classes: the register arrays, LDS rows and exchange buffers have compile-time sizes, so the
// stages are straight-line code.  A model runs in the smallest class that holds it.
constexpr int kResClasses = 3;
RNNT_HD constexpr int res_width(int cls) { return cls == 0 ? 640 : (cls == 1 ? 320 : 128); }   // widest layer
RNNT_HD constexpr int res_team(int cls) { return cls == 0 ? 32 : (cls == 1 ? 16 : 8); }         // work-groups per team
RNNT_HD constexpr int res_row(int cls) { return cls == 0 ? 640 : (cls == 1 ? 384 : 128); }      // floats per frame row in LDS

// K comes in pieces of four values: four registers and four 4x4x1 instructions in fp32, two registers
// and one 4x4x4 instruction in the bfloat16 mode.
RNNT_HD constexpr int res_piece_regs(bool bf) { return bf ? 2 : 4; }
RNNT_HD constexpr int res_pieces(int cls) { return res_width(cls) / 4; }
// LSTM stages: waves 0 .. 5 hold a sixth of K for units 0 .. 15, waves 6 and 7 an eighth per block for units 16 .. 19
RNNT_HD constexpr int res_lstm_pieces(int cls) { return (res_pieces(cls) + 5) / 6; }
// prediction-side projection: a group per pair of waves (half of K each), and an eighth of a fifth group
RNNT_HD constexpr int res_pred_own(int cls) { return (res_pieces(cls) + 31) / 32; }
RNNT_HD constexpr int res_pred_fifth(int cls) { return (res_pieces(cls) + 127) / 128; }
// joint steps per wave: 16 K values each, every eighth one of the joint width
RNNT_HD constexpr int res_joint_steps(int cls) { return res_row(cls) / 128; }
// bytes of an activation row in LDS; rows of a row group start 64 bytes apart modulo the banks
RNNT_HD constexpr int res_xrow(bool bf, int cls) { return res_width(cls) * (bf ? 2 : 4) + 64; }

// Kinds of resident decoders (which weights sit where).
enum ResidentKind {
    kResidentNone = 0,
    kResident1 = 1,       // one LSTM layer: a team inside one XCD holds everything
    kResident2 = 2,       // two layers in the bfloat16 mode: the same
    kResident2Pair = 3,   // two layers in fp32: a team on one XCD, the recurrent matrices on a second one
};

struct ResidentPlan {
    int kind;             // ResidentKind
    int cls;              // size class
    int bf;               // bfloat16 mode
    int n_xcd;            // XCDs of the device (32 compute units each)
    int n_teams;
    int units;            // LSTM units per work-group
    int jgroups;          // groups of 4 columns of the prediction-side projection per work-group
    int nout_m, n_tail;   // joint output columns on the matrix instruction, and the few after them (one per work-group)
};

struct ResidentParams {
    int H, J, V1, VT, D, blank, NOUT;
    int tdt;
    int durations[kMaxDur];
    int B, T, S, cap;
    int slots, la;        // utterances decoded at a time per team, frames per utterance and joint step
    unsigned spin_limit;
    ResidentPlan pl;
    const int *enc_len;
    const float *P;
    int *tokens, *tok_len, *frames, *durs;
    float *logits, *logps;
    int *done;
    const float *w;       // packed registers of the (main) work-groups: [rank][wave][register][lane]
    const float *w_help;  // the same of the helpers (kResident2Pair)
    const float *w_tail;  // [n_tail][res_row(cls)]
    const float *T0, *bias_l, *b_pred, *b_out;
    unsigned char *xbuf;  // exchange buffers, resident_buf(cls).bytes per team
    unsigned *form;       // one word per work-group, zero at launch: the XCD it runs on
    unsigned *abort_flag;
    int *status;
    long long *stats;     // [n_teams][kStatStride]
    int zero_stats;
    int count_rows;       // prediction steps are counted per utterance (Algorithm 1) instead of per team
};

// Byte offsets of a team's exchange buffers; every vector has kResSlots slots.
struct ResidentBuf {
    unsigned h[2], q, key, dur, lse, hr[2], pre, bytes;
};
RNNT_HD constexpr ResidentBuf resident_buf(int cls)
{
    const unsigned vec = kResSlots * kResRows * (unsigned)res_width(cls) * 4u;
    const unsigned recs = kResSlots * kResSamples * (unsigned)res_team(cls);
    ResidentBuf b{};
    b.h[0] = 0; b.h[1] = vec; b.q = 2 * vec; b.key = 3 * vec;
    b.dur = b.key + recs * 8u;
    b.lse = b.dur + kResSlots * kResSamples * kMaxDur * 4u;
    b.hr[0] = b.lse + recs * 4u; b.hr[1] = b.hr[0] + vec; b.pre = b.hr[1] + vec;
    // [layer][slot][rank][block of 16 (unit, row) pairs][lane]
    b.bytes = b.pre + 2u * kResSlots * (unsigned)res_team(cls) * 10u * 64u * 4u;
    return b;
}

// Registers per lane of a work-group, in packing order: recurrent matrices (kResident1: layer 0;
// kResident2: both layers), input matrix of the second layer, prediction-side projection, joint
// output.  The helpers of kResident2Pair hold the two recurrent matrices.
RNNT_HD constexpr int res_lstm_regs(bool bf, int cls) { return res_lstm_pieces(cls) * res_piece_regs(bf); }
RNNT_HD constexpr int res_pred_regs(bool bf, int cls) { return (res_pred_own(cls) + res_pred_fifth(cls)) * res_piece_regs(bf); }
RNNT_HD constexpr int res_joint_regs(bool bf, int cls) { return res_joint_steps(cls) * 2 * res_piece_regs(bf); }
RNNT_HD constexpr int res_main_regs(int kind, bool bf, int cls)
{
    return (kind == kResident2 ? 3 : 1) * res_lstm_regs(bf, cls) + res_pred_regs(bf, cls) + res_joint_regs(bf, cls);
}

// LDS layout in bytes (dynamic part): frames of the joint step's samples (later the step's partial
// sums), activation rows of the LSTM stages, q rows (before q arrives, partial sums of the input
// stage), tail column, partial sums of the recurrent stages and of the projection.
// rg: row groups, nmt: tiles of 16 samples.
struct ResidentLds { int p, xh, q, tail, rec, g4, tpart, bytes; };
constexpr int kResSumRow = 36;            // floats per sample row of the joint step's partial sums
RNNT_HD constexpr ResidentLds resident_lds(int kind, bool bf, int cls, int rg, int nmt)
{
    ResidentLds l{};
    const int p_frames = 16 * nmt * res_row(cls) * 4, p_sums = kResWaves * 16 * nmt * kResSumRow * 4;
    const int stage = kResWaves * rg * 1024, q = 4 * rg * (res_row(cls) + 16) * 4;
    l.p = 0;
    l.xh = p_frames > p_sums ? p_frames : p_sums;
    if (kind == kResident2Pair && l.xh < stage) l.xh = stage;         // (the helpers' partial sums)
    l.q = l.xh + (kind == kResident1 ? 1 : 2) * 4 * rg * res_xrow(bf, cls);
    l.tail = l.q + (q > stage ? q : stage);
    l.rec = l.tail + res_row(cls) * 4;
    l.g4 = l.rec + (kind == kResident2Pair ? 0 : stage);
    l.tpart = l.g4 + 2 * kResWaves * rg * 16 * 4;
    l.bytes = l.tpart + kResWaves * 2 * 16 * 4;
    return l;
}
static_assert(resident_lds(kResident2Pair, false, 0, 2, 2).bytes + 4096 <= 160 * 1024, "the largest layout and the control block fit the LDS");

// rg: row groups (of four utterances) a team decodes at the same time, 1 or 2
// nmt: tiles of 16 samples a joint step has, 1 or 2
hipError_t launch_resident(const ResidentParams &p, int rg, int nmt, bool plain, hipStream_t stream);

}  // namespace rnnt
