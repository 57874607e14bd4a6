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
constexpr int kResRows = 4;               // utterances a team decodes at the same time at most
constexpr int kResSamples = 32;           // (utterance, frame) pairs per joint step at most
constexpr int kResCalm = 16;              // joint steps after which a row's frames are halved, see the loop control
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
// prediction-side projection: fifteen of a wave's blocks are five groups of columns times three slices of K, so
// 24 slices in all
RNNT_HD constexpr int res_pred_pieces(int cls) { return (res_pieces(cls) + 23) / 24; }
// joint steps per wave: 16 K values each, every eighth one of the joint width
RNNT_HD constexpr int res_joint_steps(int cls) { return res_row(cls) / 128; }
// bytes of an activation row in LDS; the rows start 64 bytes apart modulo the banks
RNNT_HD constexpr int res_xrow(bool bf, int cls) { return res_width(cls) * (bf ? 2 : 4) + 64; }

// Kinds of resident decoders (which weights sit where).
enum ResidentKind {
    kResidentNone = 0,
    kResident1 = 1,       // one LSTM layer: a team inside one XCD holds everything
    kResident2 = 2,       // two layers in the bfloat16 mode: the same
    kResident2Pair = 3,   // two layers in fp32: a team on one XCD, the recurrent matrices on a second one
};
// kResident2Pair: most XCDs have teams, and each of the others works for up to kResServed of them
constexpr int kResServed = 2;
RNNT_HD constexpr int res_chain_xcds(int n_xcd) { return n_xcd * kResServed / (kResServed + 1); }

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
    // [layer][slot][rank][wave of the cells][lane]
    b.bytes = b.pre + 2u * kResSlots * (unsigned)res_team(cls) * 5u * 64u * 4u;
    return b;
}

// Registers per lane of a work-group, in packing order: recurrent matrices (kResident1: layer 0;
// kResident2: both layers), input matrix of the second layer, prediction-side projection, joint
// output.  The helpers of kResident2Pair hold the two recurrent matrices.
RNNT_HD constexpr int res_lstm_regs(bool bf, int cls) { return res_lstm_pieces(cls) * res_piece_regs(bf); }
RNNT_HD constexpr int res_pred_regs(bool bf, int cls) { return res_pred_pieces(cls) * res_piece_regs(bf); }
RNNT_HD constexpr int res_joint_regs(bool bf, int cls) { return res_joint_steps(cls) * 2 * res_piece_regs(bf); }
RNNT_HD constexpr int res_main_regs(int kind, bool bf, int cls)
{
    return (kind == kResident2 ? 3 : 1) * res_lstm_regs(bf, cls) + res_pred_regs(bf, cls) + res_joint_regs(bf, cls);
}

// LDS layout in bytes (dynamic part): frames of the joint step's samples, activation rows of the LSTM
// stages and partial sums of the projection (both done with when the joint step's partial sums take
// their place; so rows that no utterance is in hold anything), q rows (zeros beyond the joint width: what
// stands there is multiplied by zero weights), tail column, partial sums of the input stage and of the
// recurrent stages.
// nmt: tiles of 16 samples.
struct ResidentLds { int p, part, xh, g4, q, tail, ih, rec, tpart, bytes; };
constexpr int kResSumRow = 36;            // floats per sample row of the joint step's partial sums
RNNT_HD constexpr ResidentLds resident_lds(int kind, bool bf, int cls, int nmt)
{
    ResidentLds l{};
    const int frames = 16 * nmt * res_row(cls) * 4, sums = kResWaves * 16 * nmt * kResSumRow * 4;
    const int stage = kResWaves * 1024, q = kResRows * (res_row(cls) + 16) * 4;
    l.p = 0;
    l.part = l.xh = frames;
    // (kResident2Pair: where the first layer's rows are large enough, the projection's sums take their place)
    const int x_row = kResRows * res_xrow(bf, cls), proj = kResWaves * 60 * 16;
    const bool over = kind == kResident2Pair && x_row >= proj;
    l.g4 = over ? l.xh : l.xh + (kind == kResident1 ? 1 : 2) * x_row;
    l.q = over ? l.xh + 2 * x_row : l.g4 + proj;
    if (l.q < l.part + sums) l.q = l.part + sums;
    l.tail = l.q + q;
    l.ih = l.tail + res_row(cls) * 4;
    l.rec = l.ih + (kind == kResident1 ? 0 : stage);
    l.tpart = l.rec + (kind == kResident2Pair ? 0 : (kind == kResident2 ? 2 : 1) * stage);
    l.bytes = l.tpart + kResWaves * 2 * 16 * 4;
    return l;
}
constexpr int kResCtl = 3840;             // bytes kept for the control block
static_assert(resident_lds(kResident1, false, 0, 2).bytes + kResCtl <= 160 * 1024 && resident_lds(kResident2, true, 0, 2).bytes + kResCtl <= 160 * 1024 &&
              resident_lds(kResident2Pair, false, 0, 2).bytes + kResCtl <= 160 * 1024, "the largest layouts and the control block fit the LDS");

// nmt: tiles of 16 samples a joint step has, 1 or 2
hipError_t launch_resident(const ResidentParams &p, int nmt, bool plain, hipStream_t stream);

}  // namespace rnnt
