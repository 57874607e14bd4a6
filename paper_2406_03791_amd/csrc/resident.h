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
constexpr int kResRows = 8;               // utterances a team decodes at the same time at most (4 or 8, see resident_rows)
constexpr int kResSamples = 32;           // (utterance, frame) pairs per joint step at most
constexpr int kResCalm = 8;               // joint steps after which a row's frames may be halved, see the loop control
// Projected frames from which on they are brought to the L2 ahead of the steps that load them: what all XCDs' L2 hold.  (19 utterances of
// 333 frames, 16 MB: 618 us without, 621 with it; 32 of 500, 41 MB: 1278 and 1270.)
constexpr long long kResTouchBytes = 32 << 20;
// Rows of P of a launch of nb utterances that may be asked for, none if it stays below that.
inline int touch_rows(int nb, int T, int J) { return (long long)nb * T * J * (long long)sizeof(float) > kResTouchBytes ? nb * T : 0; }
// Where the frames `la` after a sample's are, -1 beyond the last of `rows` or for no sample (row -1).  The frame may be of the next utterance,
// or padding: it is brought to the L2 and not looked at.
RNNT_HD constexpr int touch_row(int row, int la, int rows)
{
    const int at = (int)((unsigned)row + (unsigned)la);          // (negative beyond 2^31)
    return at >= la && at < rows ? at : -1;
}
constexpr int kResList = 128;             // utterances a team takes per launch at most

// Size classes: the register arrays, LDS rows and exchange buffers have compile-time sizes, so the
// stages are straight-line code.  A model runs in the smallest class that holds it.
constexpr int kResClasses = 3;
RNNT_HD constexpr int res_width(int cls) { return cls == 0 ? 640 : (cls == 1 ? 320 : 128); }   // widest layer
RNNT_HD constexpr int res_team(int cls) { return cls == 0 ? 32 : (cls == 1 ? 16 : 8); }         // work-groups per team
RNNT_HD constexpr int res_row(int cls) { return cls == 0 ? 640 : (cls == 1 ? 384 : 128); }      // floats per frame row in LDS

// Every dense stage: a wave takes an eighth of K (80, 48 or 16 values, one after the other) in blocks of 32, one
// 16x16x32 matrix instruction each, and where it is odd a last half block of 16.  res_halves: half blocks.
RNNT_HD constexpr int res_halves(int cls) { return res_row(cls) / 128; }
// Parts of an fp32 value on the 16-bit matrix instructions: value = high + low, two fp16 numbers of 11 bits
// (the low one's sign makes 23), after a power of two that takes the largest of a row to 2^14 .. 2^15.
// Kept in as many registers as the value itself.  Against 64 bits the logits of layers of 320 and 640 are 0 to 6 % closer
// than with fp32 products in a chain.  In the narrowest class, whose chains are short, they were 7 % further
// off: its joint output has whole fp32 values (res_whole, four 16x16x4 for a half block).
constexpr int kResHiddenExp = 15;         // hidden values travel as fp16 parts of 2^15 times themselves (fp32)
constexpr float kResHuge = 1e38f;         // no bound of the joint step's operands is taken to be larger than this
RNNT_HD constexpr bool res_whole(bool bf, int cls) { return !bf && res_halves(cls) == 1; }
RNNT_HD constexpr int res_parts(bool bf) { return bf ? 1 : 2; }
// registers of a wave's share of T tiles of 16 outputs, and the place of block kb (kb == halves / 2: the half
// block), tile t, part (0 high, 1 low) among them
RNNT_HD constexpr int res_tile_regs(bool bf, int cls, int T) { return T * res_halves(cls) * 2 * res_parts(bf); }
RNNT_HD constexpr int res_tile_at(bool bf, int cls, int T, int kb, int t, int part)
{
    return kb < res_halves(cls) / 2 ? ((kb * T + t) * res_parts(bf) + part) * 4
                                    : res_halves(cls) / 2 * T * res_parts(bf) * 4 + (t * res_parts(bf) + part) * 2;
}

// Place of register `reg` of a run of n in its image of n * 64 words: groups of four, the lanes' one after the other, as they are loaded
// (n % 4 == 2: two groups of two at the end).
RNNT_HD constexpr int res_place(int n, int reg, int lane)
{
    return reg < n / 4 * 4 ? reg / 4 * 256 + lane * 4 + reg % 4 : n / 4 * 256 + lane * 2 + reg % 4;
}

// Helpers of kResident2Pair: a work-group's quarter of K in whole blocks, and the registers of a wave's three tiles of 16 outputs.
constexpr int kResQuarters = 4;
RNNT_HD constexpr int res_help_blocks(int cls) { return res_row(cls) / (32 * kResQuarters); }
RNNT_HD constexpr int res_help_regs(int cls) { return res_help_blocks(cls) * 3 * 2 * 4; }

// Kinds of resident decoders (which weights sit where).
enum ResidentKind {
    kResidentNone = 0,
    kResident1 = 1,       // one LSTM layer: a team inside one XCD holds everything
    kResident2 = 2,       // two layers in the bfloat16 mode: the same
    kResident2Pair = 3,   // two layers in fp32: a team on one XCD, the recurrent matrices on two others
};
// kResident2Pair: most XCDs have teams, and each pair of the others, one for either layer, works for up to kResServed of them.
// (Six and two of eight: with five and three, and helpers that had both matrices, 128 utterances took 5.65 instead of 5.29 ms.)
constexpr int kResServed = 6;
RNNT_HD constexpr int res_chain_xcds(int n_xcd) { return n_xcd - (n_xcd + kResServed + 1) / (kResServed + 2) * 2; }

struct ResidentPlan {
    int kind;             // ResidentKind
    int cls;              // size class
    int bf;               // bfloat16 mode
    int n_xcd;            // XCDs of the device (32 compute units each)
    int n_teams;
    int units;            // LSTM units per work-group
    int jgroups;          // groups of 4 columns of the prediction-side projection per work-group
    int nout_m, n_tail;   // joint output columns on the matrix instruction, and the few after them (one per work-group)
    int solo;             // a model for the kernel of one work-group per utterance (solo.h): n_teams work-groups, and nothing else of this
};

struct ResidentParams {
    int H, J, V1, VT, D, blank, NOUT;
    int tdt;
    int durations[kMaxDur];
    int B, T, S, cap;
    int slots;            // utterances decoded at a time per team
    int touch_rows;       // rows of P, if frames are to be brought to the L2 ahead (see the joint step), or 0
    unsigned spin_limit;
    ResidentPlan pl;
    const int *enc_len;
    const float *P;
    int *tokens, *tok_len, *frames, *durs;
    float *logits, *logps;
    int *done;
    const float *w;       // packed registers of the (main) work-groups: [rank][wave], runs of registers as in res_place
    const float *w_help;  // the same of the helpers (kResident2Pair), layer by layer
    const float *w_tail;  // [n_tail][res_row(cls)], scaled as the packed output columns
    // fp32: what sums of the scaled weights of an output are multiplied by; LSTM matrices [H][gate]
    const float *s_out, *s_pred, *s_ih, *s_hh[2];
    float q_bound;        // no q is larger (hidden values are within +-1), unless this is kResHuge
    // fp32: what P is like (TopWord), from the first utterance's words on; the number of the call, for its first launch
    const unsigned long long *p_top;
    unsigned long long *p_call;
    const float *T0, *bias_l, *b_pred, *b_out;
    unsigned char *xbuf;  // exchange buffers, resident_buf(kind, bf, cls).bytes per team
    unsigned *form;       // one word per work-group, zero at launch: the XCD it runs on
    unsigned *abort_flag;
    int *status;
    long long *stats;     // [n_teams][kStatStride]
    int zero_stats;
    int count_rows;       // prediction steps are counted per utterance (Algorithm 1) instead of per team
};

// The joint's operand z as it travels: [tile of 16 samples][wave][piece][lane], as the waves' matrix instructions take it.  Of a block of 32
// k's (a half block of 16) a lane has the eight (four) from 8 * (lane / 16) (4 * ...) on of sample lane % 16: fp32 in two pieces (one) of
// 16 bytes, bf16 in one (in half of one).
RNNT_HD constexpr unsigned res_z_wave(bool bf, int cls)
{
    return (unsigned)(bf ? res_halves(cls) / 2 * 1024 + res_halves(cls) % 2 * 512 : res_halves(cls) * 1024);
}
RNNT_HD constexpr unsigned res_z_slot(bool bf, int cls) { return kResSamples / 16 * kResWaves * res_z_wave(bf, cls); }
// Place of the four values from 4 * k4 on of sample s
RNNT_HD constexpr unsigned res_z_at(bool bf, int cls, int k4, int s)
{
    const int full = res_halves(cls) / 2, per = res_halves(cls) * 4, wave = k4 / per, in = k4 % per;
    const unsigned at = (unsigned)(s / 16 * kResWaves + wave) * res_z_wave(bf, cls);
    if (in < full * 8) {
        const unsigned lane = (unsigned)(in % 8 / 2 * 16 + s % 16);
        return bf ? at + (unsigned)(in / 8) * 1024u + lane * 16u + (unsigned)(in % 2) * 8u : at + (unsigned)(in / 8 * 2 + in % 2) * 1024u + lane * 16u;
    }
    const unsigned lane = (unsigned)((in - full * 8) * 16 + s % 16);
    return bf ? at + (unsigned)full * 1024u + lane * 8u : at + (unsigned)full * 2048u + lane * 16u;
}
// The first group of four values in the 16 bytes at `at` of a slot (bf16: the 16 bytes hold two, of one sample or of two)
RNNT_HD constexpr int res_z_k4(bool bf, int cls, unsigned at)
{
    const unsigned full = (unsigned)res_halves(cls) / 2u, in = at % res_z_wave(bf, cls), first = at / res_z_wave(bf, cls) % kResWaves * (unsigned)res_halves(cls) * 4u;
    const unsigned piece = in / 1024u, g = in / 256u % 4u;
    if (piece < full * (bf ? 1u : 2u)) return (int)(first + (bf ? piece * 8u + 2u * g : piece / 2u * 8u + 2u * g + piece % 2u));
    return (int)(first + full * 8u + (bf ? in % 1024u / 128u : g));
}

// Lanes that load a vector of hidden values, a bit each: columns 0 .. 2 * rows - 1 of sixteen (column n is of row n % rows, see Operand) of the rows in
// `active`, whose bits are 16 / rows apart: a copy of somebody else's words, or words of a row that has ended, would travel for nothing.
RNNT_HD constexpr unsigned long long res_takers(int rows, unsigned active)
{
    unsigned m = active;              // to a bit a row
    if (rows == 4) m = (m | m >> 3 | m >> 6 | m >> 9) & 0xfu;
    else { m = (m | m >> 1) & 0x3333u; m = (m | m >> 2) & 0x0f0fu; m = (m | m >> 4) & 0xffu; }
    return (m | m << rows) * 0x0001000100010001ull;
}

// Frames of each of n rows in a joint step of nt tiles of samples (nmt: of the instance; rows: of a team): dealt evenly, 31 for one row of two
// tiles, so that shifts of a word by 0 to 31 do.  (Label-dense steps, one tile of two: no more than a team of all rows has, they are not looked at.)
RNNT_HD constexpr int res_frames(int nt, int nmt, int rows, int n)
{
    const int at = n - 1;
    return (int)((nt == 2 ? 0x04040506080a101full : nmt == 1 ? 0x02020203'04050810ull : rows == 4 ? 0x04050505ull : 0x0202020304050505ull) >> ((at < 0 ? 0 : at) * 8) & 0xffu);
}
// The place among those rows that sample s is of: s / la, rounded down half a sample from where it changes, so that the last bits of
// inverse, 1 / la, say nothing.  Beyond the rows' samples it is the last place there can be: the word of rows has bits for no more.
RNNT_HD constexpr int res_turn(int s, float inverse, int rows)
{
    const int turn = (int)(((float)s + 0.5f) * inverse);
    return turn < rows ? turn : rows - 1;
}

// Byte offsets of a team's exchange buffers, every vector in kResSlots slots.
// hr, pre: kResident2Pair; pre: [layer][slot][quarter of K][rank][wave of the cells][lane]
struct ResidentBuf { unsigned h[2], z, key, dur, lse, hr[2], pre, bytes; };
RNNT_HD constexpr ResidentBuf resident_buf(int kind, bool bf, int cls, int rows)
{
    const unsigned vec = kResSlots * (unsigned)(rows * res_width(cls)) * 4u;
    const unsigned recs = kResSlots * kResSamples * (unsigned)res_team(cls);
    ResidentBuf b{};
    b.h[0] = 0; b.h[1] = vec; b.z = 2 * vec; b.key = b.z + kResSlots * res_z_slot(bf, cls);
    b.dur = b.key + recs * 8u;
    b.lse = b.dur + kResSlots * kResSamples * kMaxDur * 4u;
    b.hr[0] = b.hr[1] = b.pre = b.bytes = b.lse + recs * 4u;
    if (kind != kResident2Pair) return b;
    b.hr[1] = b.hr[0] + vec; b.pre = b.hr[1] + vec;
    b.bytes = b.pre + 2u * kResSlots * kResQuarters * (unsigned)res_team(cls) * 5u * 64u * (unsigned)rows;
    return b;
}

// Registers per lane of a work-group, in packing order: recurrent matrices (kResident1: layer 0;
// kResident2: both layers), input matrix of the second layer, prediction-side projection, joint
// output.  The helpers of kResident2Pair hold the recurrent matrices, see res_help_regs.
RNNT_HD constexpr int res_lstm_regs(bool bf, int cls) { return res_tile_regs(bf, cls, 5); }
RNNT_HD constexpr int res_pred_regs(bool bf, int cls) { return res_tile_regs(bf, cls, 2); }
RNNT_HD constexpr int res_joint_regs(bool bf, int cls) { return res_tile_regs(bf, cls, 2); }
RNNT_HD constexpr int res_main_regs(int kind, bool bf, int cls)
{
    return (kind == kResident2 ? 3 : 1) * res_lstm_regs(bf, cls) + res_pred_regs(bf, cls) + res_joint_regs(bf, cls);
}

// LDS layout in bytes (dynamic part).  p: the work-group's columns of the frames of the joint step's samples, 16 bytes for every lane of the
// waves that form the operand, z_at: their places of it.  part: the joint step's partial sums;
// before it, in their place, those of the input stage (ih).  proj: partial sums of the projection (read after
// the work-group's last barrier before the joint step).  rec0, rec: those of the first and of the top layer's
// recurrent stage, kept till the next prediction step.
// other: the partner's weights of the output layer (two tiles of samples).  tail: the tail columns (see output()),
// tpart: its partial sums.  state: cell state and recurrent pre-activations [layer][field][wave][lane] where they are
// not in registers.  scale: powers of two of the team's list (fp32).  touch: for words that are loaded for their
// lines only.
// nmt: tiles of 16 samples; rows: of a team.  Helpers: their own, from 0 on.
struct ResidentLds { int p, z_at, part, ih, rec0, proj, rec, other, tail, tpart, state, scale, touch, bytes; };
constexpr int kResSumRow = 36;            // floats per row of partial sums: of the joint step
constexpr int kResProjRow = 20;           // of the projection, as many columns as a work-group has
RNNT_HD constexpr int res_stage_row(int rows) { return rows == 4 ? 80 : 88; }        // and of the LSTM stages (eight rows in banks of their own)
constexpr int kResAlone = 81 * 1024;      // at least: more than half of a compute unit's, which so has one work-group, however few registers that takes
RNNT_HD constexpr ResidentLds resident_lds(int kind, bool bf, int cls, int nmt, int rows)
{
    ResidentLds l{};
    const int stage = kResWaves * rows * res_stage_row(rows) * 4, sums = kResWaves * 16 * nmt * kResSumRow * 4;
    l.p = 0;
    l.z_at = l.p + 3 * 64 * 16;
    l.part = l.ih = l.z_at + 3 * 64 * 4;
    int at = l.ih + (kind == kResident1 ? 0 : stage);
    if (at < l.part + sums) at = l.part + sums;
    l.proj = at; at += kResWaves * rows * kResProjRow * 4;
    if (kind == kResident2) { l.rec0 = at; at += stage; }
    l.rec = at; at += kind == kResident2Pair ? 0 : stage;
    l.other = at; at += nmt == 2 ? kResWaves * res_joint_regs(bf, cls) * 256 : 0;
    l.tail = at; at += (bf ? nmt + 1 : res_whole(bf, cls) ? 2 * nmt + 2 : 2 * nmt + 1) * res_row(cls) * 2;
    l.tpart = at; at += kResWaves * 2 * 16 * 4;
    l.state = at; at += kind == kResident2Pair ? 2 * (2 + rows / 4) * 5 * 64 * 4 : 0;
    l.scale = at; at += kind == kResident2 ? 0 : kResList * 4;
    l.touch = at; at += kind == kResident2Pair && cls == 0 && nmt == 2 ? 256 : 0;
    const int help = 2048 + 2 * (kResServed * rows / 8) * res_help_blocks(cls) * 1024;
    if (kind == kResident2Pair && at < help) at = help;
    l.bytes = (at + 15) & ~15;
    if (l.bytes < kResAlone) l.bytes = kResAlone;
    return l;
}
constexpr int kResCtl = 5504;             // bytes kept for the control block and votes
static_assert(resident_lds(kResident1, false, 0, 2, 8).bytes + kResCtl <= 160 * 1024 && resident_lds(kResident2, true, 0, 2, 8).bytes + kResCtl <= 160 * 1024 &&
              resident_lds(kResident2Pair, false, 0, 2, 8).bytes + kResCtl <= 160 * 1024, "the largest layouts and the control block fit the LDS");

// The model's matrices on the device (rows as in the model), and where their packed forms go: register images of the
// teams' and the helpers' work-groups, [rank][wave][runs of registers, see res_place]; tail columns; what sums are multiplied by; the
// scales of the rows, in the order of these, and two words, zero before: not every value is finite, and the largest
// value of q, from above (a float's bits; both fp32 only).
struct ResidentWeights { int H, J, L; const float *w_hh[2], *w_ih1, *w_pred, *b_pred, *w_out; };
struct ResidentImages { float *w, *w_help, *w_tail, *s_out, *s_pred, *s_ih, *s_hh[2], *row_scales; unsigned *check; };
hipError_t pack_resident(const ResidentPlan &pl, const ResidentWeights &rw, const ResidentImages &im, hipStream_t stream);

// nmt: tiles of 16 samples a joint step has, 1 (up to two utterances at a time per team) or 2
// end: an event for the kernel's own completion, or null (plain launches)
hipError_t launch_resident(const ResidentParams &p, int nmt, bool plain, hipStream_t stream, hipEvent_t end);

}  // namespace rnnt
