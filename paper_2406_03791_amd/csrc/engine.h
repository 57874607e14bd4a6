// Internal declarations shared by the host API, the encoder-projection kernel
// and the persistent decode kernel.
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "plan.h"

namespace rnnt {

enum Variant { kFrameLooping = 0, kLabelLooping = 1, kTdtLabelLooping = 2 };
// Kernel instance of Algorithm 1 for teams of one utterance (chosen by the launch, never a caller's variant).
constexpr int kFrameLoopingSingle = 3;

// Packed weights of one dense stage on the device.
struct StageDev {
    const float4 *w;       // [rank][wave][slot][step][lane], 16 bytes each: 4 fp32, 8 bf16 or 16 e4m3 weights
    int nks, nsteps, slots, kpad;
    long long rank_stride; // float4 elements per rank
};

struct DecodeParams {
    int F, E, H, L, J, V1, D, blank, NOUT;
    int VT;                 // output columns of the token distribution: V1, plus the big blanks of a multi-blank model
    int durations[kMaxDur]; // TDT: the durations; multi-blank: the spans of the big blanks (output columns V1 ...)
    int B, T, S, cap, variant;
    int wt;                 // WeightType of the packed stages
    int n_teams, team_size, lookahead;
    int search_steps;       // label looping: joint steps per search before the next prediction step (0: no limit)
    int groups, jteam_size; // joint groups per team and work-groups per joint group
    int plain_launch;       // ordinary instead of cooperative launch (engine flag)
    int spread;             // work-group i is rank i % team_size of team i / team_size (else team i % n_teams, rank i / n_teams)
    int serpentine;         // deal length-ranked utterances to teams 0..n-1, n-1..0, ... (else 0..n-1, 0..n-1)
    int xstride;            // floats per activation row in LDS
    int nu_max;             // most hidden units owned by a rank
    int gj_max;             // most joint output groups owned by a rank
    int gp_max;             // most prediction-projection output groups owned by a rank
    // dynamic LDS layout, offsets in floats
    int lds_xz, lds_red, lds_c, lds_part, lds_bias, lds_q;
    int lds_scale;          // scales of e4m3- or e2m1-stored weights (bfloat16 mode), see Lds::s_pred
    int sc_nb_in;           // scale blocks per row of the input stages' tables in LDS
    int rcap;               // rows the LDS state buffers are laid out for (>= rows of any team)
    int rg_planned;         // row groups the activation rows and partial sums in LDS are sized for
    int samples_cap;        // samples of a joint step the z rows and argmax candidates in LDS are sized for
    int fast_pred;          // teams of up to 4 rows: hidden vectors kept in LDS, tagged exchange (no barriers)
    int lds_hc;             // offset of the LDS copies of the hidden vectors [2][L][4][xstride]
    int n_tail;             // joint output columns nout_m .. nout_m + n_tail - 1 are computed by rank 0 .. n_tail - 1 with plain multiply-adds
    int nout_m;             // joint output columns covered by the MFMA stage (NOUT when n_tail == 0)
    int lds_tail;           // offset of a tail column's weight row [J rounded up to 4] and partial sums [waves][kMaxSamples]
    const float *w_tail;    // [n_tail][J rounded up to 4]
    int q_in_lds;           // q = W_pred h + b_pred of the team's rows is kept in LDS
    int qstride;            // floats per q row in LDS
    unsigned lds_bytes;
    unsigned spin_limit;
    const int *enc_len;     // [B]
    const float *P;         // [B, T, J] projected frames
    int *tokens; int *tok_len; int *frames; float *logits; int *durs;
    float *logps;           // [B, cap] log-softmax value of each emitted label, or NULL
    int *done;              // [B] set to 1 once an utterance's outputs are final, or NULL
    StageDev st0;                 // recurrent (h) parts of all layers
    StageDev stl[kMaxLayers];     // input parts of layers 1..L-1 (index = layer)
    StageDev spred;               // prediction-side joint projection
    StageDev sjoint;              // joint output projection
    const float *T0;        // [V1][H][4]: W_ih0 emb[v] + b_ih0 + b_hh0, gates of a unit adjacent
    const float *bias_l;    // [L][H][4]: b_ih + b_hh of layers >= 1 (layer 0 unused)
    const float *b_pred;    // [J]
    const float *b_out;     // [NOUT]
    // e4m3 / e2m1 storage in the bfloat16 mode: the power of two the codes of a weight row (e4m3)
    // or of each block of kScaleBlock weights of a row (e2m1) are multiplied by; nb = scale_blocks_of_matrix
    const float *sc_hh, *sc_ih;   // [L][H][4][nb], as bias_l (sc_ih of layer 0 unused)
    const float *sc_pred;   // [J][nb]
    const float *sc_out;    // [NOUT][nb]
    // team workspace
    float *hbuf;                  // [n_teams][2][L][kMaxRows][H]
    float *qbuf;                  // [n_teams][kMaxRows][J]
    unsigned long long *part;     // [n_teams * groups][2][kMaxSamples][jteam_size] token partial argmax
    unsigned long long *dpart;    // same for durations
    unsigned long long *lpart;    // same layout: a rank's sum of exp(logit - its maximum)
    unsigned long long *rowx;     // [n_teams][2][kMaxRows]: row state published by the owning joint group
    unsigned long long *xh;       // [n_teams][L][kMaxRows][H]: candidate hidden values as (step tag, float bits)
    unsigned long long *xq;       // [n_teams][kMaxRows][J]: q the same way
    unsigned *bar;                // [n_teams * 32]: one counter per team, 128 B apart
    unsigned *abort_flag;
    int *status;
    long long *stats;             // [n_teams][kStatStride]; phase timers after the counters
    int *xcc;                     // [n_teams * team_size]
};

// A call of many utterances takes several launches: the status word starts at zero in the call's
// first launch (zero_status) and the step counts in the first launch that uses their buffer
// (zero_stats); later launches add to them.
hipError_t launch_decode(const DecodeParams &p, bool zero_status, bool zero_stats, hipStream_t stream);

// What a call's P is like, for the resident decode kernel: the number of the call, which the decode kernel counts up (so
// a captured call does it too), and kTopParts words for every utterance, a line of memory each (one word for all blocks
// that have an utterance took 5.5 us of a projection of 17): its largest finite value, as number << 16 | upper half of the
// value, rounded up.  They only ever grow: nothing needs to be cleared between calls, an utterance's words with the
// largest number are the call's.  (Of the utterance, not of the call: one with large values costs the others no time.)
typedef unsigned long long TopWord;
constexpr int kTopParts = 16, kTopStride = 8;
constexpr size_t top_words(size_t utterances) { return (utterances * kTopParts + 1) * kTopStride; }

// What the projection kernel clears for the decode kernel behind it; nothing where NULL.
struct CallInit {
    unsigned *form = nullptr;       // meeting words of the resident decode kernel
    int n_form = 0;
    unsigned *abort_flag = nullptr;
    int *status = nullptr;
    int *tokens = nullptr, *frames = nullptr, *durs = nullptr;   // output rows [B, cap]
    float *logits = nullptr, *logps = nullptr;
    int cap = 0;
    long long *stats = nullptr;     // where the call's times go (kStatCallStart ...)
    TopWord *p_top = nullptr;       // top_words(B) words on what the call's P is like
};

// Keeps the text of a failed HIP call for rnnt_status_string; returns RNNT_ERR_HIP.
int hip_fail(hipError_t e, const char *what);

// Decode kernels of one device run one after another, whatever their streams: the work-groups of a
// decode wait for each other, so two of them that each had a part of the compute units would wait
// forever.  A cooperative launch orders itself behind the other cooperative ones of the process, at 17 to
// 55 us a call (one short utterance of a tiny model: 170 against 117 us); here every decode records an event
// after itself and waits for that of the one before, which costs nothing on the same stream, and holds for the
// decodes that one copy of this library enqueues.  (RNNT_FLAG_COOPERATIVE_LAUNCH: for callers who have others; of
// two processes with cooperative launches the runtime refused the second one's, "operation cannot be performed in the
// present state".)  `enqueue` launches the kernels (LaunchTurn).  In a stream capture, where an event from outside cannot be
// waited for, the launches stay cooperative.
constexpr int kDevices = 64;
struct LaunchOrder { std::mutex m; hipEvent_t last = nullptr; bool used = false; };
// A decode's place in that order.  plain: it may launch its kernels ordinarily.  end: the event that its last kernel may record by its own
// completion (launch_ending; ended says that it did), as an event behind it is a packet of its own in the queue, 1.1 us a call (the smallest
// model 55.5 us with a packet, 54.2 without, two utterances of the small one 59.3 and 58.0, 32 short ones of the large one 278.0 and 276.8).
struct LaunchTurn { bool plain; hipEvent_t end; bool ended; };
inline hipError_t launch_ending(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t stream, hipEvent_t end)
{
    if (end) return hipExtLaunchKernel(fn, grid, block, args, lds, stream, nullptr, end, 0);
    return hipLaunchKernel(fn, grid, block, args, lds, stream);
}
inline LaunchOrder &launch_order(int dev)
{
    static LaunchOrder devices[kDevices];
    return devices[dev];
}
template <class F>
inline int in_launch_order(hipStream_t stream, F enqueue)
{
    int dev = 0, rc = 0;
    auto ok = [&](hipError_t e, const char *what) { if (e != hipSuccess) rc = hip_fail(e, what); return e == hipSuccess; };
    if (!ok(hipGetDevice(&dev), "hipGetDevice")) return rc;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (!ok(hipStreamIsCapturing(stream, &capture), "hipStreamIsCapturing")) return rc;
    LaunchTurn turn{false, nullptr, false};
    if (dev >= kDevices || capture != hipStreamCaptureStatusNone) return enqueue(turn);
    LaunchOrder &d = launch_order(dev);
    std::lock_guard<std::mutex> lock(d.m);
    // (The event only keeps kernels of this device apart, which fence for themselves: without its own fence for the host and other devices a
    // call of one utterance takes 1.7 us less, the smallest model's 67.2 us and 65.6.)
    if (!d.last && !ok(hipEventCreateWithFlags(&d.last, hipEventDisableTiming | hipEventDisableSystemFence), "hipEventCreate")) return rc;
    if (d.used && !ok(hipStreamWaitEvent(stream, d.last, 0), "hipStreamWaitEvent")) return rc;
    turn = LaunchTurn{true, d.last, false};
    const int done = enqueue(turn);
    // (also after a failed launch: kernels of the call may be under way)
    if (!turn.ended && !ok(hipEventRecord(d.last, stream), "hipEventRecord")) return rc;
    d.used = true;
    return done;
}

// W_enc on the device.  parts: as the matrix instructions take it, [tile of 32 columns][16 k's][part][lane][8 values],
// enc_columns(J) columns, zeros beyond J; fp32: two fp16 parts of the values, after a power of two of the column;
// bfloat16 mode: one part.  bias [enc_columns(J)]; fp32 only: inverse of the powers of two [enc_columns(J)], the
// values themselves, and whether one of them is not finite.
struct EncWeights { const unsigned *parts; const float *inverse, *plain; const unsigned *not_finite; const float *bias; };
inline int enc_columns(int J) { return (J + 127) / 128 * 128; }
// w: [J][F]; scratch: J floats (bf16: unused, as inverse and check, which has to be zero before)
hipError_t pack_projection(const float *w, int F, int J, bool bf16, unsigned *parts, float *inverse, unsigned *check, float *scratch, hipStream_t stream);
hipError_t launch_encoder_projection(const float *enc_out, const int *enc_len, const EncWeights &w, float *proj, int B, int T, int F, int J,
                                     bool round_x, const CallInit &ci, hipStream_t stream);
// Clears what a further launch of the resident decode kernel within a call needs cleared.
hipError_t launch_reset_resident(unsigned *form, int n_form, unsigned *abort_flag, hipStream_t stream);
// v[i] = nearest bfloat16 value of v[i] (ties to even), in place
hipError_t launch_round_bf16(float *v, long long n, hipStream_t stream);
// T0[v][u][g] = b_ih0[g*H+u] + b_hh0[g*H+u] + sum_e W_ih0[g*H+u][e] * emb[v][e]
hipError_t launch_fold_embedding(const float *emb, const float *w_ih0, const float *b_ih0,
                                 const float *b_hh0, float *T0, int V1, int E, int H,
                                 bool round_bf16, hipStream_t stream);

}  // namespace rnnt
