// Decode of small models by a work-group per utterance: one LSTM layer, no layer wider than 64, at most 64 outputs, fp32.  (That is what the
// kernel's threads and tiles are laid out for; a compute unit would hold more.)
#pragma once
#include <hip/hip_runtime.h>

#include "plan.h"

namespace rnnt {

constexpr int kSoloWidth = 64, kSoloOutputs = 64;
constexpr int kSoloThreads = 512;         // four waves for projection, joint and argmax, four for the recurrent layer
constexpr int kSoloFrames = 16;           // frames a joint step examines
constexpr int kSoloChunk = 64;            // frames that are loaded together; two chunks are in LDS
inline bool solo_holds(int H, int J, int L, int NOUT, bool bf)
{
    return !bf && L == 1 && H <= kSoloWidth && J <= kSoloWidth && NOUT <= kSoloOutputs;
}
// Tiles of 16 outputs, as many as it takes, but for a single token behind full ones (labels and a blank, no durations behind it): its products are
// four multiply-adds a lane beside the matrix instructions instead of a tile of its own (17 outputs, a call of 20 frames and 45 steps:
// 64.1 us with two tiles, 60.7 with one and the output behind it).  As many as it takes: 128 utterances of 16 outputs 27.7 us with two tiles, 26.1 with one, of
// 48 outputs 42.9 with four and 40.5 with three, of 49 31.2 with four, 30.3 with three and one output.
RNNT_HD constexpr bool solo_last(int NOUT, int VT) { return VT == NOUT && NOUT > 16 && NOUT % 16 == 1; }
RNNT_HD constexpr int solo_tiles(int NOUT, int VT) { return (NOUT - (solo_last(NOUT, VT) ? 1 : 0) + 15) / 16; }
// Weights as the threads take them, four values each, [part][thread of 256]: sixteen parts of the recurrent
// matrix, four of the projection, a tile of outputs each, and the output behind the tiles.
RNNT_HD constexpr int solo_parts(int NOUT, int VT) { return 16 + 4 + solo_tiles(NOUT, VT) + (solo_last(NOUT, VT) ? 1 : 0); }

struct SoloParams {
    int H, J, V1, VT, D, blank, NOUT, tdt;
    int durations[kMaxDur];
    int B, T, S, cap;
    const int *enc_len;
    const float *P;
    const float4 *w;
    const float *T0, *b_pred, *b_out;
    int *tokens, *tok_len, *frames, *durs;
    float *logits, *logps;
    int *done, *status;
    long long *stats;         // a record for every one of n_records work-groups
    int n_records;
};

// VT: token outputs, as in calls.  w: solo_parts(NOUT, VT) * 256 groups of four; *check, zero before: raised if a weight is not finite
hipError_t pack_solo(const float *w_hh, const float *w_pred, const float *w_out, int H, int J, int NOUT, int VT, float4 *w, unsigned *check, hipStream_t stream);
hipError_t launch_solo(const SoloParams &p, bool plain, hipStream_t stream, hipEvent_t end);

}  // namespace rnnt
