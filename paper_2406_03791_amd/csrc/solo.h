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
RNNT_HD constexpr int solo_tiles(int NOUT) { return NOUT <= 32 ? 2 : 4; }        // of 16 outputs
// Weights as the threads take them, four values each, [part][thread of 256]: sixteen parts of the recurrent
// matrix, four of the projection, a tile of outputs each.
RNNT_HD constexpr int solo_parts(int tiles) { return 16 + 4 + tiles; }

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

// w: solo_parts(solo_tiles(NOUT)) * 256 groups of four; *check, zero before: raised if a weight is not finite
hipError_t pack_solo(const float *w_hh, const float *w_pred, const float *w_out, int H, int J, int NOUT, float4 *w, unsigned *check, hipStream_t stream);
hipError_t launch_solo(const SoloParams &p, bool plain, hipStream_t stream);

}  // namespace rnnt
