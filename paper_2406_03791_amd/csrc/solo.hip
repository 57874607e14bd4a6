// Decode kernel for small models (solo.h).
//
// One work-group per utterance, and nothing goes from one work-group to another.  Spread over the eight work-groups of a
// team of the resident kernel, as every model of one layer was, a model of 64 units and 17 outputs spent its steps on hand-overs:
// three of 0.4 to 0.5 us and the latency around them, 3.5 us a step; here vectors go through LDS, and a step takes
// 1.07 us (a call of one utterance of 20 frames 157 and 55 us).  Emitted logits are 2.1e-8 from 64 bits, rms,
// as they were.
//
// Bound by latency: a chain of cell, projection, joint, sums over the waves and argmax, with three barriers.  What can be off the chain
// is: waves 0 .. 3 run projection, joint and argmax, waves 4 .. 7 (which share their SIMDs) hold the recurrent matrix, compute
// W_hh h for the next label beside that and then have the cells' pre-activations in their registers.  The loop control is
// uniform: every wave takes the same decisions from the same sixteen results.  (Projection behind a barrier of its own, outputs
// written by a wave that has cells, and one instance for all models: 1.6 us a step.)  A tile's four matrix
// instructions and the reads of their sums are 0.075 us of a step, the rest is LDS latency (six times 100 cycles and more), barriers
// and two gate functions.
// All products are fp32 instructions: plain multiply-adds for one vector, 16x16x4 matrix instructions for the sixteen
// frames of a joint step, K in quarters over the waves.
#include <type_traits>

#include "engine.h"
#include "gate.h"
#include "solo.h"

namespace rnnt {
namespace {

typedef float s4f __attribute__((ext_vector_type(4)));

// The value at place `e` of group `i`, or 0
__device__ __forceinline__ float solo_weight(const float *w_hh, const float *w_pred, const float *w_out, int H, int J, int NOUT, int tiles, int i, int e)
{
    const int part = i >> 8, t = i & 255;
    if (part < 16) {              // gate t % 4 of unit t / 4
        const int u = t >> 2, k = part * 4 + e;
        return u < H && k < H ? w_hh[((long long)(t & 3) * H + u) * H + k] : 0.f;
    }
    if (part < 20) {              // a quarter of K of output t / 4
        const int j = t >> 2, k = (t & 3) * 16 + (part - 16) * 4 + e;
        return j < J && k < H ? w_pred[(long long)j * H + k] : 0.f;
    }
    const int o = (part - 20) * 16 + (part - 20 < tiles ? t & 15 : 0), k = (t >> 6) * 16 + (t >> 4 & 3) * 4 + e;
    return o < NOUT && k < J ? w_out[(long long)o * J + k] : 0.f;
}

__global__ void __launch_bounds__(256) pack_solo_kernel(const float *__restrict__ w_hh, const float *__restrict__ w_pred, const float *__restrict__ w_out, int H, int J, int NOUT,
                                                        int tiles, int n, float4 *__restrict__ w, unsigned *check)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float v[4];
    bool finite = true;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] = solo_weight(w_hh, w_pred, w_out, H, J, NOUT, tiles, i, e);
        finite = finite && fabsf(v[e]) < INFINITY;
    }
    w[i] = make_float4(v[0], v[1], v[2], v[3]);
    if (!finite) atomicOr(check, 1u);
}

template <int CTRL>
__device__ __forceinline__ float solo_dpp(float v)
{
    return __uint_as_float((unsigned)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), CTRL, 0xf, 0xf, true));
}
// over sixteen adjacent lanes (one instruction a step; fmaxf of a permuted value takes three)
__device__ __forceinline__ float max16(float v)
{
    asm("s_nop 1\n\tv_max_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf" : "+v"(v));
    return v;
}
__device__ __forceinline__ float sum16(float v)
{
    v += solo_dpp<0xB1>(v); v += solo_dpp<0x4E>(v); v += solo_dpp<0x141>(v);
    return v + solo_dpp<0x140>(v);
}

// acc[i / 4][i % 4] += w[i / 4][i % 4] * (x of lane FIRST + i of the sixteen), i = 0 .. 7: broadcast and multiply-add in one
// instruction, which the compiler does not make of the two
template <int FIRST>
__device__ __forceinline__ void fma_row8(const s4f *w, float x, s4f *acc)
{
    float a[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = acc[i / 4][i % 4];
#define FMA_ROW(i, wi, lane) "v_fmac_f32_dpp %" #i ", %16, %" #wi " row_newbcast:" #lane " row_mask:0xf bank_mask:0xf\n\t"
#define FMA_ROWS(l0, l1, l2, l3, l4, l5, l6, l7)                                                                                    \
    asm("s_nop 1\n\t" FMA_ROW(0, 8, l0) FMA_ROW(1, 9, l1) FMA_ROW(2, 10, l2) FMA_ROW(3, 11, l3)                                     \
        FMA_ROW(4, 12, l4) FMA_ROW(5, 13, l5) FMA_ROW(6, 14, l6) FMA_ROW(7, 15, l7)                                                \
        : "+&v"(a[0]), "+&v"(a[1]), "+&v"(a[2]), "+&v"(a[3]), "+&v"(a[4]), "+&v"(a[5]), "+&v"(a[6]), "+&v"(a[7])                           \
        : "v"(w[0][0]), "v"(w[0][1]), "v"(w[0][2]), "v"(w[0][3]), "v"(w[1][0]), "v"(w[1][1]), "v"(w[1][2]), "v"(w[1][3]), "v"(x))
    static_assert(FIRST == 0 || FIRST == 8, "half of sixteen lanes");
    if constexpr (FIRST == 0) FMA_ROWS(0, 1, 2, 3, 4, 5, 6, 7);
    else FMA_ROWS(8, 9, 10, 11, 12, 13, 14, 15);
#undef FMA_ROWS
#undef FMA_ROW
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i / 4][i % 4] = a[i];
}

// LDS, in floats: a ring of 2 * kSoloChunk frames, T0, the waves' partial sums [wave][frame][outputs], those of an output beyond the
// tiles [frame][wave][lane / 16] (rows of 20: sixteen frames' rows in banks of their own), h, and the
// results of the frames (label, duration, logit, log-probability), and the table of durations
constexpr int kSoloLastRow = 20;
struct SoloLds { int frames, t0, part, last, h, res, dur, total; };
RNNT_HD constexpr SoloLds solo_lds(int V1, int tiles)
{
    SoloLds l{};
    l.frames = 0;
    l.t0 = 2 * kSoloChunk * kSoloWidth;
    l.part = l.t0 + V1 * 4 * kSoloWidth;
    l.last = l.part + 4 * kSoloFrames * (tiles * 16 + 4);
    l.h = l.last + kSoloFrames * kSoloLastRow;
    l.res = l.h + kSoloWidth;
    l.dur = l.res + 4 * kSoloFrames;
    l.total = l.dur + kMaxDur;
    return l;
}
static_assert(solo_lds(kSoloOutputs, 4).total * 4 <= 160 * 1024, "the largest model fits the LDS");

// TILES: of 16 outputs; LAST: and one more behind them; WALK: TDT and multi-blank models, where not every blank moves on by one frame
template <int TILES, bool LAST, bool WALK>
__global__ void __launch_bounds__(kSoloThreads) solo_kernel(const SoloParams p)
{
    extern __shared__ __align__(16) float lds[];
    constexpr int PS = TILES * 16 + 4, W = kSoloWidth, NF = kSoloFrames;
    const SoloLds lo = solo_lds(p.V1, TILES);
    const int tid = threadIdx.x, lane = tid & 63, t256 = tid & 255, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool chain = wave < 4;
    if (chain) __builtin_amdgcn_s_setprio(2);        // (0.4 to 0.9 % of a call: the SIMD's other wave is ready early enough)
    if (blockIdx.x == 0) {
        if (tid == 0) p.stats[kStatDecodeStart] = wall_clock64();
        for (int i = gridDim.x + tid; i < p.n_records; i += kSoloThreads)
            for (int c = 0; c < kStatCounters; ++c) p.stats[(long long)i * kStatStride + c] = 0;
    }
    // What is read before the first step is asked for in one go, the first utterance's frames as soon as their places are cleared: one trip to
    // memory where there were three or four, one after the other (one utterance of 20 frames 54.0 and 52.2 us, 12 of 150 frames 341 and 337).
    const unsigned lds_frames = (unsigned)(uintptr_t)(__attribute__((address_space(3))) float *)(lds + lo.frames);
    // A chunk of an utterance's frames, straight into LDS: a wave's instruction takes four frames, its lanes pieces of
    // 16 bytes; piece k4 of a frame lies at k4 with its bits xored with the frame's last four, so that sixteen
    // frames' pieces of the same k sit in different banks.
    auto load_chunk = [&](int b, int len, int c) {
#pragma unroll
        for (int i = 0; i < kSoloChunk / 4 / 8; ++i) {
            const int f = c * kSoloChunk + (wave * (kSoloChunk / 4 / 8) + i) * 4, fl = f + (lane >> 4), k4 = (lane ^ fl) & 15;
            const char *src = reinterpret_cast<const char *>(p.P + ((long long)b * p.T + f) * p.J);
            const unsigned off = (unsigned)(min(fl, len - 1) - f) * (unsigned)(p.J * 4) + (unsigned)k4 * 16u;
            const unsigned to = (unsigned)__builtin_amdgcn_readfirstlane((int)(lds_frames + (unsigned)(f & (2 * kSoloChunk - 1)) * (W * 4)));
            if (f < len && k4 * 4 < p.J)
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2" :: "v"(off), "s"(to), "s"(src) : "memory");
        }
    };
    auto frames_there = [&]() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
    const int first_raw = p.enc_len[blockIdx.x], first_len = min(max(first_raw, 0), p.T);       // (no more blocks than utterances)
    for (int i = tid; i < 2 * kSoloChunk * W / 4; i += kSoloThreads) reinterpret_cast<s4f *>(lds + lo.frames)[i] = (s4f){0.f, 0.f, 0.f, 0.f};       // (beyond the joint width it stays so)
    // Weights: the recurrent matrix's, or those of projection and joint.
    s4f w[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        w[i] = (s4f){0.f, 0.f, 0.f, 0.f};
        if (!chain || i < 4 + TILES + LAST) w[i] = reinterpret_cast<const s4f *>(p.w)[(chain ? 16 + i : i) * 256 + t256];
    }
    const float b_pred = (t256 >> 2) < p.J ? p.b_pred[t256 >> 2] : 0.f;
    float b_out[TILES];
#pragma unroll
    for (int c = 0; c < TILES; ++c) b_out[c] = (tid & 15) * TILES + c < p.NOUT ? p.b_out[(tid & 15) * TILES + c] : 0.f;
    const float b_last = LAST ? p.b_out[TILES * 16] : 0.f;
    __syncthreads();
    load_chunk(blockIdx.x, first_len, 0);
    load_chunk(blockIdx.x, first_len, 1);
    // (a unit's four gates at a time)
#pragma unroll 4
    for (int i = tid; i < p.V1 * W; i += kSoloThreads) {
        const int v = i / W, u = i - v * W;
        reinterpret_cast<s4f *>(lds + lo.t0)[i] = u < p.H ? reinterpret_cast<const s4f *>(p.T0)[(long long)v * p.H + u] : (s4f){0.f, 0.f, 0.f, 0.f};
    }
    if (tid < W) lds[lo.h + tid] = 0.f;
    // (opaque, so that they are not read again)
#pragma unroll
    for (int i = 0; i < 16; ++i) asm volatile("" : "+v"(w[i]));
    float *part = lds + lo.part, *hv = lds + lo.h;
    s4f q = {0.f, 0.f, 0.f, 0.f};                // of the lane's k's of a joint step
    int *res = reinterpret_cast<int *>(lds + lo.res), *res_d = res + 2 * NF;        // label and logit, duration
    float *res_lp = lds + lo.res + 3 * NF;
    int *durations = reinterpret_cast<int *>(lds + lo.dur);
    if (tid < kMaxDur) durations[tid] = p.durations[tid];
    const bool tdt = WALK && p.tdt;
    const bool writer = tid == 255;               // of all outputs, in a wave that waits for the cells next
    long long n_pred = 0, n_joint = 0, n_samples = 0;
    int flags = 0;

    for (int b = blockIdx.x; b < p.B; b += gridDim.x) {
        const bool is_first = b == (int)blockIdx.x;
        const int raw = is_first ? first_raw : p.enc_len[b], len = min(max(raw, 0), p.T);
        if (raw != len) flags |= 1;
        int t = 0, n = 0, cnt = 0, last = p.blank, have = 1;
        bool need = true, pending = false;
        __syncthreads();              // (nobody reads the last utterance's frames any more; T0 is there)
        if (!is_first) {
            load_chunk(b, len, 0);
            load_chunk(b, len, 1);
        }
        float c = 0.f, pre = 0.f, t0 = lds[lo.t0 + last * (4 * W) + t256];
        frames_there();
        __syncthreads();
        while (t < len) {
            // the lane's part of frame t + lane % 16
            auto frame_values = [&]() {
                const int f = (t + (lane & 15)) & (2 * kSoloChunk - 1), k4 = wave * 4 + (lane >> 4);
                return *reinterpret_cast<const s4f *>(lds + lo.frames + f * W + ((k4 ^ f) & 15) * 4);
            };
            s4f pv = {0.f, 0.f, 0.f, 0.f};
            if (need) {
                ++n_pred;
                if (!chain) {
                    // the cell: lanes of a unit hold the gates i, f, g, o
                    const float act = gate_act(pre + t0, (lane & 3) == 2);
                    const float i_ = solo_dpp<0x00>(act), f_ = solo_dpp<0x55>(act), g_ = solo_dpp<0xAA>(act), o_ = solo_dpp<0xFF>(act);
                    c = fmaf(f_, c, i_ * g_);
                    const float h = o_ * gate_act(c, true);
                    if ((lane & 3) == 0) hv[t256 >> 2] = h;
                }
                if (pending) { frames_there(); pending = false; }
                __syncthreads();
                if (chain) {
                    pv = frame_values();
                    // projection: four lanes per output, a quarter of K each
                    s4f acc;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const s4f x = reinterpret_cast<const s4f *>(hv)[(lane & 3) * 4 + i];
                        acc[i] = w[i][0] * x[0];
#pragma unroll
                        for (int e = 1; e < 4; ++e) acc[i] = fmaf(w[i][e], x[e], acc[i]);
                    }
                    float o = (acc[0] + acc[1]) + (acc[2] + acc[3]);
                    o += solo_dpp<0xB1>(o); o += solo_dpp<0x4E>(o);
                    // The sixteen values are those that this wave's part of the joint step needs, four of them in every sixteen lanes that
                    // need those: broadcasts inside the sixteen (through LDS, and with T0's value read where the cell needs it, 0.03 us a step
                    // more).
                    o += b_pred;
                    q = (s4f){solo_dpp<0x150>(o), solo_dpp<0x154>(o), solo_dpp<0x158>(o), solo_dpp<0x15c>(o)};
                    asm volatile("" : "+v"(pv));
                }
            } else {
                if (pending) {
                    frames_there();
                    pending = false;
                    __syncthreads();
                }
                if (chain) pv = frame_values();
            }
            // joint step: frames t .. t + 15, a quarter of K per wave
            ++n_joint;
            const int left = len - t;
            n_samples += min(left, NF);
            if (chain) {
                const int m16 = lane & 15, g = lane >> 4;
                s4f sum[TILES];
                float last_sum = 0.f;
#pragma unroll
                for (int o = 0; o < TILES; ++o) sum[o] = (s4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float z = fmaxf(pv[e] + q[e], 0.f);
#pragma unroll
                    for (int o = 0; o < TILES; ++o) sum[o] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[4 + o][e], z, sum[o], 0, 0, 0);
                    if (LAST) last_sum = fmaf(w[4 + TILES][e], z, last_sum);
                }
                if (LAST) lds[lo.last + m16 * kSoloLastRow + wave * 4 + g] = last_sum;
#pragma unroll
                for (int o = 0; o < TILES; ++o) *reinterpret_cast<s4f *>(part + (wave * NF + m16) * PS + o * 16 + g * 4) = sum[o];
            } else if (need) {
                // W_hh h, in eight sums: a lane reads four of h's values and has the others from its fifteen neighbours (all 64 values read
                // by every lane keep the LDS from the projection's reads: 0.5 to 0.8 % of a call, with the frames' read moved up)
                float x[4];
                s4f acc[2];
#pragma unroll
                for (int i = 0; i < 4; ++i) x[i] = hv[i * 16 + (lane & 15)];
                acc[0] = acc[1] = (s4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    fma_row8<0>(w + i * 4, x[i], acc);
                    fma_row8<8>(w + i * 4 + 2, x[i], acc);
                }
                const s4f a = acc[0] + acc[1];
                pre = (a[0] + a[1]) + (a[2] + a[3]);
            }
            __syncthreads();
            if (chain) {
                // sixteen lanes per frame, TILES outputs each
                struct __align__(TILES % 2 ? 4 : 4 * TILES) Outs { float of[TILES]; };
                const int s = t256 >> 4, l = lane & 15, first = l * TILES;
                Outs o[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = *reinterpret_cast<const Outs *>(part + (i * NF + s) * PS + first);
                float v[TILES], mine = -INFINITY;
#pragma unroll
                for (int i = 0; i < TILES; ++i) {
                    v[i] = ((o[0].of[i] + o[1].of[i]) + (o[2].of[i] + o[3].of[i])) + b_out[i];
                    mine = fmaxf(mine, first + i < p.VT ? v[i] : -INFINITY);
                }
                const float last_v = LAST ? sum16(lds[lo.last + s * kSoloLastRow + l]) + b_last : -INFINITY;
                // the lowest of equal outputs (none: they are all NaN, and a frame with nothing else is a blank)
                int k = -1;
#pragma unroll
                for (int i = TILES - 1; i >= 0; --i) k = first + i < p.VT && v[i] == mine ? first + i : k;
                float m = max16(mine);
                const unsigned hit = (unsigned)(__ballot(mine == m && k >= 0) >> (lane & 48)) & 0xffffu;
                const int lead = hit ? __builtin_ctz(hit) : 0;
                int best = hit ? k : p.blank;
                if (LAST) {
                    const bool above = last_v > m || (hit == 0u && last_v == m);
                    best = above ? TILES * 16 : best;
                    m = above ? last_v : m;
                }
                if (l == lead) *reinterpret_cast<int2 *>(res + s * 2) = make_int2(best, __float_as_int(m + 0.0f));
                if (tdt) {
                    float dm = -INFINITY;
#pragma unroll
                    for (int i = 0; i < TILES; ++i) dm = fmaxf(dm, first + i >= p.VT && first + i < p.NOUT ? v[i] : -INFINITY);
                    const float top = max16(dm);
                    int d = -1;
#pragma unroll
                    for (int i = TILES - 1; i >= 0; --i) d = first + i >= p.VT && first + i < p.NOUT && v[i] == top ? first + i : d;
                    const unsigned dhit = (unsigned)(__ballot(dm == top && d >= 0) >> (lane & 48)) & 0xffffu;
                    const int dlead = dhit ? __builtin_ctz(dhit) : 0;
                    // (the first one where all are NaN)
                    if (l == dlead) res_d[s] = durations[dhit ? min(d - p.VT, kMaxDur - 1) : 0];
                }
                if (p.logps) {
                    float e = 0.f;
#pragma unroll
                    for (int i = 0; i < TILES; ++i) e += first + i < p.VT && v[i] > -INFINITY ? expf(v[i] - m) : 0.f;
                    e = sum16(e);
                    if (LAST) e += last_v > -INFINITY ? expf(last_v - m) : 0.f;
                    if (l == 0) res_lp[s] = -logf(e);
                }
            }
            __syncthreads();
            // loop control, uniform
            const int2 got = *reinterpret_cast<const int2 *>(res + (lane & (NF - 1)) * 2);
            const int mine = got.x, dur = tdt ? res_d[lane & (NF - 1)] : 0;
            int pos = 0;
            bool found = false;
            if constexpr (!WALK) {
                const unsigned labels = (unsigned)__ballot(mine != p.blank) & 0xffffu;
                const int avail = min(left, NF);
                pos = __builtin_ctz(labels | 1u << avail);
                found = pos < avail;
            } else {
                while (pos < NF && pos < left) {
                    const int k = __builtin_amdgcn_readlane(mine, pos);
                    if (k != p.blank && k < p.V1) { found = true; break; }
                    pos += max(k >= p.V1 ? __builtin_amdgcn_readfirstlane(durations[(k - p.V1) & (kMaxDur - 1)]) : (tdt ? min(__builtin_amdgcn_readlane(dur, pos), kFarthest) : 1), 1);
                }
            }
            int adv = pos;
            if (adv > 0) n = 0;
            if (found) {
                const int k = __builtin_amdgcn_readlane(mine, pos), d = tdt ? __builtin_amdgcn_readlane(dur, pos) : 0;
                last = k;
                // (asked for here, it is there when the rest of the loop control is done)
                t0 = lds[lo.t0 + last * (4 * W) + t256];
                if (writer) {
                    if (cnt < p.cap) {
                        const long long o = (long long)b * p.cap + cnt;
                        p.tokens[o] = k;
                        if (p.frames) p.frames[o] = t + pos;
                        if (p.logits) p.logits[o] = __int_as_float(__builtin_amdgcn_readlane(got.y, pos));
                        if (p.logps) p.logps[o] = res_lp[pos];
                        if (p.durs) p.durs[o] = d;
                    } else {
                        flags |= 2;
                    }
                }
                ++cnt;
                if (tdt && d > 0) { adv += min(d, kFarthest); n = 0; }
                else if (++n == p.S) { ++adv; n = 0; }
            }
            t = adv >= left ? len : t + adv;
            need = found;
            // the chunks of frames t and after
            if (t < len) {
                const int at = t / kSoloChunk;
                for (int i = max(have + 1, at); i <= at + 1; ++i) { load_chunk(b, len, i); have = i; pending = true; }
            }
        }
        if (writer) {
            p.tok_len[b] = cnt;
            if (p.done) __hip_atomic_store(p.done + b, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    if (writer) {
        if (flags) __hip_atomic_fetch_or(p.status, flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        long long *s = p.stats + (long long)blockIdx.x * kStatStride;
        s[kStatPred] = n_pred; s[kStatJoint] = n_joint; s[kStatSamples] = n_samples; s[kStatPolls] = 0;
        atomicMax(reinterpret_cast<unsigned long long *>(p.stats + kStatDecodeEnd), (unsigned long long)wall_clock64());
    }
}

template <int TILES, bool LAST, bool WALK>
hipError_t launch_tiles(const SoloParams &p, bool plain, hipStream_t stream, hipEvent_t end)
{
    const void *fn = reinterpret_cast<const void *>(&solo_kernel<TILES, LAST, WALK>);
    const unsigned lds = (unsigned)solo_lds(p.V1, TILES).total * 4u;
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(solo_lds(kSoloOutputs, TILES).total * 4));
    if (e != hipSuccess) return e;
    SoloParams pc = p;
    void *args[] = {&pc};
    const dim3 grid((unsigned)(p.B < p.n_records ? p.B : p.n_records)), block(kSoloThreads);
    if (plain) return launch_ending(fn, grid, block, args, lds, stream, end);
    return hipLaunchCooperativeKernel(fn, grid, block, args, lds, stream);
}

}  // namespace

hipError_t pack_solo(const float *w_hh, const float *w_pred, const float *w_out, int H, int J, int NOUT, int VT, float4 *w, unsigned *check, hipStream_t stream)
{
    const int n = solo_parts(NOUT, VT) * 256;
    hipLaunchKernelGGL(pack_solo_kernel, dim3((unsigned)(n / 256)), dim3(256), 0, stream, w_hh, w_pred, w_out, H, J, NOUT, solo_tiles(NOUT, VT), n, w, check);
    return hipGetLastError();
}

hipError_t launch_solo(const SoloParams &p, bool plain, hipStream_t stream, hipEvent_t end)
{
    // what the kernel is laid out for
    if (p.H < 1 || p.H > kSoloWidth || p.J < 1 || p.J > kSoloWidth || p.J % 4 != 0 || p.NOUT > kSoloOutputs || p.V1 > p.NOUT || p.B < 1 || p.n_records < 1)
        return hipErrorInvalidValue;
    const bool walk = p.tdt || p.VT != p.V1;
    auto launch = [&](auto tiles, auto last) {
        return walk ? launch_tiles<decltype(tiles)::value, decltype(last)::value, true>(p, plain, stream, end)
                    : launch_tiles<decltype(tiles)::value, decltype(last)::value, false>(p, plain, stream, end);
    };
    std::integral_constant<int, 1> one;
    std::integral_constant<int, 2> two;
    std::integral_constant<int, 3> three;
    const int tiles = solo_tiles(p.NOUT, p.VT);
    if (solo_last(p.NOUT, p.VT)) return tiles == 1 ? launch(one, std::true_type()) : tiles == 2 ? launch(two, std::true_type()) : launch(three, std::true_type());
    switch (tiles) {
    case 1: return launch(one, std::false_type());
    case 2: return launch(two, std::false_type());
    case 3: return launch(three, std::false_type());
    default: return launch(std::integral_constant<int, 4>(), std::false_type());
    }
}

}  // namespace rnnt
