// Decode kernel with register-resident weights (device code, instantiated by resident_inst.hip).
//
// The step chain of a decode (a prediction step, a joint step, and again) is bound by latency:
// three dense stages and four hand-overs between work-groups per label.  Two things make it
// short here.  (1) Every weight of the step is held in the registers of one compute unit for the
// whole launch: eight waves of 256 registers, of which up to 190 hold weights, so a stage reads
// nothing but its input vector (streamed out of L2, the weights took 5 to 27 us of a step).  (2) A team
// of work-groups sits inside one XCD, so its hand-overs go through that XCD's L2: a store that stays
// in the L2 and a load that passes by the L1 hand 640 floats to 32 work-groups in 0.70 us, where
// stores and loads through the memory side take 1.3 us (4 x 640 floats: 0.88 against 1.4 us).
// 32 utterances of a two-layer model of 640 units: 4.35 ms in the kernel that streams its weights, 1.14 here, one of 500
// frames 1.63 and 0.41.
//
// Work split inside a team of `ts` work-groups: LSTM units, projection columns and output columns
// in contiguous ranges.  Every dense stage is the same: K in eighths over the waves, tiles of 16 outputs
// (the gates of four units, or columns) by 16 columns of the operand on v_mfma 16x16x32, and the waves' partial sums
// meet in LDS.  Columns of the LSTM stages and the projection are the team's utterances, those of the joint output are samples.
// A wave receives its eighth of an operand straight into registers (Operand; the joint's: ask_z).
//
// A team decodes four utterances at a time, or eight where its list has as many (resident_rows): two parts of eight rows are the sixteen
// columns that the matrix instructions of the LSTM stages and the projection have in any case, so a prediction step of eight takes 0.4 us more
// than one of four; four frames of every row in a joint step where there were eight, but the longest of six teams of 128 utterances takes 433 joint steps instead
// of 567 (200 to 500 frames, the sweep's draw).
//
// The joint's operand z = relu(P + q) is formed once in the team: every work-group has its own columns of the projection, adds
// those of the samples' frames (80 bytes a sample) and hands z on in q's place.  Formed from q by every work-group for itself it took
// nine vector instructions for two values and two LDS reads, 32 times over, and the samples' whole frames in LDS, 80 KB.  What
// bounds the hand-over is the size: a compute unit takes 8 KB in 0.11 us (32 of them the same 8 KB of an XCD's L2), 16 fp32 samples of
// 640 in 0.94 us where q of four utterances takes 0.75.  So 32 samples go to a work-group as one tile of 16, for its own
// and its partner's columns (`half`): as two tiles, for its own columns alone, they took longer than q did (32 utterances 1208 us with
// q, 1249, and 1160 with half; partners' weights in the frames' place in LDS).  Against q handed on: 32 utterances (three draws) 1083, 1318, 1359 us and
// 1037, 1264, 1303, bfloat16 mode 850, 925, 925 and 777, 846, 843, 128 utterances 3967 and 3808, one 281 and 278, the small model 344 and 320.
//
// fp32 values run on the 16-bit matrix instructions as two fp16 parts each, weights and vectors alike: 23 bits,
// all four products (the joint of the widest class: three, see there), fp32 sums.  On the fp32 instructions a step's stages were
// bound by the matrix pipe, which they share with everything else: a 4x4 one per row group and 32 k's, 16x16x4 in
// the joint step.  A joint step of 32 utterances 9.7 to 8.8 us, of one utterance 7.8 to 6.6, of a model of the
// narrowest class 4.2 to 4.0 (with phase timers).
//
// Two-layer fp32 models have more weights than one XCD's registers hold (24 MB against 12 + 4):
// there six XCDs with a team each keep the input, projection and output matrices and run the whole step chain;
// two XCDs of helpers, one for either layer, keep the recurrent matrices and compute W_hh h of the candidate states,
// which the chain needs only at the next label: their hand-overs across the XCDs, 1.2 us each way, run beside the rest
// of the step.
//
// Utterances are decoded label-looping fashion: every utterance has its own frame index, a joint
// step examines `la` frames of every utterance in work (16 or 32 in all; half as many in label-dense stretches of two-layer
// fp32 models, see the end of the loop), and the next prediction step runs as soon as one
// of them has a label, or a little later (see the loop control).  A team takes a list of utterances and decodes up to R at a time;
// when one ends the next of the list takes its place, or, if there is none, the others get its frames.
//
// Exchange: a vector's buffer has four slots used in turn; words are 32-bit floats, all ones
// meaning "not there yet" (readers poll the data itself).  A work-group puts that mark back into
// slot n - 2 when it publishes step n: by then it has received something of step n - 1 from
// everyone, which everyone sent after reading step n - 2; and it waits for that store before it
// publishes step n + 1, so nobody can look for step n + 2's data in a slot that still holds old data.
// (No wait for the store as such: a wave's loads and stores are counted in the order they were issued in, and every wave
// polls for a vector, or waits for its frames, behind its stores of a step and ahead of the barrier that its
// work-group's next words of that kind come after.  A wave that skips such a poll needs a wait in its place.)
//
// Registers decide what the code looks like: values that could be kept for the whole loop are worked out
// where they are used (lane_id), state that few waves need lies in LDS, arguments that few steps need are
// read again (args_again).  A spilled weight is a load from memory in the middle of a stage.
#pragma once
#include <type_traits>

#include "engine.h"
#include "gate.h"
#include "parts.h"
#include "resident.h"

namespace rnnt {
namespace {

typedef float r4f __attribute__((ext_vector_type(4)));
typedef unsigned r4u __attribute__((ext_vector_type(4)));
typedef unsigned r2u __attribute__((ext_vector_type(2)));
typedef short r4s __attribute__((ext_vector_type(4)));
typedef __bf16 r8b __attribute__((ext_vector_type(8)));
typedef _Float16 r8h __attribute__((ext_vector_type(8)));
typedef _Float16 r4h __attribute__((ext_vector_type(4)));

constexpr unsigned kMark = 0xffffffffu;    // no data yet

constexpr unsigned kStop = 0xfffffffeu;    // to the helpers: the team is done

// Rows in work: every wave keeps a copy of its own and takes the same decisions from the same
// results, so loop control needs no work-group barrier.
struct __align__(16) RRow { int t, len, n, cnt; };       // frame, frames, labels of this frame, labels; t >= len: idle
// (Tables of eight places: with four, 128 bytes from wave to wave instead of 240, the small model's calls took 2 % longer.)
struct RRows {
    static constexpr int kPlaces = 8;
    static_assert(kResRows <= kPlaces, "a place for every row");
    RRow s[kPlaces];
    int b[kPlaces];                   // utterance
    int since[kPlaces], next;         // t some steps ago; first utterance of the list that no row has had
};

// Columns that the waves forming the joint's operand have lanes for, in steps of one tile: a work-group has 20 at most, and these lanes read what
// they do not send (limited to the 20, the index took a register that the weights need).
constexpr int kResFormed = 40;

struct RCtl {
    RRows rows[kResWaves];
    int s_k[kResSamples], s_d[kResSamples];        // results of a joint step
    float s_v[kResSamples], s_lp[kResSamples];
    int n_list, ok, st_clamped, st_overflow;
    int dur[kMaxDur];
    unsigned seen[2][kResWaves];      // helpers: what a wave has seen of the teams' vectors
    unsigned short list_b[kResList];
    int list_len[kResList];
    // this work-group's slices of the biases: second layer [unit][gate], projection, output and tail column; and of
    // what sums are multiplied by (fp32): the same and [layer][unit][gate] of the recurrent matrices
    float b1[kResUnits * 4], s1[kResUnits * 4], sh[2][kResUnits * 4];
    __align__(16) float bp[kResFormed], sp[kResFormed];
    float2 bo[2][16], so[2][16];      // with two tiles of samples: of this work-group and its partner, the even rank first
    float bt[2], st[2];
    float scale[RRows::kPlaces];      // fp32: of the utterances in work, see joint_scale
};
__shared__ RCtl rc;
static_assert(sizeof(RCtl) + 256 <= kResCtl, "the control block has its place, and what the compiler keeps for votes of a work-group");

// Phase timers (100 MHz wall clock), compiled in only for profiling builds.
#ifdef RNNT_PROFILE
__shared__ long long res_prof[24];
__shared__ long long res_prof_last;
#define RES_MARK(slot) do { __builtin_amdgcn_sched_barrier(0); if (threadIdx.x == 0) { long long t_ = wall_clock64(); res_prof[slot] += t_ - res_prof_last; res_prof_last = t_; } __builtin_amdgcn_sched_barrier(0); } while (0)
#else
#define RES_MARK(slot) do { } while (0)
#endif

// Weights: in groups of four registers, as the matrix instructions take them (half blocks: two groups of two).
typedef float r2f __attribute__((ext_vector_type(2)));
template <int N> struct RegW {
    r4f q[N / 4];
    r2f rest;                         // N % 4 == 2
};
// A wave's loads of weights all go out before the first is waited for, sixteen bytes at a time: 8.0 us of a launch of the largest
// class (12.4 in single words, 32 in flight).
// PAIRS: eight bytes at a time, as relaxed atomics that are not put together again.  For bf16 with two recurrent layers, whose
// registers are full: groups of four from one load left it 8 that are written out and read back in every step (one utterance:
// 2.5 % of a call).
__device__ __forceinline__ float load_one(const float *at) { return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT); }
__device__ __forceinline__ r2f load_pair(const float *at)
{
    return __builtin_bit_cast(r2f, __hip_atomic_load(reinterpret_cast<const long long *>(at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT));
}
// Asks for registers [first, first + N) of the wave's packed run, see res_place.
template <bool PAIRS, int N>
__device__ __forceinline__ void load_regs(RegW<N> &r, const float *src, int first, int lane)
{
    static_assert(N % 2 == 0, "pairs");
    src += first * 64;
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
        const float *at = src + i * 256 + lane * 4;
        if constexpr (PAIRS) {
            const r2f a = load_pair(at), b = load_pair(at + 2);
            r.q[i] = (r4f){a.x, a.y, b.x, b.y};
        } else r.q[i] = *reinterpret_cast<const r4f *>(at);
    }
    if (N % 4) {
        const float *at = src + N / 4 * 256 + lane * 2;
        if constexpr (PAIRS) r.rest = (r2f){load_one(at), load_one(at + 1)};
        else r.rest = *reinterpret_cast<const r2f *>(at);
    }
}
// The empty asm makes each value opaque, so that it stays in its registers and is never read from memory again.
template <int N>
__device__ __forceinline__ void keep_regs(RegW<N> &r)
{
#pragma unroll
    for (int i = 0; i < N / 4; ++i) asm volatile("" : "+v"(r.q[i]));
    if (N % 4) asm volatile("" : "+v"(r.rest));
}

// The lane's number, worked out anew wherever it is used: a register that holds it, or anything that
// the compiler could work out ahead from it, is one that the weights do not get.
__device__ __forceinline__ int lane_id()
{
    unsigned zero = 0;
    asm volatile("" : "+s"(zero));
    return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
}

struct RCtx {
    int wave, rank;
    bool local;                       // every work-group of the team sits on the same XCD
    __amdgpu_buffer_rsrc_t buf;       // the team's exchange buffers
    int polls;
};

// The mark, in a register only where it is stored: constants of two and four words took six registers for the whole loop.
__device__ __forceinline__ unsigned mark_here()
{
    unsigned m;
    asm volatile("v_mov_b32 %0, -1" : "=v"(m));
    return m;
}
// A word for the team, and the mark into the slot that everyone has read (byte offsets `now` and `old` of
// the slots): stores that stay in the XCD's L2, or go through to the memory side (sc1).
__device__ __forceinline__ void put(const RCtx &x, unsigned off, unsigned now, unsigned old, unsigned v)
{
    if (x.local) {
        __builtin_amdgcn_raw_buffer_store_b32(v, x.buf, (int)off, (int)now, 0);
        __builtin_amdgcn_raw_buffer_store_b32(kMark, x.buf, (int)off, (int)old, 0);
    } else {
        __builtin_amdgcn_raw_buffer_store_b32(v, x.buf, (int)off, (int)now, 16);
        __builtin_amdgcn_raw_buffer_store_b32(kMark, x.buf, (int)off, (int)old, 16);
    }
}
__device__ __forceinline__ void put2(const RCtx &x, unsigned off, unsigned now, unsigned old, r2u v)
{
    const unsigned m = mark_here();
    const r2u mark = {m, m};
    if (x.local) {
        __builtin_amdgcn_raw_buffer_store_b64(v, x.buf, (int)off, (int)now, 0);
        __builtin_amdgcn_raw_buffer_store_b64(mark, x.buf, (int)off, (int)old, 0);
    } else {
        __builtin_amdgcn_raw_buffer_store_b64(v, x.buf, (int)off, (int)now, 16);
        __builtin_amdgcn_raw_buffer_store_b64(mark, x.buf, (int)off, (int)old, 16);
    }
}
__device__ __forceinline__ void put_mark(const RCtx &x, unsigned off, unsigned old)
{
    if (x.local) __builtin_amdgcn_raw_buffer_store_b32(kMark, x.buf, (int)off, (int)old, 0);
    else __builtin_amdgcn_raw_buffer_store_b32(kMark, x.buf, (int)off, (int)old, 16);
}
__device__ __forceinline__ void put_mark2(const RCtx &x, unsigned off, unsigned old)
{
    const unsigned m = mark_here();
    const r2u mark = {m, m};
    if (x.local) __builtin_amdgcn_raw_buffer_store_b64(mark, x.buf, (int)off, (int)old, 0);
    else __builtin_amdgcn_raw_buffer_store_b64(mark, x.buf, (int)off, (int)old, 16);
}
__device__ __forceinline__ void put_far(const RCtx &x, unsigned off, unsigned imm, unsigned v)
{
    __builtin_amdgcn_raw_buffer_store_b32(v, x.buf, (int)off, (int)imm, 16);
}
// loads past the L1 (sc1)
__device__ __forceinline__ r4u get4(const RCtx &x, unsigned off, unsigned imm)
{
    return __builtin_bit_cast(r4u, __builtin_amdgcn_raw_buffer_load_b128(x.buf, (int)off, (int)imm, 16));
}
__device__ __forceinline__ r2u get2(const RCtx &x, unsigned off, unsigned imm)
{
    return __builtin_bit_cast(r2u, __builtin_amdgcn_raw_buffer_load_b64(x.buf, (int)off, (int)imm, 16));
}
__device__ __forceinline__ unsigned get1(const RCtx &x, unsigned off, unsigned imm)
{
    return __builtin_amdgcn_raw_buffer_load_b32(x.buf, (int)off, (int)imm, 16);
}
// a float as it travels: the two bit patterns with a meaning become the ordinary NaN
__device__ __forceinline__ unsigned word_of(float v)
{
    const unsigned u = __float_as_uint(v);
    return u >= kStop ? 0x7fc00000u : u;
}

// One more poll of a wait has failed; true when the wait has to give up.
__device__ __forceinline__ bool wait_expired(const ResidentParams &p, unsigned &spins)
{
    asm volatile("" ::: "memory");
    ++spins;
    if ((spins & 127u) == 0 && __hip_atomic_load(p.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return true;
    if (spins > p.spin_limit) {
        __hip_atomic_store(p.abort_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    }
    return false;
}

__device__ __forceinline__ bool has_mark(r4u v) { return max(max(v.x, v.y), max(v.z, v.w)) == kMark; }

// N 16-byte pieces per thread: all loads in flight together, all of them again while a lane of the
// wave misses a word.
template <int N>
__device__ __forceinline__ void receive(const ResidentParams &p, RCtx &x, const unsigned (&off)[N], unsigned imm, r4u (&v)[N], bool takes = true)
{
    unsigned spins = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = (r4u){0u, 0u, 0u, 0u};
    for (;;) {
        bool missing = false;
        if (takes) {
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] = get4(x, off[i], imm);
#pragma unroll
            for (int i = 0; i < N; ++i) missing = missing || has_mark(v[i]);
        }
        if (__ballot(missing) == 0ull) break;
        if (wait_expired(p, spins)) { rc.ok = 0; break; }
    }
    x.polls += __builtin_amdgcn_readfirstlane((int)spins);
}
// The same with the first loads ahead of what is done meanwhile.
template <int N>
__device__ __forceinline__ void request(const RCtx &x, const unsigned (&off)[N], unsigned imm, r4u (&v)[N], bool takes = true)
{
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = (r4u){0u, 0u, 0u, 0u};
    if (takes) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = get4(x, off[i], imm);
    }
}
template <int N>
__device__ __forceinline__ void receive_rest(const ResidentParams &p, RCtx &x, const unsigned (&off)[N], unsigned imm, r4u (&v)[N], bool takes = true)
{
    bool missing = false;
#pragma unroll
    for (int i = 0; i < N; ++i) missing = missing || has_mark(v[i]);
    if (__ballot(missing) == 0ull) return;
    ++x.polls;
    receive<N>(p, x, off, imm, v, takes);
}

template <int CTRL>
__device__ __forceinline__ float dppf(float v)
{
    return __uint_as_float((unsigned)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), CTRL, 0xf, 0xf, true));
}
// maximum over groups of 2, 4, 8 or 16 adjacent lanes (one instruction a step; fmaxf of a permuted value
// takes three)
template <int LANES>
__device__ __forceinline__ float lane_max(float v)
{
    asm("s_nop 1\n\tv_max_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf" : "+v"(v));
    if (LANES > 2) asm("s_nop 1\n\tv_max_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf" : "+v"(v));
    if (LANES > 4) asm("s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf" : "+v"(v));
    if (LANES > 8) asm("s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf" : "+v"(v));
    return v;
}
template <int LANES>
__device__ __forceinline__ float lane_sum(float v)
{
    v += dppf<0xB1>(v);
    if (LANES > 2) v += dppf<0x4E>(v);
    if (LANES > 4) v += dppf<0x141>(v);
    if (LANES > 8) v += dppf<0x140>(v);
    return v;
}

// Matrix instruction on a block of a wave's share of K: `w` and `z` from the registers of that block on, four
// of either (32 k's), two for a half block (bfloat16 mode).  A matrix instruction that adds to what one of the other kind right
// before it leaves gives wrong sums (the compiler places no wait between them): where a sum takes both kinds, the
// half block comes first and a wait after it, of 32 cycles or for a read of the sum (there; ordered: nothing moves
// across), or it is two sums.
template <bool BF>
__device__ __forceinline__ r4f tile_mfma(r4f w, const unsigned *z, r4f acc)
{
    const r4u zv = {z[0], z[1], z[2], z[3]};
    if constexpr (BF) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(r8b, w), __builtin_bit_cast(r8b, zv), acc, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(r8h, w), __builtin_bit_cast(r8h, zv), acc, 0, 0, 0);
}
// fp32 values, of a half block
__device__ __forceinline__ r4f whole_mfma(r4f w, const unsigned *z, r4f acc)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[e], __uint_as_float(z[e]), acc, 0, 0, 0);
    return acc;
}
template <bool BF>
__device__ __forceinline__ r4f tile_mfma(r2f w, const unsigned *z, r4f acc)
{
    const r2u zv = {z[0], z[1]};
    if constexpr (BF) return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(r4s, w), __builtin_bit_cast(r4s, zv), acc, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(r4h, w), __builtin_bit_cast(r4h, zv), acc, 0, 0, 0);
}
// the weights of block kb of tile t
template <bool BF, int CLS, int T, int KB, int PART, int N>
__device__ __forceinline__ auto weights_of(const RegW<N> &w, int t)
{
    const int at = res_tile_at(BF, CLS, T, KB, t, PART);
    if constexpr (KB < res_halves(CLS) / 2) return w.q[at / 4];
    else return at / 4 == N / 4 ? w.rest : (at % 4 ? w.q[at / 4].zw : w.q[at / 4].xy);
}

// fp32: both parts of the half block's weights, the high ones first, as one instruction takes them that multiplies both: the
// operand's sixteen k's twice.  (A half block's own instruction takes as long as a whole block's, one for each part, and waits between the
// two kinds: 32 utterances 1185 us, 1169 with this, one layer 899 and 880, the small model 278 and 271, 128 utterances 3017 and 2997.)
// An instruction aligns its products with the largest of them, so the small ones lose bits beside large ones.  In the joint step the products
// with one low part have an instruction of their own, and low times low, which is nothing, goes with high times high.  In the projection of the
// classes with no more than one whole block beside the half one, low and high parts of the weights have an instruction each, by zeros in
// the other's place (stage, TWO).  Logits from 64 bits, against half blocks with instructions of their own, means of 60 to 80 models: layers of 320
// +0.24 % (+-0.07) with low beside high parts in all stages, +0.01 % (+-0.07) as it is (eight utterances 0.9 % longer; the recurrent stage in two as well -0.10 %,
// 1.8 % longer), layers of 128 +0.50 and -0.38 % (+-0.2), of 640 +0.02 and -0.01 % (+-0.05).
template <int CLS, int T, int N>
__device__ __forceinline__ r4f both_parts(const RegW<N> &w, int t) { return w.q[res_tile_at(false, CLS, T, res_halves(CLS) / 2, t, 0) / 4]; }

__device__ __forceinline__ void ordered() { __builtin_amdgcn_sched_barrier(0); }

// Reads a matrix instruction's result: the compiler places what wait that needs after the instruction, if any.
__device__ __forceinline__ void there(r4f sum)
{
    const int v = __builtin_amdgcn_readfirstlane((int)__float_as_uint(sum.x));
    asm volatile("" :: "s"(v));
}

// compile-time loop: f(std::integral_constant<int, I>) for I = LO .. HI - 1
template <int LO, int HI, class F>
__device__ __forceinline__ void static_for(F f)
{
    if constexpr (LO < HI) {
        f(std::integral_constant<int, LO>());
        static_for<LO + 1, HI>(f);
    }
}

// Hidden values as they travel, one word each: fp16 parts of 2^15 times the value (high in the low half), or bf16.
template <bool BF>
__device__ __forceinline__ unsigned hidden_word(float h)
{
    if (BF) return bf16_pair(h, 0.f);
    unsigned high, low;
    h *= (float)(1 << kResHiddenExp);
    f16_parts(h, h, high, low);
    const unsigned u = __builtin_amdgcn_perm(low, high, 0x05040100u);
    return u >= kStop ? 0x7e007e00u : u;
}

// The operand of a dense stage: the wave's eighth of K of the rows' hidden values, columns 0 .. 15 of the matrix
// instructions.  R rows take R columns; fp32: R with the high parts are followed by R with the low ones, so a product
// with the weights' high and one with their low parts give all four (the columns beyond are nobody's).  A lane loads four words of a block, exchanges halves with the lane R columns on (whose words are the
// block's other four of the same row and group), and has what the instruction takes: nothing of it
// goes through LDS, and a wave goes on as soon as its own eighth is there.
template <bool BF, int CLS, int R>
struct Operand {
    static_assert(R == 4 || R == 8, "two parts of every row are 8 or 16 columns");
    static constexpr int NH = res_halves(CLS), NF = NH / 2, NB = NF + (NH & 1);
    unsigned z[NH * 2];
    // words of block i for the lane: byte offset in a vector of rows of `W` words; n4 pieces of four words a row, the
    // last one stands for those beyond (their weights are zeros)
    static __device__ __forceinline__ unsigned offset(int i, int wave, int lane, int n4)
    {
        const int n = lane & 15, g = lane >> 4, other = (n / R) & 1, row = n & (R - 1);
        const int k4 = wave * (NH * 4) + i * 8 + (i < NF ? 2 * g + other : g);
        return (unsigned)(row * (res_width(CLS) * 4)) + (unsigned)min(k4, n4 - 1) * 16u;
    }
    __device__ __forceinline__ void set(const r4u (&v)[NB], int lane)
    {
        const bool other = ((lane & 15) / R) & 1;
        const unsigned keep = !BF && other ? 0x07060302u : 0x05040100u, send = !BF && !other ? 0x07060302u : 0x05040100u;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const unsigned k0 = __builtin_amdgcn_perm(v[i].y, v[i].x, keep), k1 = __builtin_amdgcn_perm(v[i].w, v[i].z, keep);
            if (i < NF) {
                const unsigned s0 = __builtin_amdgcn_perm(v[i].y, v[i].x, send), s1 = __builtin_amdgcn_perm(v[i].w, v[i].z, send);
                constexpr int UP = 0x110 + R, DOWN = 0x100 + R, FIRST = (1 << (R / 4)) - 1, SECOND = FIRST << (R / 4);       // banks of four lanes
                z[i * 4] = (unsigned)__builtin_amdgcn_update_dpp((int)k0, (int)s0, UP, 0xf, SECOND, false);
                z[i * 4 + 1] = (unsigned)__builtin_amdgcn_update_dpp((int)k1, (int)s1, UP, 0xf, SECOND, false);
                z[i * 4 + 2] = (unsigned)__builtin_amdgcn_update_dpp((int)k0, (int)s0, DOWN, 0xf, FIRST, false);
                z[i * 4 + 3] = (unsigned)__builtin_amdgcn_update_dpp((int)k1, (int)s1, DOWN, 0xf, FIRST, false);
            } else {
                z[i * 4] = k0; z[i * 4 + 1] = k1;
            }
        }
    }
    __device__ __forceinline__ void receive_from(const ResidentParams &p, RCtx &x, unsigned base, int n4, unsigned long long take)       // take: res_takers
    {
        unsigned off[NB];
        r4u v[NB];
        const int lane = lane_id();
#pragma unroll
        for (int i = 0; i < NB; ++i) off[i] = offset(i, x.wave, lane, n4);
        receive<NB>(p, x, off, base, v, __builtin_amdgcn_inverse_ballot_w64(take));
        set(v, lane);
    }
};

// A dense stage with T tiles of 16 outputs: the sums over the wave's eighth of K go to LDS, [wave][row][ROW floats].
// fp32: the products with the weights' low parts come before the others, to be added at their own size.
// behind(): done while the matrix instructions end.
struct Nothing { __device__ __forceinline__ void operator()() const {} };
template <bool BF, int CLS, int R, int T, int ROW, class F = Nothing>
__device__ __forceinline__ void stage(const RegW<res_tile_regs(BF, CLS, T)> &w, const Operand<BF, CLS, R> &x, float *sums, int wave, F behind = F())
{
    constexpr int NH = res_halves(CLS), NF = NH / 2;
    constexpr bool MIXED = BF && NF > 0 && NH % 2 != 0, APART = MIXED && T < 4;
    r4f sum[T], half[T];
#pragma unroll
    for (int t = 0; t < T; ++t) sum[t] = half[t] = (r4f){0.f, 0.f, 0.f, 0.f};
    auto block = [&](auto kb_, auto part_) {
        constexpr int kb = decltype(kb_)::value, part = decltype(part_)::value;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            r4f &to = APART && kb == NF ? half[t] : sum[t];
            to = tile_mfma<BF>(weights_of<BF, CLS, T, kb, part>(w, t), x.z + kb * 4, to);
        }
    };
    std::integral_constant<int, NF> last;
    std::integral_constant<int, 0> high;
    std::integral_constant<int, 1> low;
    if constexpr (BF && NH % 2 != 0) {
        block(last, high);
        if constexpr (MIXED && !APART) {
            ordered();
#pragma unroll
            for (int t = 0; t < T; ++t) asm volatile("" : "+v"(sum[t]));
            asm volatile("s_nop 15\n\ts_nop 15");
            ordered();
        }
    }
    if constexpr (!BF) {
        static_for<0, NF>([&](auto kb_) { block(kb_, low); });
        if constexpr (NH % 2 != 0) {
            constexpr bool TWO = NF < 2 && T == 2;
            const unsigned z0 = x.z[NF * 4], z1 = x.z[NF * 4 + 1];
            const unsigned low_only[4] = {0u, 0u, z0, z1}, high_only[4] = {z0, z1, 0u, 0u}, both[4] = {z0, z1, z0, z1};
            if constexpr (TWO) {
#pragma unroll
                for (int t = 0; t < T; ++t) sum[t] = tile_mfma<BF>(both_parts<CLS, T>(w, t), low_only, sum[t]);
            }
#pragma unroll
            for (int t = 0; t < T; ++t) sum[t] = tile_mfma<BF>(both_parts<CLS, T>(w, t), TWO ? high_only : both, sum[t]);
        }
    }
    static_for<0, NF>([&](auto kb_) { block(kb_, high); });
    behind();
    const int lane = lane_id(), n = lane & 15;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        r4f v = sum[t];
        if constexpr (APART) v += half[t];
        if (!BF) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] += dppf<0x100 + R>(v[i]);
        }
        if (n < R && (t * 16 + 16 <= ROW || t * 16 + (lane >> 4) * 4 < ROW)) *reinterpret_cast<r4f *>(sums + (wave * R + n) * ROW + t * 16 + (lane >> 4) * 4) = v;
    }
}

// What a lane finishes in the LSTM stages, waves 0 .. 4: of unit 4 wave + lane / 16 and row lane / LR % R (LR = 16 / R lanes a row), gate
// lane % 4 (four rows), or two gates from 2 * (lane % 2) on (eight rows).
template <int R> struct RGates {
    static constexpr int N = R / 4;
    float g[N];
};
// Its sums over the waves:
template <int R>
__device__ __forceinline__ RGates<R> stage_sum(const float *sums, int blk, int lane)
{
    constexpr int LR = 16 / R, N = RGates<R>::N, ROW = res_stage_row(R);
    typedef float Group __attribute__((ext_vector_type(N)));
    const float *s = sums + ((unsigned)lane / LR & (R - 1)) * ROW + (blk * 4 + ((unsigned)lane >> 4)) * 4 + (lane & (LR - 1)) * N;
    Group o[kResWaves];
#pragma unroll
    for (int w = 0; w < kResWaves; ++w) o[w] = *reinterpret_cast<const Group *>(s + w * R * ROW);
    const Group sum = ((o[0] + o[1]) + (o[2] + o[3])) + ((o[4] + o[5]) + (o[6] + o[7]));
    RGates<R> v;
    if constexpr (N == 1) v.g[0] = sum[0];
    else { v.g[0] = sum[0]; v.g[1] = sum[1]; }
    return v;
}

// LSTM cell on the adjacent lanes of a unit and row: lane j of four holds the pre-activation of gate j of i, f, g, o, or lane j of
// two those of gates 2 j and 2 j + 1. Every lane gets the results.
template <int R>
__device__ __forceinline__ void cell(const RGates<R> &pre, int j, float c_old, float &c_new, float &h)
{
    float i_, f_, g_, o_;
    if constexpr (R == 4) {
        const float act = gate_act(pre.g[0], j == 2);
        i_ = dppf<0x00>(act); f_ = dppf<0x55>(act); g_ = dppf<0xAA>(act); o_ = dppf<0xFF>(act);
    } else {
        const float a = gate_act(pre.g[0], j == 1), b = gate_act(pre.g[1], false);
        i_ = dppf<0xA0>(a); f_ = dppf<0xA0>(b); g_ = dppf<0xF5>(a); o_ = dppf<0xF5>(b);          // (lanes 0, 0, 2, 2 and 1, 1, 3, 3)
    }
    c_new = fmaf(f_, c_old, i_ * g_);
    h = o_ * gate_act(c_new, true);
}

// What the prediction step does with a row's candidate state: take it, or start afresh (else nothing).
constexpr int kTake = 1 << 30, kFresh = (int)(1u << 31);

// fp32: the power of two that takes the bound max P + max q of an utterance to 2^14 .. 2^15, which its operands of the
// joint step, as they travel, are multiplied by.  (Of infinite values of P the finite ones count.)
__device__ __forceinline__ float joint_scale(TopWord top, float q_bound)
{
    const float bound = fminf(__uint_as_float((unsigned)top << 16) + q_bound, kResHuge);
    return __uint_as_float((268u << 23) - max(__float_as_uint(bound) & 0x7f800000u, 27u << 23));
}

// Where the largest operand of a sample in a lane's quarter of the wave's eighth of K has to lie for two fp16 parts to hold them
// as well as fp32 does: parts are off by 2^-25 at most, which is 2^-23 of the least one; beyond the most there are none.
constexpr float kResLeast = 0.25f, kResMost = 65504.f;
// Samples (lane % 16) that parts do not hold, of ballots of the lanes whose largest operand is below the least one (and not
// zero), not below it, and beyond the most.  One quarter in which all that is not zero is small is nothing unusual behind a
// relu; it matters where hardly anything else is there: two such, or one, and not two quarters with ordinary values.
__device__ __forceinline__ unsigned unheld(unsigned long long small, unsigned long long fine, unsigned long long beyond)
{
    auto any = [](unsigned long long m) { const unsigned b = (unsigned)m | (unsigned)(m >> 32); return b | b >> 16; };
    auto two = [](unsigned long long m) {
        const unsigned a = (unsigned)m, b = (unsigned)(m >> 32), both = a & b, one = a | b;
        return both | both >> 16 | (one & one >> 16);
    };
    return ((two(small) & ~two(fine)) | (any(small) & ~any(fine)) | any(beyond)) & 0xffffu;
}

__device__ __forceinline__ float inverse_power(float two_to_n) { return __uint_as_float(0x7f000000u - __float_as_uint(two_to_n)); }

// Byte offset of step n's slot among slots of `bytes`.  (In a scalar register by force: the compiler multiplies in a
// vector instruction and puts a loop over its lanes' values around every load and store that takes the offset.)
__device__ __forceinline__ unsigned slot_at(unsigned n, unsigned bytes)
{
    return (unsigned)__builtin_amdgcn_readfirstlane((int)((n & (kResSlots - 1)) * bytes));
}

// The kernel's arguments read again from memory: for what few waves and few steps need, and which would
// take scalar registers (and vector registers that they are spilled to) for the whole loop.
typedef const ResidentParams __attribute__((address_space(4))) *Args;
__device__ __forceinline__ Args args_again()
{
    Args a = (Args)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(a));
    return a;
}

// End of a row: outputs are written by one work-group of the team.
__device__ __forceinline__ void res_finish_row(int b, int cnt)
{
    const Args a = args_again();
    a->tok_len[b] = cnt;
    if (a->done) __hip_atomic_store(a->done + b, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ int from_lane(int v, int lane) { return __builtin_amdgcn_ds_bpermute(lane << 2, v); }

// KIND: ResidentKind; BF: bfloat16 mode; CLS: size class; NMT: tiles of 16 samples of a joint step; R: rows of a team; ONE: no team has
// more than one utterance
template <int KIND, bool BF, int CLS, int NMT, int R, bool ONE>
__global__ void __launch_bounds__(kResThreads, 1) resident_kernel(const ResidentParams p)
{
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int NL = KIND == kResident1 ? 1 : 2;
    constexpr bool PAIR = KIND == kResident2Pair;
    constexpr int W = res_width(CLS), ROW = res_row(CLS), TS = res_team(CLS);
    constexpr int NH = res_halves(CLS), NF = NH / 2, NB = NF + (NH & 1), LREGS = res_lstm_regs(BF, CLS);
    constexpr bool WHOLE = res_whole(BF, CLS);
    static_assert(!ONE || (NMT == 1 && R == 4), "sixteen frames of the one utterance");
    constexpr int LR = 16 / R, GL = R / 4, RB = R == 4 ? 2 : 3;      // lanes per row in the loop control and the cells, gates of such a lane; bits of a row's number
    constexpr int STAGE_ROW = res_stage_row(R);
    typedef Operand<BF, CLS, R> Op;
    constexpr bool HALVES = PAIR && NMT == 2;     // steps with one tile of samples as well, see after the loop
    constexpr int NREC = PAIR ? 0 : NL;          // recurrent matrices the chain's work-groups hold
    constexpr ResidentBuf bo = resident_buf(KIND, BF, CLS, R);
    constexpr ResidentLds lo = resident_lds(KIND, BF, CLS, NMT, R);
    constexpr unsigned VROW = W * 4u, VSLOT = R * VROW;                      // rows of hidden values
    constexpr unsigned ZSLOT = res_z_slot(BF, CLS), ZWAVE = res_z_wave(BF, CLS);   // the joint's operand
    constexpr int JREGS = res_joint_regs(BF, CLS);
    constexpr int ZS = 16 * NMT;                 // samples of the longest joint step
    constexpr int kFormers = 3;                  // see publish_z
    constexpr unsigned KSLOT = kResSamples * TS * 8u, DSLOT = kResSamples * kMaxDur * 4u;
    constexpr unsigned QSLOT = TS * 5u * 64u * 4u * GL, PSLOT = kResQuarters * QSLOT;         // pre-activations: a quarter of K, all

    RCtx x;
    const int tid0 = threadIdx.x, lane0 = tid0 & 63;         // (for the work before and after the loop)
    x.wave = __builtin_amdgcn_readfirstlane(tid0 >> 6);
    x.polls = 0;
    // Work-groups go to the XCDs round-robin: index % n_xcd is the XCD, index / n_xcd the place on it.
    const int n_xcd = p.pl.n_xcd, xcd = blockIdx.x % n_xcd, place = blockIdx.x / n_xcd;
    const int chain_xcds = PAIR ? res_chain_xcds(n_xcd) : n_xcd, helper_xcds = n_xcd - chain_xcds;
    const bool helper = PAIR && xcd >= chain_xcds;
    const int n_teams = p.pl.n_teams;
    x.rank = place % TS;
    if (p.zero_stats && blockIdx.x == 0 && tid0 == 0) p.stats[kStatDecodeStart] = wall_clock64();
    // utterances of a team: rank q * n_teams + m of the sorted lengths, m serpentine
    auto list_of = [&](int team) {
        int n = 0;
        for (int q = 0; q * n_teams < p.B; ++q) n += q * n_teams + ((q & 1) ? n_teams - 1 - team : team) < p.B;
        return n;
    };
    auto buffers_of = [&](int team) { return __builtin_amdgcn_make_buffer_rsrc(p.xbuf + (size_t)team * bo.bytes, 0, (int)bo.bytes, 0x00020000); };
    // This work-group's team; a helper's first.  Helpers' XCDs go in pairs, an XCD for either layer, and the teams' go
    // round the pairs.
    const int team = (helper ? (xcd - chain_xcds) / 2 : xcd) + chain_xcds * (place / TS), pairs = helper_xcds / 2;
    const int my_layer = (xcd - chain_xcds) & 1;
    auto serves = [&](int i) { return (xcd - chain_xcds) / 2 + i * pairs < chain_xcds && list_of(team + i * pairs) > 0; };
    if (!helper && list_of(team) == 0) {
        if (p.zero_stats && x.rank == 0 && tid0 < kStatCounters) p.stats[(long long)team * kStatStride + tid0] = 0;
        return;
    }
    x.buf = buffers_of(team);

    // ---- put the mark into this work-group's share of every buffer -----------------------------
    // (through to the memory side: whether the team may keep its words in the L2 is known below)
    auto put_marks = [&](unsigned from, unsigned to) {
        const r4u mark = {kMark, kMark, kMark, kMark};
        for (unsigned o = from + ((unsigned)x.rank * kResThreads + (unsigned)tid0) * 16u; o < to; o += TS * kResThreads * 16u)
            __builtin_amdgcn_raw_buffer_store_b128(mark, x.buf, (int)o, 0, 16);
    };
    if (!helper) {
        put_marks(0u, bo.z);
        put_marks(bo.key, bo.pre);
        // (of the operand beyond the joint width, which nobody sends: zeros)
        const int j4 = p.J >> 2;
        for (unsigned o = ((unsigned)x.rank * kResThreads + (unsigned)tid0) * 16u; o < kResSlots * ZSLOT; o += TS * kResThreads * 16u) {
            const int k4 = res_z_k4(BF, CLS, o % ZSLOT);
            const unsigned a = k4 < j4 ? kMark : 0u, b = BF && (o % ZWAVE) < (unsigned)NF * 1024u ? (k4 + 1 < j4 ? kMark : 0u) : a;
            __builtin_amdgcn_raw_buffer_store_b128((r4u){a, a, b, b}, x.buf, (int)(bo.z + o), 0, 16);
        }
    } else {
        bool any = false;
        for (int i = 0; i < kResServed; ++i)
            if (serves(i)) {
                x.buf = buffers_of(team + i * pairs); any = true;
                // (zeros where no unit is: nobody sends these words)
                for (unsigned o = ((unsigned)x.rank * kResThreads + (unsigned)tid0) * 16u; o < kResSlots * PSLOT; o += TS * kResThreads * 16u) {
                    const int word = (int)(o / 4u) % (TS * 320 * GL), r = word / (320 * GL), lu = word % (320 * GL) / (16 * GL);
                    const unsigned v = lu < p.pl.units && r * p.pl.units + lu < p.H ? kMark : 0u;
                    __builtin_amdgcn_raw_buffer_store_b128((r4u){v, v, v, v}, x.buf, (int)(bo.pre + my_layer * kResSlots * PSLOT + o), 0, 16);
                }
            }
        if (!any) return;
    }
    if (tid0 == 0) { rc.ok = 1; rc.n_list = 0; rc.st_clamped = 0; rc.st_overflow = 0; }
    if (tid0 < kResSamples) { rc.s_k[tid0] = p.blank; rc.s_d[tid0] = 0; }
    if (tid0 < kMaxDur) rc.dur[tid0] = p.durations[tid0];
    if (tid0 < RRows::kPlaces) rc.scale[tid0] = 1.f;
    if (lane0 < RRows::kPlaces) {
        RRows &w = rc.rows[x.wave];
        w.s[lane0] = RRow{0, 0, 0, 0}; w.b[lane0] = w.since[lane0] = w.next = 0;
    }
    for (int i = tid0 * 16; i < lo.bytes; i += kResThreads * 16) *reinterpret_cast<r4u *>(lds + i) = (r4u){0, 0, 0, 0};
    // the marks have to be in memory before this work-group says that it is there
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    // ---- the team meets: everyone announces the XCD it runs on --------------------------------
    auto announce = [&]() {
        if (tid0 == 0) {
            const unsigned id = (__builtin_amdgcn_s_getreg((3 << 11) | 20) & 0xfu) + 1u;
            __hip_atomic_store(p.form + blockIdx.x, id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    // Waits for team t in the first waves: lanes 0 .. TS-1 of the first for the chain's work-groups and (both) of the
    // next two for the helpers of either layer; true when the chain's all sit on one XCD.
    auto meet = [&](int t, bool both) {
        const int side = x.wave, r = lane0;
        const bool mine = r < TS && (side == 0 || (both && side < 3));
        unsigned v = 1;
        if (mine) {
            const int on = t % chain_xcds, at = side ? chain_xcds + on % pairs * 2 + side - 1 : on;
            const unsigned *slot = p.form + ((t / chain_xcds) * TS + r) * n_xcd + at;
            unsigned spins = 0;
            v = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            while (v == 0u) {
                if (wait_expired(p, spins)) { rc.ok = 0; break; }
                v = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            x.polls += __builtin_amdgcn_readfirstlane((int)spins);
        }
        const unsigned first = (unsigned)__builtin_amdgcn_readfirstlane((int)v);
        return __syncthreads_and(!(mine && side == 0 && v != first)) != 0;
    };
    // The waves that load the next step's frames beside the cells are the last to see the hidden vector, and share their SIMDs
    // with waves that have cells: from the step's results to their loads they go first.  32 utterances 1286 us without, 1280 with it, TDT 883
    // and 880, 128 utterances 4173 and 4150, bfloat16 mode 873 and 866, 57 with e4m3 weights 727 and 716, 14 of a one-layer model 467 and
    // 461 (means of up to eight draws).  The waves with cells first: 0.6 % longer than without.  fp32 models with one tile of samples: no difference.
    constexpr bool FRAMES_FIRST = NMT == 2 || BF;
    constexpr bool TOUCH = PAIR && CLS == 0 && NMT == 2;          // see the joint step
    const bool has_cells = x.wave < 5;          // finishes 16 (unit, row) pairs of the LSTM stages, see stage_sum
    // (beyond the buffer for waves without cells, whose loads give zeros: a branch around the loads would make the
    // compiler wait for them where it waits for an older one)
    unsigned pre_wave = has_cells ? ((unsigned)x.rank * 5u + (unsigned)x.wave) * (256u * GL) : 0x80000000u;
    asm volatile("" : "+s"(pre_wave));
    const int h4 = p.H >> 2;

    if constexpr (PAIR) if (helper) {
        // ---- helpers: W_hh of a layer times the candidate vectors -----------------------------
        // A work-group has a quarter of K and eighty units: with all of K and twenty units, the work-groups fetched four times
        // as much from the memory side (72 KB each in 3 us, most of it not there yet), and results came too late for
        // the next step: 8.5 us a step of 32 utterances now, 9.4 then, of 128 utterances 9.0 and 9.8.  The chain adds the quarters.
        // Twenty tiles of four units, three for the first four waves and two for the others (waves w and w + 4
        // share a SIMD), which need no sums from each other.  The columns of the matrix instructions are the rows of two
        // teams of four rows, in two parts, or of one team of eight.
        static_assert(!BF, "the rows in two parts are the sixteen columns");
        constexpr int PER = 8 / R;                // teams of a set of columns
        constexpr int HB = res_help_blocks(CLS), HREGS = res_help_regs(CLS);
        const int quarter = x.rank & 3, first_unit = (x.rank >> 2) * 80, tile0 = x.wave < 4 ? x.wave * 3 : x.wave * 2 + 4;
        const bool third = x.wave < 4;
        RegW<HREGS> w;
        announce();
        load_regs<false>(w, p.w_help + ((long long)(my_layer * TS + x.rank) * kResWaves + x.wave) * HREGS * 64, 0, lane0);
        keep_regs(w);
        unsigned live = 0;
#pragma unroll
        for (int i = 0; i < kResServed; ++i)
            if (serves(i)) { (void)meet(team + i * pairs, false); live |= 1u << i; }
        // LDS: the scales of the work-group's outputs; twice, for vectors that come and those in work, [set of columns][block][lane]
        constexpr int SETS = kResServed / PER, AREA = SETS * HB * 1024, AT = 2048;
        static_assert(AT + 2 * AREA <= lo.bytes, "the helpers' layout fits");
        for (int i = tid0; i < 320; i += kResThreads)
            reinterpret_cast<float *>(lds)[i] = first_unit * 4 + i < p.H * 4 ? p.s_hh[my_layer][first_unit * 4 + i] : 0.f;
        __syncthreads();
        const unsigned area_m0 = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds + AT));
        const unsigned pre_at = bo.pre + my_layer * kResSlots * PSLOT + quarter * QSLOT;
        const unsigned apart = (unsigned)pairs * bo.bytes;       // from one team to the next
        const unsigned char *base = p.xbuf + (size_t)team * bo.bytes;
        x.buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(base), 0, (int)((kResServed - 1) * apart + bo.bytes), 0x00020000);
        // Where the lane's words of block 0 are in a vector, of teams of four rows columns 8 .. 15 being the second, see Operand::offset; and where its
        // results go (beyond the buffer: nowhere)
        const int col = lane0 & 15, g = lane0 >> 4;
        const unsigned row_at = (my_layer ? bo.hr[1] : bo.hr[0]) + (unsigned)(lane0 & (R - 1)) * VROW + (PER == 2 && (lane0 & 8) ? apart : 0u);
        const int piece = quarter * (HB * 8) + 2 * g + (col / R & 1);
        const bool has_words = (lane0 & (R - 1)) < p.slots;
        unsigned to[3];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const int u = first_unit + (tile0 + t) * 4 + g, of = u / p.pl.units, lu = u - of * p.pl.units;
            to[t] = u < p.H && (col & R) == 0 ? (((unsigned)of * 5u + (unsigned)(lu >> 2)) * (64u * GL) + (unsigned)((lu & 3) * (16 * GL) + (col & (R - 1)) * 4)) * 4u : 0x80000000u;
        }
        // bit i: the two bits of the number of team i's next vector, modulo the slots
        unsigned low = ~0u, high = 0;
        auto slot_of = [](unsigned low_, unsigned high_, int i) { return (low_ >> i & 1u) | (high_ >> i & 1u) << 1; };
        // Loads of (set of columns, block) go round the waves: f(set, block)
        constexpr unsigned OF_SET = (1u << PER) - 1u;
        auto own = [&](auto f) {
#pragma unroll
            for (int i = 0; i < (SETS * HB + kResWaves - 1) / kResWaves; ++i) {
                const int at = x.wave + i * kResWaves, q = at / HB;
                if (at < SETS * HB && (live >> (q * PER) & OF_SET) != 0u) f(q, at - q * HB);
            }
        };
        unsigned spins = 0, par = 0;
        auto ask = [&]() {
            own([&](int q, int kb) {
                const unsigned a = slot_of(low, high, q * PER) * VSLOT, b = slot_of(low, high, q * PER + PER - 1) * VSLOT, of = live >> (q * PER) & OF_SET;
                const bool second = PER == 2 && (lane_id() & 8) != 0;
                if (has_words && (of & (second ? 2u : 1u)) != 0u)
                    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2 sc1"
                                 :: "v"(row_at + (unsigned)min(piece + kb * 8, h4 - 1) * 16u + (unsigned)(q * PER) * apart + (second ? b : a)),
                                    "s"(area_m0 + par * AREA + (unsigned)((q * HB + kb) * 1024)), "s"(base) : "memory");
            });
        };
        int stored = 0;                            // stores after the last loads were asked for
        ask();
        while (live != 0u && rc.ok) {
            // the loads, without the stores behind them (which take their time to the memory side as well)
            if (stored == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            else if (stored < 6) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
            else if (stored < 8) asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
            else if (stored < 12) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
            else if (R == 4 || stored < 24) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(24)" ::: "memory");
            stored = 0;
            const int area = AT + (int)par * AREA;
            unsigned f = 0;                        // bits 0 ..: words of team i's vector are missing; bits 8 ..: it says stop
            own([&](int q, int kb) {
                const r4u v = *reinterpret_cast<const r4u *>(lds + area + (q * HB + kb) * 1024 + lane_id() * 16);
                const unsigned long long m = __ballot(has_words && has_mark(v)), stop = __ballot(v.x == kStop);
                constexpr unsigned long long FIRST = PER == 2 ? 0x00ff00ff00ff00ffull : ~0ull;
                f |= (((m & FIRST) != 0ull ? 1u : 0u) | ((stop & FIRST) != 0ull ? 256u : 0u) | ((m & ~FIRST) != 0ull ? 2u : 0u) | ((stop & ~FIRST) != 0ull ? 512u : 0u)) << (q * PER);
            });
            if (lane_id() == 0) rc.seen[par][x.wave] = f;
            __syncthreads();
            unsigned any = 0;
#pragma unroll
            for (int i = 0; i < kResWaves; ++i) any |= rc.seen[par][i];
            any = (unsigned)__builtin_amdgcn_readfirstlane((int)any);
            const unsigned all = live & ~any;      // the vectors that are there
            live &= ~(all & (any >> 8));
            unsigned todo = all & live;
            const unsigned low0 = low, high0 = high;
            high ^= low & todo; low ^= todo;
            par ^= 1u;
            ask();
            if (all == 0u) {
                if (wait_expired(p, spins)) rc.ok = 0;
                continue;
            }
            spins = 0;
            while (todo != 0u) {
                const int one = __builtin_ctz(todo);
                todo &= todo - 1u;
                const int two = PER == 2 && todo != 0u ? __builtin_ctz(todo) : -1;
                if (PER == 2) todo &= todo - (todo != 0u ? 1u : 0u);
                const int lane = lane_id(), of = (lane & 8) != 0 && two >= 0 ? two : one;
                const int at = PER == 2 ? area + (of >> 1) * (HB * 1024) + ((lane & ~8) | (of & 1) << 3) * 16 : area + one * (HB * 1024) + lane * 16;
                unsigned z[HB * 4];
#pragma unroll
                for (int kb = 0; kb < HB; ++kb) {
                    const r4u v = *reinterpret_cast<const r4u *>(lds + at + kb * 1024);
                    const bool other = (lane & R) != 0;
                    const unsigned keep = other ? 0x07060302u : 0x05040100u, send = other ? 0x05040100u : 0x07060302u;
                    const unsigned k0 = __builtin_amdgcn_perm(v.y, v.x, keep), k1 = __builtin_amdgcn_perm(v.w, v.z, keep);
                    const unsigned s0 = __builtin_amdgcn_perm(v.y, v.x, send), s1 = __builtin_amdgcn_perm(v.w, v.z, send);
                    constexpr int UP = 0x110 + R, DOWN = 0x100 + R, LOWER = R == 4 ? 0x5 : 0x3, UPPER = 0xf ^ LOWER;       // (banks of four lanes)
                    z[kb * 4] = (unsigned)__builtin_amdgcn_update_dpp((int)k0, (int)s0, UP, 0xf, UPPER, false);
                    z[kb * 4 + 1] = (unsigned)__builtin_amdgcn_update_dpp((int)k1, (int)s1, UP, 0xf, UPPER, false);
                    z[kb * 4 + 2] = (unsigned)__builtin_amdgcn_update_dpp((int)k0, (int)s0, DOWN, 0xf, LOWER, false);
                    z[kb * 4 + 3] = (unsigned)__builtin_amdgcn_update_dpp((int)k1, (int)s1, DOWN, 0xf, LOWER, false);
                }
                r4f sum[3];
#pragma unroll
                for (int t = 0; t < 3; ++t) sum[t] = (r4f){0.f, 0.f, 0.f, 0.f};
                auto multiply = [&](auto tiles_) {
#pragma unroll
                    for (int part = 1; part >= 0; --part)
#pragma unroll
                        for (int kb = 0; kb < HB; ++kb)
#pragma unroll
                            for (int t = 0; t < decltype(tiles_)::value; ++t) sum[t] = tile_mfma<false>(w.q[(kb * 3 + t) * 2 + part], z + kb * 4, sum[t]);
                };
                if (third) multiply(std::integral_constant<int, 3>());
                else multiply(std::integral_constant<int, 2>());
                const unsigned slot1 = slot_of(low0, high0, one), slot2 = two >= 0 ? slot_of(low0, high0, two) : 0u;
                const bool second = PER == 2 && (lane & 8) != 0;
                const unsigned mine = second ? (two >= 0 ? (unsigned)two * apart + slot2 * PSLOT : 0x80000000u) : (unsigned)one * apart + slot1 * PSLOT;
                const unsigned clear = second ? (two >= 0 ? (unsigned)two * apart + (slot2 ^ 2u) * PSLOT : 0x80000000u) : (unsigned)one * apart + (slot1 ^ 2u) * PSLOT;
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    if (t == 2 && !third) break;
                    r4f v = sum[t];
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] += dppf<0x100 + R>(v[i]);
                    v *= *reinterpret_cast<const r4f *>(lds + ((tile0 + t) * 16 + g * 4) * 4);
                    const r4u o = {word_of(v[0]), word_of(v[1]), word_of(v[2]), word_of(v[3])}, mark = {kMark, kMark, kMark, kMark};
                    // (no lane condition around the stores: every one has to be counted)
                    const unsigned out = (to[t] | mine) >> 31 ? 0x80000000u : to[t] + mine;
                    const unsigned old = (to[t] | clear) >> 31 ? 0x80000000u : to[t] + clear;
                    __builtin_amdgcn_raw_buffer_store_b128(o, x.buf, (int)out, (int)pre_at, 16);
                    __builtin_amdgcn_raw_buffer_store_b128(mark, x.buf, (int)old, (int)pre_at, 16);
                    stored += 2;
                }
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // (nothing is on its way into LDS when the work-group ends)
        if (!rc.ok && threadIdx.x == 0) __hip_atomic_fetch_or(p.status, 4, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }

    // ---- the chain's work-groups ---------------------------------------------------------------
    announce();
    // What else is read before the first step comes first, in three trips to memory (lengths and small tables, scales, weights).
    // The ranks of the utterances are worked out from the LDS: each of 32 lengths read by one lane alone, one after the other,
    // and tables a piece at a time took 11 us, this 4.6; up to the first step 16 us in place of 27 (32 utterances, fp32,
    // two layers).  With the weights asked for before all that, the same call took 0.6 % longer.
    // fp32: what the joint's operands of an utterance are multiplied by, see joint_scale
    float *list_scale = reinterpret_cast<float *>(lds + lo.scale);
    // (the lengths, in the place of the joint step's sums)
    static_assert(kResList * (CLS == 0 ? 8 : CLS == 1 ? 16 : 32) * 4 <= kResWaves * 16 * NMT * kResSumRow * 4, "the lengths of a launch fit there");
    int *lengths = reinterpret_cast<int *>(lds + lo.part);
    for (int b = tid0; b < p.B; b += kResThreads) {
        const int raw = p.enc_len[b];
        if (raw < 0 || raw > p.T) rc.st_clamped = 1;
        lengths[b] = min(max(raw, 0), p.T);
    }
    const int u0 = x.rank * p.pl.units, nu = max(0, min(p.pl.units, p.H - u0));
    const int g0 = x.rank * p.pl.jgroups, njg = max(0, min(p.pl.jgroups, (p.J >> 2) - g0));
    // A joint step of two tiles of samples is shared out by columns and samples: the work-groups of even and the next odd rank have both
    // their columns, the even one for the first tile, the odd one for the second (`half`), so that what a work-group receives
    // of the operand is one tile.  Its partner's weights of the output layer are in LDS.  A column of the tail goes with the rank's others.
    const int half = NMT == 2 ? x.rank & 1 : 0;
    const int tcol0 = p.pl.nout_m + x.rank - half, n_tails = max(0, min(NMT, p.pl.nout_m + p.pl.n_tail - tcol0));
    {
        const int at = tid0;
        const bool gate = at < nu * 4, col = at < njg * 4;
        const int ocol = (x.rank - half) * 32 + at;
        const bool out = at < 32 * NMT && ocol < p.pl.nout_m;
        float b1 = 0.f, s1 = 0.f, sh[NL] = {}, bp = 0.f, sp = 0.f, bo_ = 0.f, so_ = 0.f, bt = 0.f, st = 0.f;
        if (gate) {
            if (NL > 1) { b1 = p.bias_l[((long long)p.H + u0) * 4 + at]; s1 = p.s_ih[u0 * 4 + at]; }
#pragma unroll
            for (int l = 0; l < NREC; ++l) sh[l] = p.s_hh[l][u0 * 4 + at];
        }
        if (col) { bp = p.b_pred[g0 * 4 + at]; sp = p.s_pred[g0 * 4 + at]; }
        if (out) { bo_ = p.b_out[ocol]; so_ = p.s_out[ocol]; }
        if (at < n_tails) { bt = p.b_out[tcol0 + at]; st = p.s_out[tcol0 + at]; }
        if (at < kResUnits * 4) {
            rc.b1[at] = b1; rc.s1[at] = s1;
#pragma unroll
            for (int l = 0; l < NREC; ++l) rc.sh[l][at] = sh[l];
        }
        if (at < kResFormed) { rc.bp[at] = bp; rc.sp[at] = sp; }
        if (at < 3 * 64) reinterpret_cast<unsigned *>(lds + lo.z_at)[at] = res_z_at(BF, CLS, g0 + at / ZS, at % ZS);
        if (at < 32 * NMT) { reinterpret_cast<float *>(rc.bo)[at] = bo_; reinterpret_cast<float *>(rc.so)[at] = so_; }
        if (at < NMT) { rc.bt[at] = bt; rc.st[at] = st; }
    }
    for (int i = tid0; i < n_tails * ROW; i += kResThreads) {
        const int k = i / ROW;
        const float w = p.w_tail[(long long)(tcol0 - p.pl.nout_m) * ROW + i];
        // (rows of 16-bit values: high parts, low parts, for either column, zeros; or bf16 values; or rows of fp32 values)
        unsigned short *row = reinterpret_cast<unsigned short *>(lds + lo.tail);
        unsigned high = __float_as_uint(w) >> 16, low = 0;
        if (!BF) f16_parts(w, 0.f, high, low);
        if (WHOLE) reinterpret_cast<float *>(row)[i] = w;
        else if (BF) row[i] = (unsigned short)high;
        else { row[i + k * ROW] = (unsigned short)high; row[i + (k + 1) * ROW] = (unsigned short)low; }
    }
    __syncthreads();
    // utterances of the team: ranked by length (longest first, ties by index), dealt in serpentine
    // order; empty ones are complete from the start
    for (int b = tid0; b < p.B; b += kResThreads) {
        const int len = lengths[b];
        int pos = 0;
#pragma unroll 8
        for (int o = 0; o < p.B; ++o) pos += (lengths[o] > len || (lengths[o] == len && o < b)) ? 1 : 0;
        const int q = pos / n_teams, m = pos - q * n_teams;
        if (((q & 1) ? n_teams - 1 - m : m) == team) {
            rc.list_b[q] = (unsigned short)b; rc.list_len[q] = len;
            if (len > 0) atomicAdd(&rc.n_list, 1);       // the empty ones are the last of the list
            else if (x.rank == 0) res_finish_row(b, 0);
        }
    }
    __syncthreads();
    if constexpr (!BF && !WHOLE) {
        // sixteen lanes to an utterance of the list
        static_assert(kTopParts == 16, "a word for each of sixteen lanes");
        for (int q = tid0 >> 4; q < rc.n_list; q += kResThreads / 16) {
            TopWord top = p.p_top[((long long)rc.list_b[q] * kTopParts + (lane0 & 15)) * kTopStride];
#pragma unroll
            for (int i = 1; i < 16; i *= 2) top = max(top, (TopWord)__shfl_xor((long long)top, i));
            if ((lane0 & 15) == 0) list_scale[q] = joint_scale(top, p.q_bound);
        }
    }
    RegW<LREGS> w_hh[NREC > 0 ? NREC : 1], w_ih;
    RegW<res_pred_regs(BF, CLS)> w_pr;
    RegW<res_joint_regs(BF, CLS)> w_ou;
    {
        const float *src = p.w + (long long)(x.rank * kResWaves + x.wave) * res_main_regs(KIND, BF, CLS) * 64;
        int first = 0;
#pragma unroll
        for (int l = 0; l < NREC; ++l) { load_regs<KIND == kResident2>(w_hh[l], src, first, lane0); first += LREGS; }
        if (NL > 1) { load_regs<KIND == kResident2>(w_ih, src, first, lane0); first += LREGS; }
        load_regs<KIND == kResident2>(w_pr, src, first, lane0); first += res_pred_regs(BF, CLS);
        load_regs<KIND == kResident2>(w_ou, src, first, lane0);
        if constexpr (NMT == 2) {
            // the partner's, for the same wave
            static_assert(JREGS % 4 == 0, "whole groups of four registers");
            const float *from = p.w + ((long long)((x.rank ^ 1) * kResWaves + x.wave) * res_main_regs(KIND, BF, CLS) + first) * 64 + lane0 * 4;
            const unsigned to = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)(lds + lo.other) + (unsigned)x.wave * (JREGS * 256u);
#pragma unroll
            for (int i = 0; i < JREGS / 4; ++i)
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(from + i * 256), "s"(__builtin_amdgcn_readfirstlane((int)(to + i * 1024u))) : "memory");
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
#pragma unroll
        for (int l = 0; l < NREC; ++l) keep_regs(w_hh[l]);
        if (NL > 1) keep_regs(w_ih);
        keep_regs(w_pr);
        keep_regs(w_ou);
    }
    // What a lane finishes in the LSTM stages, see stage_sum: a row of the team, a unit and a gate.  Worked
    // out where it is used: kept for the whole loop, values like these take the registers that the
    // weights need.
    struct Place { int row, j, lu, gu; bool ok; };
    auto place_of = [&](int lane) {
        Place l;
        l.row = (int)((unsigned)lane / LR) & (R - 1); l.j = lane & (LR - 1);
        l.lu = x.wave * 4 + (lane >> 4);
        l.ok = l.lu < nu && l.j == 0 && l.row < p.slots;      // the lanes that publish it
        l.gu = min(u0 + l.lu, p.H - 1);
        return l;
    };
    // (joint output: a wave takes every eighth step of K for both column tiles)
    const unsigned lds_p = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)(lds + lo.p);
    float *part = reinterpret_cast<float *>(lds + lo.part);          // joint sums, see there
    float *tpart = reinterpret_cast<float *>(lds + lo.tpart);        // [wave][tile][16]
    float *sums_pr = reinterpret_cast<float *>(lds + lo.proj), *sums_ih = reinterpret_cast<float *>(lds + lo.ih);
    float *sums_rec0 = reinterpret_cast<float *>(lds + lo.rec0), *sums_top = reinterpret_cast<float *>(lds + lo.rec);

    if (!BF && !WHOLE && p.p_call && x.rank == 0 && team == 0 && tid0 == 0) ++*p.p_call;        // (of those here nobody reads it)
    x.local = meet(team, PAIR);
    bool ok = rc.ok != 0;

    // state of the lane's cell, [layer]: committed and candidate cell value; recurrent pre-activations W_hh h of the
    // committed vector (kResident2Pair: in LDS, where the others have their recurrent sums; the weights need the registers)
    // and, kResident2Pair, of the last step's candidate, a word from every quarter of K as far as it is there, kMark where not
    float *state = reinterpret_cast<float *>(lds + lo.state);
    auto stored = [&]() { return state + x.wave * 64 + lane_id(); };               // (fields 5 * 64 floats apart)
    constexpr int FIELD = 5 * 64;
    typedef RGates<R> Gates;
    Gates first_sum{};
    constexpr int FIELDS = 2 + GL;
    float cs[NL], cc[NL];
    Gates ps[NL];
    unsigned pre[NL][kResQuarters][GL];
    auto clear_state = [&](int l) {
        cs[l] = cc[l] = 0.f;
#pragma unroll
        for (int e = 0; e < GL; ++e) ps[l].g[e] = 0.f;
    };
#pragma unroll
    for (int l = 0; l < NL; ++l) {
        clear_state(l);
#pragma unroll
        for (int i = 0; i < kResQuarters; ++i)
#pragma unroll
            for (int e = 0; e < GL; ++e) pre[l][i][e] = 0u;
    }
    auto keep_state = [&](int l) {
        float *to = stored() + l * FIELDS * FIELD;
        to[0] = cs[l]; to[FIELD] = cc[l];
#pragma unroll
        for (int e = 0; e < GL; ++e) to[(2 + e) * FIELD] = ps[l].g[e];
    };
    unsigned n_pred = 0, n_joint = 0;

    RRows &rows = rc.rows[x.wave];
    int n_samples = 0, row_steps = 0;
    // What the loop control leaves for the steps: of the row that the lane finishes cells of, the last label
    // (and, in lane_const, what the prediction step does with the candidate state); of sample `lane`, its row
    // of the projected frames, -1 for none.
    int last = p.blank, pidx = -1;
    // What a lane needs of the loop control's tables, packed (a register each would be one too many): rows of the
    // samples lane / 2, four times the wave plus lane / 16 (of the work-group's tile), and lane (RB bits each, at 0, 14 and 17);
    // bytes to the words of a row of T0 that its cell takes (RB .. 13); the place of sample `lane` among its row's
    // (5 bits, at 20); its own row's first sample (5, at 25); kTake and kFresh.
    int lane_const = kFresh;
    // Rows that take part in the joint step (one bit in four, as in LEADS), and the frames of each: the samples are dealt
    // evenly to the rows with an utterance (res_frames), so that the last ones of a team's list go on faster when the others have
    // ended.  With eight frames a row whatever
    // its neighbours do, 32 utterances on six teams took 178, 170 and 151 joint steps instead of 161, 160 and 139 (three
    // draws; 1544, 1450 and 1348 us instead of 1470, 1412 and 1283), 19 of a multi-blank model 105, 89 and 69 instead of
    // 85, 76 and 54 (846, 760 and 602 us instead of 757, 711 and 520).
    unsigned part_rows = 0;
    // Rows with an utterance, and the lanes that take their hidden values (res_takers): a row that has ended without another utterance never
    // gets one, so its words stay where they are.  They are what eight rows cost a team where most have ended: one utterance of 2000 labels among
    // 127 blank ones 16.0 ms with all rows' words, 14.2 without those of ended rows (four rows, all words 14.1), among 255 16.8 and 15.0 (14.5), bfloat16
    // mode 14.2 and 12.1 (12.8), 19 utterances of a multi-blank model 633 and 615 us.  As a test of every lane's bit at every poll, and ended rows' words
    // not sent either, up to 1 % longer in calls of 9 to 24 utterances.
    unsigned active_rows = 0;
    unsigned long long takers = 0;
    int la = 0;
    auto part_samples = [&]() { return __builtin_popcount(part_rows) * la; };
    auto lay_out = [&](auto nt_, int lane, unsigned of) {
        part_rows = of;
        const int n = __builtin_popcount(of);
        la = res_frames(decltype(nt_)::value, NMT, R, n);
        unsigned rows_of = 0;            // the rows that take part, one after the other, RB bits each
        int at = 0;
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (of >> (r * LR) & 1u) { rows_of |= (unsigned)r << at; at += RB; }
        const float inverse = __builtin_amdgcn_rcpf((float)la);
        auto turn_of = [&](int s) {
            if constexpr (R == 4) return (s >= la ? 1 : 0) + (s >= 2 * la ? 1 : 0) + (s >= 3 * la ? 1 : 0);
            else return res_turn(s, inverse, R);
        };
        auto row_of = [&](int s) { return (int)(rows_of >> (turn_of(s) * RB) & (R - 1)); };
        const int s = lane & (ZS - 1);
        const Place l = place_of(lane);
        const int first = __builtin_popcount(of & ((1u << (lane & (16 - LR))) - 1u)) * la;
        lane_const = row_of(lane / 2 & (ZS - 1)) | l.gu * 16 + l.j * (4 * GL) |
                     row_of(((x.wave * 4 + (lane >> 4)) & 15) + (decltype(nt_)::value == 2 ? half * 16 : 0)) << 14 | row_of(s) << 17 |
                     ((s - turn_of(s) * la) & 31) << 20 | (first & 31) << 25 | (lane_const & (kTake | kFresh));
    };
    std::integral_constant<int, NMT> all_tiles;
    // Samples of the next joint step: the next `la` frames of every row in work.
    auto set_up_samples = [&](int lane, int t, int b, int len) {
        const int from = (lane_const >> 17 & (R - 1)) * (LR * 4);                         // (bytes: LR lanes per row)
        const int base = __builtin_amdgcn_ds_bpermute(from, b * p.T + t), left = __builtin_amdgcn_ds_bpermute(from, len - t);
        const int off = lane_const >> 20 & 31;
        pidx = ((lane & (ZS - 1)) < part_samples() && off < left) ? base + off : -1;
        n_samples += __popcll(__ballot(pidx >= 0 && lane < ZS));
    };
    // Frames of the joint's operand: four columns of sample lane % ZS to LDS, [four columns][sample].
    auto load_frames = [&](int cg, bool mine) {
        const unsigned to = (unsigned)__builtin_amdgcn_readfirstlane((int)(lds_p + (unsigned)(cg * ZS) * 16u));
        const int at = cg + lane_id() / ZS;
        if (mine && pidx >= 0 && at < njg)
            asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(p.P + (long long)pidx * p.J + (g0 + at) * 4), "s"(to) : "memory");
    };
    // Two columns of a sample for a lane, four columns of 32 samples for a wave (of 16: eight): waves kFormers and after.
    auto publish_z = [&](auto nt_, unsigned n) {
        const int lane = lane_id(), s = lane / 2 & (ZS - 1), cg = (x.wave - kFormers) * (32 / ZS) + lane / (2 * ZS), row = lane_const & (R - 1);
        static_assert((kResWaves - kFormers) * (32 / ZS) * 4 <= kResFormed, "the tables have a place for every lane");
        const float *v = sums_pr + row * kResProjRow + min(cg, kResProjRow / 4 - 1) * 4 + (lane & 1) * 2;
        r2f o[kResWaves];
#pragma unroll
        for (int w = 0; w < kResWaves; ++w) o[w] = *reinterpret_cast<const r2f *>(v + w * (R * kResProjRow));
        const r2f frame = *reinterpret_cast<const r2f *>(lds + lo.p + (cg * ZS + s) * 16 + (lane & 1) * 8);
        const unsigned to = reinterpret_cast<const unsigned *>(lds + lo.z_at)[cg * ZS + s] + (lane & 1) * (BF ? 4u : 8u);
        const r2f bias = *reinterpret_cast<const r2f *>(rc.bp + cg * 4 + (lane & 1) * 2), by = *reinterpret_cast<const r2f *>(rc.sp + cg * 4 + (lane & 1) * 2);
        float scale = 1.f;
        if constexpr (!BF && !WHOLE) scale = rc.scale[row];
        const r2f sum = ((o[0] + o[1]) + (o[2] + o[3])) + ((o[4] + o[5]) + (o[6] + o[7]));
        float z[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const float q = BF ? sum[i] + bias[i] : WHOLE ? fmaf(sum[i], by[i], bias[i]) : fmaf(sum[i], by[i], bias[i]) * scale;
            z[i] = fmaxf(BF || WHOLE ? frame[i] + q : fmaf(frame[i], scale, q), 0.f);
        }
        const unsigned now = bo.z + slot_at(n, ZSLOT), old = bo.z + slot_at(n + 2, ZSLOT);
        if (cg < njg) {
            if (decltype(nt_)::value < NMT && s >= 16 * decltype(nt_)::value) {
                if constexpr (BF) put_mark(x, to, old);
                else put_mark2(x, to, old);
            } else if constexpr (BF) put(x, to, now, old, bf16_pair(z[0], z[1]));
            else put2(x, to, now, old, (r2u){__float_as_uint(z[0]), __float_as_uint(z[1])});
        }
    };
    // Rows that want one get the next utterances of the list.  (Control state is by row: every lane works on
    // row lane / LR % R, and the first of LR lanes below 16 stands for its row in ballots.)
    constexpr unsigned long long LEADS = R == 4 ? 0x1111ull : 0x5555ull;
    bool queued = false;               // utterances of the list wait for a row
    auto refill = [&](int lane, bool want, int &b, int &len) {
        const unsigned long long m = __ballot(want) & LEADS;
        if (m == 0ull) return false;
        const int next = rows.next, at = next + __popcll(m & ((1ull << (lane & (16 - LR))) - 1ull));
        const bool got = want && at < rc.n_list;
        if (got) { b = rc.list_b[at]; len = rc.list_len[at]; }
        // (one place for all waves: they write the same, between the same barriers)
        if constexpr (!BF && !WHOLE)
            if (got) rc.scale[(int)((unsigned)lane / LR) & (R - 1)] = list_scale[at];
        rows.next = next + __popcll(m);
        queued = __builtin_amdgcn_readfirstlane(rc.n_list) > __builtin_amdgcn_readfirstlane(next) + __popcll(m);
        return got;
    };
    __syncthreads();                  // the list is complete
    bool any_active, need_pred, later = false;
    RRow only{};                      // ONE: the row, and its utterance
    int only_b = 0;
    {
        int b = 0, len = 0;
        const int r = (int)((unsigned)lane0 / LR) & (R - 1);
        const bool got = refill(lane0, r < p.slots, b, len);
        if (got) { rows.b[r] = b; rows.s[r].len = len; }
        const unsigned long long m = __ballot(got) & LEADS;
        any_active = need_pred = m != 0ull;
        active_rows = (unsigned)m; takers = res_takers(R, active_rows);
        row_steps = __popcll(m);
        lay_out(all_tiles, lane0, (unsigned)m);
        set_up_samples(lane0, 0, b, len);
        if constexpr (ONE) { only.len = __builtin_amdgcn_readfirstlane(len); only_b = __builtin_amdgcn_readfirstlane(b); }
    }
    // the row of the embedding table (folded into the first layer) that the next prediction step adds
    Gates t0{};
    const unsigned t0_row = (unsigned)p.H * 16u;
    auto load_t0 = [&]() {
        t0 = Gates{};
        if (has_cells)
            t0 = *reinterpret_cast<const Gates *>(reinterpret_cast<const char *>(p.T0) + (__umul24((unsigned)last, t0_row) + ((unsigned)lane_const & (0x3fffu & ~(R - 1u)))));
    };
    // kResident2Pair: W_hh h of the last step's candidates of a layer as far as it is there
    auto load_pre = [&](unsigned n, int l, unsigned (&to)[kResQuarters][GL]) {
        const unsigned slot = bo.pre + slot_at(n, PSLOT) + (unsigned)l * kResSlots * PSLOT;
        const unsigned o = pre_wave + (unsigned)lane_id() * (4u * GL);
#pragma unroll
        for (int i = 0; i < kResQuarters; ++i) {
            if constexpr (GL == 1) to[i][0] = get1(x, o, slot + i * QSLOT);
            else {
                const r2u v = get2(x, o, slot + i * QSLOT);
                to[i][0] = v.x; to[i][1] = v.y;
            }
        }
    };
    auto no_pre = [&](const unsigned (&w)[kResQuarters][GL]) {
        unsigned m = 0u;
#pragma unroll
        for (int i = 0; i < kResQuarters; ++i)
#pragma unroll
            for (int e = 0; e < GL; ++e) m = max(m, w[i][e]);
        return __ballot(m == kMark) != 0ull;
    };
    auto wait_pre = [&](unsigned n, int l) {
        // (the first look apart, which does not wait for stores behind the loads)
        if (!no_pre(pre[l])) return;
        unsigned spins = 0;
        do {
            if (wait_expired(p, spins)) { rc.ok = 0; break; }
            load_pre(n, l, pre[l]);
        } while (no_pre(pre[l]));
        x.polls += __builtin_amdgcn_readfirstlane((int)spins);
    };
    if (need_pred) load_t0();
#ifdef RNNT_PROFILE
    if (tid0 == 0) { for (int i = 0; i < 24; ++i) res_prof[i] = 0; res_prof_last = wall_clock64(); }
#endif

    // Steps with NT tiles of samples: until the team is done, or the other number of tiles suits its rows better.
    auto steps = [&](auto nt_) {
    constexpr int NT = decltype(nt_)::value;
    constexpr int NS = 16 * NT;
    bool change = false;
    while (ok && any_active && !change) {
        // a stage's sum for the lane, as it is to be used
        auto sum_of = [&](const float *sums, const float *scales) {
            const int lane = lane_id();
            Gates v = stage_sum<R>(sums, x.wave, lane);
            if constexpr (!BF) {
#pragma unroll
                for (int e = 0; e < GL; ++e) v.g[e] *= scales[(x.wave * 4 + (lane >> 4)) * 4 + (lane & (LR - 1)) * GL + e];
            }
            return v;
        };
        const unsigned jn = ++n_joint;
        const unsigned long long take = ONE ? res_takers(R, 1u) : takers;
        // A wave's part of the operand, an eighth of K of a tile's samples
        constexpr int PIECES = BF ? NB : NH;
        r4u zw[PIECES];
        auto ask_z = [&]() {
            const unsigned lane = (unsigned)lane_id(), at = bo.z + slot_at(jn, ZSLOT) + (unsigned)((NT == 2 ? half * kResWaves : 0) + x.wave) * ZWAVE;
#pragma unroll
            for (int i = 0; i < PIECES; ++i) {
                if (BF && i == NF) {
                    const r2u v = get2(x, lane * 8u, at + i * 1024u);
                    zw[i] = (r4u){v.x, v.y, 0u, 0u};
                } else zw[i] = get4(x, lane * 16u, at + i * 1024u);
            }
        };
        // Waits for the words that were asked for; the largest one (they are not negative, so as a float too)
        auto wait_z = [&]() {
            unsigned spins = 0, m;
            for (;;) {
                m = 0u;
#pragma unroll
                for (int i = 0; i < PIECES; ++i) m = max(max(max(zw[i].x, zw[i].y), max(zw[i].z, zw[i].w)), m);
                if (__ballot(m == kMark) == 0ull) break;
                if (wait_expired(p, spins)) { rc.ok = 0; break; }
                ask_z();
            }
            x.polls += __builtin_amdgcn_readfirstlane((int)spins);
            return __uint_as_float(m);
        };
        if (need_pred) {
            // ---- prediction step -----------------------------------------------------------------
            ++n_pred;
            const unsigned n = n_pred;
            if (PAIR && n > 1) wait_pre(n - 1, 0);
            RES_MARK(0);
            if constexpr (PAIR && !ONE) {
                const float *from = stored();
#pragma unroll
                for (int l = 0; l < NL; ++l) {
                    clear_state(l);
                    if (has_cells) {
                        cs[l] = from[l * FIELDS * FIELD]; cc[l] = from[(l * FIELDS + 1) * FIELD];
#pragma unroll
                        for (int e = 0; e < GL; ++e) ps[l].g[e] = from[(l * FIELDS + 2 + e) * FIELD];
                    }
                }
            }
            // rows that emitted take their candidate state, fresh rows start from zero (kResident2: the second
            // layer's while the first one's vector is on its way; kResident2Pair: not before its own cell, the helpers
            // have till then)
            auto commit = [&](int l) {
                // (Zero for waves without cells, but from a variable: with a constant the compiler waits for the row of T0, and with it
                // for everything, between the loads of two frames: bfloat16 mode 1035 instead of 962 us for 32 utterances.)
                Gates pc;
#pragma unroll
                for (int e = 0; e < GL; ++e) {
                    pc.g[e] = __uint_as_float(pre[l][0][e]);
                    if constexpr (PAIR) pc.g[e] = (pc.g[e] + __uint_as_float(pre[l][1][e])) + (__uint_as_float(pre[l][2][e]) + __uint_as_float(pre[l][3][e]));
                }
                if constexpr (!PAIR)
                    if (has_cells) pc = NL == 1 ? first_sum : sum_of(l == 0 ? sums_rec0 : sums_top, rc.sh[l]);
                if constexpr (ONE && PAIR) {
                    // (it emitted, or nothing would be predicted: all that the cell keeps is its last candidate, in a register: one utterance 326 and 320 us.
                    // Models whose weights leave more room, which kept it there before, took up to 0.9 % longer.)
                    cs[l] = cc[l];
#pragma unroll
                    for (int e = 0; e < GL; ++e) ps[l].g[e] = n > 1 ? pc.g[e] : 0.f;
                    return;
                }
                const bool take = lane_const & kTake, fresh_row = lane_const & kFresh;       // (bits: as a chain of comparisons it became branches)
                cs[l] = take ? cc[l] : cs[l]; cs[l] = fresh_row ? 0.f : cs[l];
#pragma unroll
                for (int e = 0; e < GL; ++e) { ps[l].g[e] = take ? pc.g[e] : ps[l].g[e]; ps[l].g[e] = fresh_row ? 0.f : ps[l].g[e]; }
            };
            // publishes the lane's hidden value of a layer and clears the slot of two steps ago
            unsigned word = 0;
            auto publish_h = [&](int layer, const Place &l, float h) {
                word = hidden_word<BF>(h);
                // (l.gu is u0 + l.lu where a lane publishes; of one layer's models the small one was 1.4 % slower without its limit)
                if (l.ok) put(x, (unsigned)l.row * VROW + (unsigned)(NL > 1 ? u0 + l.lu : l.gu) * 4u, bo.h[layer] + slot_at(n, VSLOT), bo.h[layer] + slot_at(n + 2, VSLOT), word);
            };
            // The same to the helpers, when the team's own vector is there: loads and stores of a wave are counted in one
            // order, so polls behind these stores wait for the memory side to take them (label looping of 32 utterances 1470 us with the
            // stores before the polls, 1374 us now, together with the polls apart, below).
            // (No condition around the stores, or what was loaded before them would be waited for together with them.  They are done, the
            // marks among them, when the wave's next polls are: of the second layer's vector, or of the joint's operand, wait_z.)
            auto forward_h = [&](int layer) {
                const Place l = place_of(lane_id());
                const unsigned o = has_cells && l.ok ? (unsigned)l.row * VROW + (unsigned)(u0 + l.lu) * 4u : 0x80000000u;
                put_far(x, o, bo.hr[layer] + slot_at(n, VSLOT), word);
                put_far(x, o, bo.hr[layer] + slot_at(n + 2, VSLOT), kMark);
            };
            // Polls of its own for either kind of wave.  The compiler knows by register what is on its way from memory, not by
            // wave: behind a common branch around the cells it waits for T0's row, and so for the stores just made
            // or the frames, before a register that the row may still come to is used for the polls.  (The two copies: bfloat16
            // mode 978 us with a common branch, 957 us with two; one utterance 529 and 515 us.)
            Op x1;
            if (has_cells) {
                commit(0);
                const Place l = place_of(lane_id());
                float h;
                Gates in;
#pragma unroll
                for (int e = 0; e < GL; ++e) in.g[e] = ps[0].g[e] + t0.g[e];
                cell<R>(in, l.j, cs[0], cc[0], h);
                publish_h(0, l, h);
                if constexpr (PAIR && !ONE) keep_state(0);
                if constexpr (NREC > 1) commit(1);
                if (NMT == 2 && later) {
                    const int lane = lane_id(), r = (int)((unsigned)lane / LR) & (R - 1);
                    const RRow o = rows.s[r];
                    set_up_samples(lane, o.t, rows.b[r], o.len);
                    later = false;
                }
                RES_MARK(1);
                x1.receive_from(p, x, bo.h[0] + slot_at(n, VSLOT), h4, take);
            } else {
                // The work-group's columns of the joint step's frames, by the waves that have the least to do here.  A wave's loads return in
                // order, so these waves see the hidden vector when their frames are there: at about the time it comes.
                load_frames((x.wave - 5) * (64 / ZS), true);
                if constexpr (FRAMES_FIRST) __builtin_amdgcn_s_setprio(0);
                x1.receive_from(p, x, bo.h[0] + slot_at(n, VSLOT), h4, take);
#pragma unroll
                for (int e = 0; e < GL; ++e)
                    asm volatile("" :: "v"(t0.g[e]), "v"(pre[0][0][e]), "v"(pre[0][1][e]), "v"(pre[0][2][e]), "v"(pre[0][3][e]));
            }
            RES_MARK(2);
            if constexpr (NL > 1) {
                const Op x0 = x1;
                // (The second layer's results come during the stage.  Asked for at the end of the last step as well, they were there
                // sooner, but no step was shorter: with one utterance 6.83 against 6.78 us.  Eight rows: twice as many registers, and four of weights
                // were read back in every step; asked for behind the stage, 128 utterances 3048 and 3014 us.)
                // The vector goes to the helpers behind the matrix instructions, which end meanwhile: ahead of them it takes 0.1 us of a step
                // (32 utterances 1158 and 1151 us, TDT 811 and 804, one utterance 373 and 370.  The second layer's behind the projection: no gain.)
                if (PAIR && R == 4) load_pre(n - 1, NL - 1, pre[NL - 1]);
                stage<BF, CLS, R, 5, STAGE_ROW>(w_ih, x0, sums_ih, x.wave, [&]() {
                    if constexpr (PAIR) { ordered(); forward_h(0); ordered(); }
                });
                if (PAIR && R == 8) load_pre(n - 1, NL - 1, pre[NL - 1]);
                __syncthreads();
                RES_MARK(3);
                if constexpr (PAIR) {
                    if (n > 1) wait_pre(n - 1, NL - 1);
                    RES_MARK(4);
                    commit(NL - 1);
                }
                if (has_cells) {
                    const Place l = place_of(lane_id());
                    float h;
                    Gates in = sum_of(sums_ih, rc.s1);
#pragma unroll
                    for (int e = 0; e < GL; ++e) in.g[e] += ps[1].g[e] + rc.b1[l.lu * 4 + l.j * GL + e];
                    cell<R>(in, l.j, cs[1], cc[1], h);
                    publish_h(1, l, h);
                    if constexpr (PAIR && !ONE) keep_state(1);
                }
                RES_MARK(5);
                // (while the hand-over is on its way) the recurrent part of the next step's first layer
                if constexpr (NREC > 1) {
                    r4u v[NB];
                    auto places = [&](unsigned (&off)[NB], int lane) {
#pragma unroll
                        for (int i = 0; i < NB; ++i) off[i] = Op::offset(i, x.wave, lane, h4);
                    };
                    stage<BF, CLS, R, 5, STAGE_ROW>(w_hh[0], x0, sums_rec0, x.wave, [&]() {
                        unsigned off[NB];
                        const int lane = lane_id();
                        places(off, lane);
                        request<NB>(x, off, bo.h[1] + slot_at(n, VSLOT), v, __builtin_amdgcn_inverse_ballot_w64(take));
                        ordered();
                    });
                    RES_MARK(6);
                    unsigned off[NB];
                    const int lane = lane_id();
                    places(off, lane);
                    receive_rest<NB>(p, x, off, bo.h[1] + slot_at(n, VSLOT), v, __builtin_amdgcn_inverse_ballot_w64(take));
                    x1.set(v, lane);
                } else {
                    RES_MARK(6);
                    // A poll that comes too early is repeated after 0.25 us, and slows down what it waits for: the first one
                    // 320 cycles on.  (32 utterances 1292, 1316 and 1144 us without the pause, three draws, 1266, 1285, 1120 with 128
                    // cycles, 1263, 1281, 1115 with 192, 1256, 1277, 1108 with 320, 1267, 1285, 1116 with 448; one utterance 525, 522, 521, 522, 522.
                    // Narrower classes, calls of 1 to 96 utterances of 320 or 128 units, 65 to 170 us: 48 of 320 units 1.2 % shorter with it, the others
                    // within 0.4 %.  Pauses before the other polls: no gain, there is work in between.)
                    __builtin_amdgcn_s_sleep(5);
                    x1.receive_from(p, x, bo.h[1] + slot_at(n, VSLOT), h4, take);
                    if (PAIR) forward_h(1);
                }
            }
            RES_MARK(7);
            // prediction-side joint projection
            stage<BF, CLS, R, 2, kResProjRow>(w_pr, x1, sums_pr, x.wave);
            // this wave's frames are in LDS (what the other waves have stored by now, marks too, their polls for z wait for)
            if (x.wave >= 5) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (x.wave >= kFormers) publish_z(nt_, jn);
            RES_MARK(8);
            // (while z is on its way) the recurrent part of the top layer's next step
            if constexpr (NREC > 0) {
                // (The first tile is asked for when the work that fills the time is all but done.)
                stage<BF, CLS, R, 5, STAGE_ROW>(w_hh[NREC - 1], x1, sums_top, x.wave, [&]() { ask_z(); ordered(); });
            } else {
                ask_z();
            }
            RES_MARK(9);
            RES_MARK(10);
        } else {
            if constexpr (FRAMES_FIRST) __builtin_amdgcn_s_setprio(0);
            if (x.wave >= kFormers) {
                load_frames((x.wave - kFormers) * (32 / ZS), lane_id() < 32);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                publish_z(nt_, jn);
            }
            RES_MARK(11);
            ask_z();
        }
        // ---- joint step ----------------------------------------------------------------------------
        // The frames that come after those of this step are brought to the XCD's L2 meanwhile, a work-group asking for a word of every
        // line of one: the frames' loads of the next step are what the waves without cells wait for.  (Into LDS, where nobody reads them: a
        // register would be waited for.  By the wave that is done first; its next wait, for the keys, is 1.5 us on.)  128 utterances, whose
        // projected frames are in no L2 any more, 4147 us without and 4075 with it, 80 utterances 2988 and 2965, 32 utterances 1278 and
        // 1270, TDT 879 and 879.  (One tile of samples: no gain; one-layer and bfloat16 models: weights spilled.  A scalar branch around
        // it instead of touch_rows: 32 utterances 0.3 % longer than without.)
        if constexpr (TOUCH) if (x.wave == 0) {
            static_assert(TS == kResSamples, "a sample for every work-group");
            const int lane = lane_id(), s = x.rank + (lane >> 5) * TS, k = (lane & 31) * 32;          // (upper half of the lanes: beyond NS)
            const int row = touch_row(from_lane(pidx, s & (kResSamples - 1)), la, p.touch_rows);
            const unsigned to = (unsigned)__builtin_amdgcn_readfirstlane((int)(lds_p + (unsigned)(lo.touch - lo.p)));
            if (s < NS && row >= 0 && k < p.J)
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" :: "v"(p.P + (long long)row * p.J + k), "s"(to) : "memory");
        }
        {
            // A wave has an eighth of K for both column tiles.  fp32: every product is that of two fp16 parts of
            // either side (after a power of two of the utterance, see joint_scale; layers of 640: without low times low, which made the joint step 0.1 us longer and
            // the logits' error 2 % smaller), in one sum.  (Products with a low part in sums of their own made the logits' error
            // 1 to 6 % smaller, but twelve registers of the two-layer models' input weights had to be loaded from memory
            // in every step: input stage 1.18 instead of 0.96 us.)
            // (a half block comes first)
            auto block_of = [](int b) { return NH % 2 != 0 ? (b + NB - 1) % NB : b % NB; };
            unsigned again = 0;              // samples whose operand has too few bits in parts, or none
            {
                const float top = wait_z();
                if constexpr (!BF && !WHOLE) {
                    const unsigned long long fine = __ballot(top >= kResLeast), small = __ballot(top > 0.f) & ~fine, beyond = __ballot(top > kResMost);
                    if ((small | beyond) != 0ull) again = unheld(small, fine, beyond);
                }
            }
            RES_MARK(10);
            // the partner's weights of column tile c
            auto partner = [&](auto i_, auto part_, int c, int lane) {
                constexpr int i = decltype(i_)::value, N = i < NF ? 4 : 2;
                const int reg = res_tile_at(BF, CLS, 2, i, c, decltype(part_)::value);
                return *reinterpret_cast<const std::conditional_t<N == 4, r4f, r2f> *>(lds + lo.other + x.wave * (JREGS * 256) + reg / 4 * 1024 + lane * 16 + reg % 4 * 4);
            };
            // where column tile c's sums go, the work-group's own (0, 1) and its partner's (2, 3)
            auto sums_at = [&](int c, int lane) {
                const int side = NT == 2 ? (c < 2 ? half : 1 - half) : 0;
                return reinterpret_cast<r4f *>(part + ((x.wave * NT + side) * 16 + (lane & 15)) * kResSumRow + (c & 1) * 16 + (lane >> 4) * 4);
            };
            constexpr int CT = NT == 2 ? 4 : 2;               // column tiles
            std::integral_constant<int, 0> high;
            std::integral_constant<int, 1> low;
            // the operand as the matrix instructions take it: from a block's first register on, the high parts and then the low ones (else: as it came)
            auto parts_at = [](int i) { return BF || WHOLE ? i * 4 : i * 8; };
            unsigned z[PIECES * 4];
            static_for<0, NB>([&](auto i_) {
                constexpr int i = decltype(i_)::value, at = parts_at(i), N = i < NF ? 4 : 2;
                if constexpr (BF || WHOLE) {
                    z[at] = zw[i].x; z[at + 1] = zw[i].y; z[at + 2] = zw[i].z; z[at + 3] = zw[i].w;
                } else {
#pragma unroll
                    for (int e = 0; e < N; ++e) {
                        const r4u v = zw[i * 2 + e / 2];
                        f16_parts(__uint_as_float(e % 2 ? v.z : v.x), __uint_as_float(e % 2 ? v.w : v.y), z[at + e], z[at + N + e]);
                    }
                }
            });
            auto output = [&](auto tail_) {
                constexpr bool TAIL = decltype(tail_)::value;
                const r4f zero = {0.f, 0.f, 0.f, 0.f};
                // fp32: the work-group's own columns and the tail, then its partner's (registers)
                constexpr int AT = BF ? CT : 2, AHEAD = 2, BEYOND = 2;
                constexpr bool APART = NT == 2 && !BF && !WHOLE;
                // The partner's weights, sixteen bytes a lane, in the order of their use: the half block's of both column tiles, then high and low
                // part of a block's first tile, of its second.  Two reads, then four, are on their way while what is there is used (all of a block
                // asked for when it was its turn, every block waited for the LDS: 32 utterances 1173 us and 1163 now, TDT 829 and 819, one layer 871 and
                // 852, 128 utterances 2996 and 2985; three throughout 1168, 822, 855, 2966; three and five: registers spilled).
                constexpr int HALF = NH % 2 * 2, GROUPS = APART ? HALF + NF * 4 : 0;
                r4f pw[GROUPS + 1];
                unsigned from = 0;
                auto ask_weights = [&](auto lo_, auto hi_) {
                    static_for<decltype(lo_)::value, decltype(hi_)::value>([&](auto q_) {
                        constexpr int q = decltype(q_)::value, f = q - HALF;
                        constexpr int reg = f < 0 ? res_tile_at(BF, CLS, 2, NF, q, 0) : res_tile_at(BF, CLS, 2, f / 4, f / 2 % 2, f % 2);
                        pw[q] = *reinterpret_cast<const r4f *>(lds + from + (unsigned)(reg / 4 * 1024));
                    });
                };
                static_for<0, APART ? 1 : CT / AT>([&](auto own_) {
                    constexpr int c0 = decltype(own_)::value * 2;
                    r4f big[AT], tb = zero;
#pragma unroll
                    for (int c = 0; c < AT; ++c) big[c] = zero;
                    static_for<0, NB>([&](auto b_) {
                        constexpr int b = decltype(b_)::value, i = block_of(b);
                        constexpr bool FULL = i < NF;
                        std::integral_constant<int, i> block;
                        const unsigned *zh = z + parts_at(i), *zl = zh + (FULL ? 4 : 2);
                        if constexpr (BF && NH % 2 != 0 && NF > 0 && b == 1) {
                            // the sums of the half block have to be there
#pragma unroll
                            for (int c = 0; c < AT; ++c) there(big[c]);
                            if (TAIL && c0 == 0) there(tb);
                        }
                        ordered();
                        const int lane = lane_id(), m16 = lane & 15, g = lane >> 4;
                        constexpr bool BOTH = !BF && !WHOLE && !FULL;          // see both_parts
                        const unsigned zlh[4] = {zl[0], zl[1], zh[0], zh[1]}, zhl[4] = {zh[0], zh[1], zl[0], zl[1]};
                        if constexpr (BOTH) {
                            r4f w[AT];
#pragma unroll
                            for (int c = 0; c < AT; ++c) w[c] = both_parts<CLS, 2>(w_ou, c);
#pragma unroll
                            for (int c = 0; c < AT; ++c) big[c] = tile_mfma<BF>(w[c], zlh, big[c]);
#pragma unroll
                            for (int c = 0; c < AT; ++c) big[c] = tile_mfma<BF>(w[c], zhl, big[c]);
                        } else if constexpr (WHOLE) {
#pragma unroll
                            for (int c = 0; c < 2; ++c) {
                                r4f w = w_ou.q[c];
                                if constexpr (c0 != 0) w = *reinterpret_cast<const r4f *>(lds + lo.other + x.wave * (JREGS * 256) + c * 1024 + lane * 16);
                                big[c] = whole_mfma(w, zh, big[c]);
                            }
                        } else {
                            typedef std::conditional_t<FULL, r4f, r2f> Group;
                            Group wh[AT], wl[AT];
#pragma unroll
                            for (int c = 0; c < AT; ++c) {
                                const bool own = c0 + c < 2;
                                if (own) wh[c] = weights_of<BF, CLS, 2, i, 0>(w_ou, c0 + c);
                                else wh[c] = partner(block, high, c0 + c - 2, lane);
                                if constexpr (!BF) {
                                    if (own) wl[c] = weights_of<BF, CLS, 2, i, 1>(w_ou, c0 + c);
                                    else wl[c] = partner(block, low, c0 + c - 2, lane);
                                }
                            }
                            if constexpr (!BF) {
                                if constexpr (NF < 2) {
#pragma unroll
                                    for (int c = 0; c < AT; ++c) big[c] = tile_mfma<BF>(wl[c], zl, big[c]);
                                }
#pragma unroll
                                for (int c = 0; c < AT; ++c) big[c] = tile_mfma<BF>(wh[c], zl, big[c]);
#pragma unroll
                                for (int c = 0; c < AT; ++c) big[c] = tile_mfma<BF>(wl[c], zh, big[c]);
                            }
#pragma unroll
                            for (int c = 0; c < AT; ++c) big[c] = tile_mfma<BF>(wh[c], zh, big[c]);
                        }
                        // the tail columns: high and low parts (bfloat16 mode: values) are rows of their own of the
                        // operand, the others zeros
                        if constexpr (TAIL && c0 == 0 && WHOLE) {
                            tb = whole_mfma(*reinterpret_cast<const r4f *>(lds + lo.tail + (min(m16, NMT) * ROW + x.wave * 16 + g * 4) * 4), zh, tb);
                        } else if constexpr (TAIL && c0 == 0) {
                            const auto w = *reinterpret_cast<const std::conditional_t<FULL, r4f, r2f> *>(lds + lo.tail + (min(m16, BF ? NMT : 2 * NMT) * ROW + x.wave * (NH * 16) + i * 32 + g * (FULL ? 8 : 4)) * 2);
                            if constexpr (BOTH) tb = tile_mfma<BF>((r4f){w.x, w.y, w.x, w.y}, zhl, tb);
                            else {
                                if constexpr (!BF) tb = tile_mfma<BF>(w, zl, tb);
                                tb = tile_mfma<BF>(w, zh, tb);
                            }
                        }
                        ordered();
                    });
                    const int lane = lane_id();
                    if (TAIL && c0 == 0 && lane < 16) {
#pragma unroll
                        for (int k = 0; k < NMT; ++k) tpart[(x.wave * 2 + k) * 16 + lane] = BF || WHOLE ? tb[k] : tb[k * 2] + tb[k * 2 + 1];
                    }
                    // every wave's sums to LDS, [wave][side][sample][column]
#pragma unroll
                    for (int c = 0; c < AT; ++c) *sums_at(c0 + c, lane) = big[c];
                });
                if constexpr (APART) {
                    // groups asked for when `n` have been used
                    constexpr auto asked = [](int n) { return n + AHEAD + (n >= HALF ? BEYOND : 0) < GROUPS ? n + AHEAD + (n >= HALF ? BEYOND : 0) : GROUPS; };
                    from = (unsigned)(lo.other + x.wave * (JREGS * 256) + lane_id() * 16);
                    ordered();
                    ask_weights(std::integral_constant<int, 0>(), std::integral_constant<int, asked(0)>());
                    ordered();
                    r4f big[2] = {zero, zero};
                    static_for<0, HALF>([&](auto c_) {
                        constexpr int c = decltype(c_)::value;
                        const unsigned *zh = z + parts_at(NF), *zl = zh + 2;
                        const unsigned zlh[4] = {zl[0], zl[1], zh[0], zh[1]}, zhl[4] = {zh[0], zh[1], zl[0], zl[1]};
                        big[c] = tile_mfma<BF>(pw[c], zlh, big[c]);
                        big[c] = tile_mfma<BF>(pw[c], zhl, big[c]);
                        ordered();
                        ask_weights(std::integral_constant<int, asked(c)>(), std::integral_constant<int, asked(c + 1)>());
                        ordered();
                    });
                    static_for<0, NF * 2>([&](auto u_) {
                        constexpr int u = decltype(u_)::value, c = u % 2, q = HALF + u * 2;
                        const unsigned *zh = z + parts_at(u / 2), *zl = zh + 4;
                        if constexpr (NF < 2) big[c] = tile_mfma<BF>(pw[q + 1], zl, big[c]);
                        big[c] = tile_mfma<BF>(pw[q], zl, big[c]);
                        big[c] = tile_mfma<BF>(pw[q + 1], zh, big[c]);
                        big[c] = tile_mfma<BF>(pw[q], zh, big[c]);
                        ordered();
                        ask_weights(std::integral_constant<int, asked(q)>(), std::integral_constant<int, asked(q + 2)>());
                        ordered();
                    });
                    const int lane = lane_id();
#pragma unroll
                    for (int c = 0; c < 2; ++c) *sums_at(2 + c, lane) = big[c];
                }
            };
            const bool with_tail = NT == NMT ? n_tails > 0 : half < n_tails;
            if (with_tail) output(std::true_type());
            else output(std::false_type());
            if constexpr (!BF && !WHOLE) {
                // Samples whose operand parts do not hold in the wave's eighth, far below the bound or infinite, are computed once more
                // as fp32 products (the weights' parts added up again).  The lane's e-th value of
                // a block times its e-th weight is one 16x16x4 instruction.
                // (Of the step's own samples: what rows without an utterance, and places without a frame, hold may be of any size.)
                if (again != 0u) again &= (unsigned)__ballot(pidx >= 0) >> (NT == 2 ? half * 16 : 0);
                if (again != 0u) {
                    const int lane = lane_id(), m16 = lane & 15, g = lane >> 4;
                    const float scale = rc.scale[from_lane(lane_const, (NT == 2 ? half * 16 : 0) + m16) >> 17 & (R - 1)], back = inverse_power(scale);
                    const bool mine = (again >> m16 & 1u) != 0u;
                    ask_z();
#pragma unroll 1
                    for (int c2 = 0; c2 < CT; c2 += 2) {
                        r4f sum[2], tail = {0.f, 0.f, 0.f, 0.f};
                        sum[0] = sum[1] = tail;
                        static_for<0, NB>([&](auto k_) {
                            constexpr int k = decltype(k_)::value, N = k < NF ? 8 : 4;
                            typedef _Float16 Halves __attribute__((ext_vector_type(N)));
                            float z[N];
#pragma unroll
                            for (int j = 0; j < N / 4; ++j) {
                                const float4 v = __builtin_bit_cast(float4, zw[k * 2 + j]);
                                z[j * 4] = v.x * back * scale; z[j * 4 + 1] = v.y * back * scale;        // (infinite where the sum is)
                                z[j * 4 + 2] = v.z * back * scale; z[j * 4 + 3] = v.w * back * scale;
                            }
#pragma unroll
                            for (int c = 0; c < 2; ++c) {
                                auto wh = weights_of<BF, CLS, 2, k, 0>(w_ou, c), wl = weights_of<BF, CLS, 2, k, 1>(w_ou, c);
                                if (NT == 2 && c2 != 0) { wh = partner(k_, high, c, lane); wl = partner(k_, low, c, lane); }
                                asm volatile("" : "+v"(wh), "+v"(wl));           // (not added up ahead: that takes registers for the whole loop)
                                const Halves hi = __builtin_bit_cast(Halves, wh), lw = __builtin_bit_cast(Halves, wl);
#pragma unroll
                                for (int e = 0; e < N; ++e) sum[c] = __builtin_amdgcn_mfma_f32_16x16x4f32((float)hi[e] + (float)lw[e], z[e], sum[c], 0, 0, 0);
                                ordered();
                            }
                            if (with_tail && c2 == 0) {
                                const _Float16 *w = reinterpret_cast<const _Float16 *>(lds + lo.tail) + min(m16, NMT) * 2 * ROW + x.wave * (NH * 16) + k * 32 + g * N;
#pragma unroll
                                for (int e = 0; e < N; ++e) tail = __builtin_amdgcn_mfma_f32_16x16x4f32(m16 < NMT ? (float)w[e] + (float)w[ROW + e] : 0.f, z[e], tail, 0, 0, 0);
                            }
                        });
                        if (mine) {
                            if (with_tail && c2 == 0 && g == 0) {
#pragma unroll
                                for (int k = 0; k < NMT; ++k) tpart[(x.wave * 2 + k) * 16 + m16] = tail[k];
                            }
#pragma unroll
                            for (int c = 0; c < 2; ++c) *sums_at(c2 + c, lane) = sum[c];
                        }
                    }
                }
            }
            RES_MARK(12);
            // sixteen lanes per sample, two columns each
            __syncthreads();
            RES_MARK(13);
            const int tid = (x.wave * 64 + lane_id());
            if (tid < 16 * NT * 16) {
                // (two tiles: the first four waves the columns of the even rank, the others those of the odd one, as that rank's)
                const int side = NT == 2 ? x.wave >> 2 : half, rank = x.rank - half + side;
                const int at = tid >> 4, s = NT == 2 ? half * 16 + (at & 15) : at, col = (tid & 15) * 2, gcol = rank * 32 + col;
                const int n_tok = min(p.VT, p.pl.nout_m) - rank * 32;        // token columns among them
                const bool dur_cols = p.tdt && p.VT < p.pl.nout_m && rank * 32 + 32 > p.VT;      // they hold duration columns
                const int tcol = tcol0 + side;
                float2 o[kResWaves];
#pragma unroll
                for (int w = 0; w < kResWaves; ++w)
                    o[w] = *reinterpret_cast<const float2 *>(part + (w * NT * 16 + at) * kResSumRow + col);
                const float2 bias = rc.bo[side][tid & 15], scale = rc.so[side][tid & 15];
                static_assert(kResWaves == 8, "eight lanes add the waves' sums of the tail column");
                float tw = 0.f, back = 1.f;
                if constexpr (!BF && !WHOLE) back = inverse_power(rc.scale[lane_const >> 14 & (R - 1)]);
                const bool tail_here = side < n_tails;
                if (tail_here) tw = tpart[((tid & 7) * 2 + side) * 16 + (at & 15)];
                const float l0 = (((o[0].x + o[1].x) + (o[2].x + o[3].x)) + ((o[4].x + o[5].x) + (o[6].x + o[7].x))) * scale.x * back + bias.x;
                const float l1 = (((o[0].y + o[1].y) + (o[2].y + o[3].y)) + ((o[4].y + o[5].y) + (o[6].y + o[7].y))) * scale.y * back + bias.y;
                const float m0 = col < n_tok ? l0 : -INFINITY, m1 = col + 1 < n_tok ? l1 : -INFINITY;
                const float mine = fmaxf(m0, m1);
                float m = lane_max<16>(mine);
                // the first lane of the sixteen that holds the maximum publishes (without a token column: lane 0)
                const unsigned hit = (unsigned)(__ballot(mine == m && col < n_tok) >> (tid & 48)) & 0xffffu;
                const int first = hit ? __builtin_ctz(hit) : 0;
                int ix = hit ? (m0 == m ? gcol : gcol + 1) : 0x7fffffff;
                float tail = -INFINITY;
                if (tail_here) {
                    tail = lane_sum<8>(tw) * rc.st[side] * back + rc.bt[side];
                    if (tcol >= p.VT) {
                        if ((tid & 15) == 0) {
                            const unsigned d = ((unsigned)s * kMaxDur + (unsigned)(tcol - p.VT)) * 4u;
                            put(x, d, bo.dur + slot_at(jn, DSLOT), bo.dur + slot_at(jn + 2, DSLOT), word_of(tail));
                        }
                        tail = -INFINITY;
                    } else if (tail > m) {
                        m = tail; ix = tcol;
                    }
                }
                if (dur_cols) {
                    // duration columns inside the column tiles
#pragma unroll
                    for (int c = 0; c < 2; ++c)
                        if (gcol + c >= p.VT && gcol + c < p.pl.nout_m) {
                            const unsigned d = ((unsigned)s * kMaxDur + (unsigned)(gcol + c - p.VT)) * 4u;
                            put(x, d, bo.dur + slot_at(jn, DSLOT), bo.dur + slot_at(jn + 2, DSLOT), word_of(c ? l1 : l0));
                        }
                }
                const unsigned ko = ((unsigned)s * TS + (unsigned)rank) * 8u;
                if ((tid & 15) == first)
                    put2(x, ko, bo.key + slot_at(jn, KSLOT), bo.key + slot_at(jn + 2, KSLOT), (r2u){word_of(m), (unsigned)ix});
                if (p.logps) {
                    float e = (m0 > -INFINITY ? expf(m0 - m) : 0.f) + (m1 > -INFINITY ? expf(m1 - m) : 0.f);
                    e = lane_sum<16>(e);
                    if (tail > -INFINITY) e += expf(tail - m);
                    if ((tid & 15) == 0)
                        put(x, ko / 2, bo.lse + slot_at(jn, KSLOT / 2), bo.lse + slot_at(jn + 2, KSLOT / 2), word_of(e));
                }
            }
        }
        if constexpr (NT < NMT) {
            // the samples that this step does not have: the marks that their words of step jn + 2 need
            const int tid = x.wave * 64 + lane_id(), s = tid >> 4;
            if (s >= NS && s < NS * 2) {
                const int gcol = x.rank * 32 + (tid & 15) * 2, tcol = tcol0 + half;
                const bool dur_cols = p.tdt && p.VT < p.pl.nout_m && x.rank * 32 + 32 > p.VT;
                const unsigned ko = ((unsigned)s * TS + (unsigned)x.rank) * 8u, ds = (unsigned)s * kMaxDur * 4u;
                const bool lead = (tid & 15) == 0;
                if (lead) put_mark2(x, ko, bo.key + slot_at(jn + 2, KSLOT));
                if (lead && p.logps) put_mark(x, ko / 2, bo.lse + slot_at(jn + 2, KSLOT / 2));
                if (lead && half < n_tails && tcol >= p.VT) put_mark(x, ds + (unsigned)(tcol - p.VT) * 4u, bo.dur + slot_at(jn + 2, DSLOT));
                if (dur_cols) {
#pragma unroll
                    for (int c = 0; c < 2; ++c)
                        if (gcol + c >= p.VT && gcol + c < p.pl.nout_m)
                            put_mark(x, ds + (unsigned)(gcol + c - p.VT) * 4u, bo.dur + slot_at(jn + 2, DSLOT));
                }
            }
        }
        RES_MARK(14);
        // One layer: what the next prediction step's cells add to the row of T0, while the keys travel (one layer of 640, 32 utterances 870 us and 854
        // with it, 8 571 and 559, the small model 271 and 266.  Two layers in bfloat16 have no register for it; through LDS: no gain.)
        if constexpr (NL == 1)
            if (need_pred && has_cells) first_sum = sum_of(sums_top, rc.sh[0]);
        // ---- argmax over the team: TS / 2 adjacent lanes per sample, two candidates per lane --------
        {
            const int tid = (x.wave * 64 + lane_id()), lane = tid & 63;
            constexpr int L = TS / 2;
            static_assert(16 * NT * L <= kResThreads, "one piece per thread");
            const int s = tid / L;
            if ((x.wave * 64) / L < NS) {
                const unsigned off[1] = {(unsigned)tid * 16u};
                r4u v[1];
                // TDT: the sample's durations, one or two for each of the first lanes, come along
                constexpr int ND = L >= kMaxDur ? 1 : kMaxDur / L;
                const int li = lane & (L - 1), di = (li * ND) & (kMaxDur - 1);
                unsigned dv[ND];
                if (p.tdt) {
                    const int v0 = rc.dur[di], v1 = rc.dur[di + ND - 1];
                    unsigned spins = 0;
                    const unsigned o = ((off[0] / (L * 16u)) * kMaxDur + (unsigned)di) * 4u;
                    for (;;) {
                        v[0] = get4(x, off[0], bo.key + slot_at(jn, KSLOT));
                        bool missing = false;
#pragma unroll
                        for (int i = 0; i < ND; ++i) dv[i] = get1(x, o + i * 4u, bo.dur + slot_at(jn, DSLOT));
#pragma unroll
                        for (int i = 0; i < ND; ++i) missing = missing || (di + i < p.D && dv[i] == kMark);
                        if (__ballot(missing || has_mark(v[0])) == 0ull) break;
                        if (wait_expired(p, spins)) { rc.ok = 0; break; }
                    }
                    x.polls += __builtin_amdgcn_readfirstlane((int)spins);
                    // best duration, the lowest index on ties, and the first one where all are NaN
                    const float d0 = di < p.D ? __uint_as_float(dv[0]) : -INFINITY, d1 = ND > 1 && di + 1 < p.D ? __uint_as_float(dv[ND - 1]) : -INFINITY;
                    const float dm = lane_max<L>(fmaxf(d0, d1));
                    const bool odd = ND > 1 && di + 1 < p.D && d1 == dm && d0 != dm;
                    const unsigned hit = (unsigned)(__ballot((d0 == dm && di < p.D) || odd) >> (lane & ~(L - 1))) & ((1u << L) - 1u);
                    if (li == (hit ? __builtin_ctz(hit) : 0)) rc.s_d[s] = odd ? v1 : v0;
                } else {
                    receive<1>(p, x, off, bo.key + slot_at(jn, KSLOT), v);
                }
                const float va = __uint_as_float(v[0].x), vb = __uint_as_float(v[0].z);
                const int ia = (int)v[0].y, ib = (int)v[0].w;
                const bool second = vb > va || (vb == va && ib < ia);
                const float bv = second ? vb : va;
                const int bi = second ? ib : ia;
                const float m = lane_max<L>(bv);
                // ranks hold ascending columns; tail columns come after all others
                const bool top = bv == m;
                const unsigned h1 = (unsigned)(__ballot(top && bi < p.pl.nout_m) >> (lane & ~(L - 1))) & ((1u << L) - 1u);
                const unsigned h2 = (unsigned)(__ballot(top) >> (lane & ~(L - 1))) & ((1u << L) - 1u);
                const bool win = (lane & (L - 1)) == __ffs((int)(h1 ? h1 : h2)) - 1;
                float lp2 = 0.f;
                if (p.logps) {
                    unsigned e0, e1, spins = 0;
                    for (;;) {
                        e0 = get1(x, off[0] >> 1, bo.lse + slot_at(jn, KSLOT / 2));
                        e1 = get1(x, (off[0] >> 1) + 4u, bo.lse + slot_at(jn, KSLOT / 2));
                        if (__ballot(e0 == kMark || e1 == kMark) == 0ull) break;
                        if (wait_expired(p, spins)) { rc.ok = 0; break; }
                    }
                    // a work-group without a token column has -inf for its maximum and contributes nothing
                    float t = 0.f;
                    if (va > -INFINITY) t += __uint_as_float(e0) * expf(va - m);
                    if (vb > -INFINITY) t += __uint_as_float(e1) * expf(vb - m);
                    t = lane_sum<L>(t);
                    lp2 = -logf(t);
                }
                if (win) {
                    rc.s_k[s] = (unsigned)bi < (unsigned)p.VT ? bi : p.blank;
                    rc.s_v[s] = m + 0.0f;
                    if (p.logps) rc.s_lp[s] = lp2;
                }
            }
            RES_MARK(15);
        }
        // ---- loop control of one utterance: the same, with everything but the results of the frames uniform -------------------
        // (Tables of rows, their places in a step and the choice of those that wait are nothing to one row.  us a call: one utterance 341 and 326, five with
        // log-probabilities 229 and 222, small model, eight, 263 and 244, multi-blank, four, 308 and 292, bfloat16 mode, eight, 161 and 152.)
        if constexpr (ONE) {
            const int lane = lane_id(), at = lane & 15;
            if (PAIR) load_pre(n_pred, 0, pre[0]);           // (as below)
            __syncthreads();
            RES_MARK(16);
            if (FRAMES_FIRST && !has_cells) __builtin_amdgcn_s_setprio(2);
            const int mine = rc.s_k[at], left = only.len - only.t, avail = min(16, left);
            int pos = 0, dval = 0;
            bool found = false;
            if (!(p.tdt || p.VT != p.V1)) {
                pos = __builtin_ctz(((unsigned)__ballot(mine != p.blank) & 0xffffu) | 1u << avail);
                found = pos < avail;
            } else {
                // where the walk goes to from every frame, then frame by frame
                int d = 0;
                if (mine >= p.V1) d = max(rc.dur[(mine - p.V1) & (kMaxDur - 1)], 1);            // big blank: its span of frames
                else if (mine == p.blank) d = p.tdt ? min(max(rc.s_d[at], 1), kFarthest) : 1;
                const unsigned labels = (unsigned)__ballot(d == 0);
                while (pos < avail && !(found = (labels >> pos & 1u) != 0u)) pos += __builtin_amdgcn_readlane(d, pos);
            }
            const bool writer = x.rank == 0 && x.wave == kResWaves - 1 && lane == 0;
            int adv = pos;
            if (adv > 0) only.n = 0;
            if (found) last = __builtin_amdgcn_readlane(mine, pos);
            load_t0();
            if (found) {
                if (p.tdt) dval = __builtin_amdgcn_readfirstlane(rc.s_d[pos]);
                if (writer) {
                    const Args a = args_again();
                    if (only.cnt < a->cap) {
                        const long long o = (long long)only_b * a->cap + only.cnt;
                        a->tokens[o] = last;
                        if (a->frames) a->frames[o] = only.t + pos;
                        if (a->logits) a->logits[o] = rc.s_v[pos];
                        if (a->logps) a->logps[o] = rc.s_lp[pos];
                        if (a->durs) a->durs[o] = dval;
                    } else {
                        rc.st_overflow = 1;
                    }
                }
                ++only.cnt;
                if (p.tdt && dval > 0) { adv += min(dval, kFarthest); only.n = 0; }
                else if (++only.n == p.S) { ++adv; only.n = 0; }
            }
            any_active = adv < left;
            only.t += adv;
            if (!any_active && writer) res_finish_row(only_b, only.cnt);
            need_pred = found && any_active;
            lane_const = (lane_const & ~(kTake | kFresh)) | (need_pred ? kTake : 0);
            const int now = min(16, only.len - only.t);
            pidx = at < now ? only_b * p.T + only.t + at : -1;
            if (any_active) n_samples += now;
            if (need_pred) ++row_steps;
        } else
        // ---- loop control: every wave for itself, lane = row (outputs: the last wave, which has the least to do next) ------
        {
            const int lane = lane_id(), r = (int)((unsigned)lane / LR) & (R - 1);
            RRow w = rows.s[r];
            int b = rows.b[r];
            // (on its way during the rest: the helpers' results take 0.85 us, and what is left of the step 0.75)
            if (PAIR) load_pre(n_pred, 0, pre[0]);
            __syncthreads();
            RES_MARK(16);
            if (FRAMES_FIRST && !has_cells) __builtin_amdgcn_s_setprio(2);
            const int mine = rc.s_k[lane & (kResSamples - 1)], row0 = lane_const >> 25 & 31;
            // (a row that does not take part has nothing left for now)
            const bool in = (part_rows >> (lane & (16 - LR)) & 1u) != 0u;
            const int left = in ? w.len - w.t : 0;
            const bool lead = lane < 16 && (lane & (LR - 1)) == 0;     // stands for its row
            const bool writer = x.rank == 0 && x.wave == kResWaves - 1 && lead;
            const bool walk = p.tdt || p.VT != p.V1;
            int pos, dval = 0;
            bool found;
            if (!walk) {
                // a blank moves on by one frame: the first label among the frames the row still has
                const unsigned labels = (unsigned)__ballot(mine != p.blank);
                const unsigned avail = (unsigned)max(0, min(la, left));
                pos = __builtin_ctz((labels >> row0) | (1u << avail));
                found = pos < (int)avail;
            } else {
                // lane = sample: the offset (from the row's frame) that the walk goes to from it, its own for a label
                // or beyond the row's frames, and the lane of that offset, its own where the walk leaves the step;
                // then the hops are doubled until every one reaches its end
                const int si = lane_const >> 20 & 31;
                int d = 0;
                if (mine >= p.V1) d = max(rc.dur[(mine - p.V1) & (kMaxDur - 1)], 1);            // big blank: its span of frames
                else if (mine == p.blank) d = p.tdt ? min(max(rc.s_d[lane & (kResSamples - 1)], 1), kFarthest) : 1;
                if (pidx < 0) d = 0;
                const int to = si + d;
                int hop = (d > 0 && to < la ? lane + d : lane) << 2;
                for (int i = 1; i < la; i *= 2) hop = __builtin_amdgcn_ds_bpermute(hop, hop);
                hop = __builtin_amdgcn_ds_bpermute(row0 << 2, hop);
                pos = __builtin_amdgcn_ds_bpermute(hop, to);
                found = pos < la && pos < left;
            }
            const int s = min(row0 + pos, kResSamples - 1);
            const int k = rc.s_k[s];
            if (p.tdt) dval = rc.s_d[s];
            // the label's row of the embedding table is what the next prediction step waits for
            if (found) last = k;
            load_t0();
            int adv = left > 0 ? pos : 0;
            if (adv > 0) w.n = 0;
            if (found) {
                if (writer) {
                    const Args a = args_again();
                    if (w.cnt < a->cap) {
                        const long long o = (long long)b * a->cap + w.cnt;
                        a->tokens[o] = k;
                        if (a->frames) a->frames[o] = w.t + pos;
                        if (a->logits) a->logits[o] = rc.s_v[s];
                        if (a->logps) a->logps[o] = rc.s_lp[s];
                        if (a->durs) a->durs[o] = dval;
                    } else {
                        rc.st_overflow = 1;
                    }
                }
                ++w.cnt;
                if (p.tdt && dval > 0) { adv += min(dval, kFarthest); w.n = 0; }
                else if (++w.n == p.S) { ++adv; w.n = 0; }
            }
            w.t += adv;
            const bool ended = left > 0 && adv >= left;
            int action = found && !ended ? kTake : 0;
            if (__ballot(ended) != 0ull) {
                if (writer && ended) res_finish_row(b, w.cnt);
                const bool got = refill(lane, ended, b, w.len);
                if (got) { w.t = w.n = w.cnt = 0; action = kFresh; last = p.blank; }
                if (lead) rows.b[r] = b;
                load_t0();
            }
            if (in) lane_const = (lane_const & ~(kTake | kFresh)) | action;
            const unsigned active = (unsigned)(__ballot(w.t < w.len) & LEADS);
            const unsigned moved = (unsigned)__ballot((lane_const & (kTake | kFresh)) != 0) & active;      // rows whose next step has new inputs
            any_active = active != 0u;
            if (active != active_rows) { active_rows = active; takers = res_takers(R, active); }
            const int n_moved = __builtin_popcount(moved), n_search = __builtin_popcount(active) - n_moved;
            // The next step is a prediction step if a row has new inputs, unless half as many or more are still looking for
            // their label: then these have the next joint step, and all its samples, to themselves, at 4 us instead of 8 (two-layer fp32
            // models) or 6.5.  But where no utterance waits for a row any more, the row with the most frames left does not wait: it is what
            // the team's time ends with.  (32 utterances, three draws, with a prediction step at every label 1402, 1383 and 1242 us, against
            // 1348, 1367 and 1182; as many or more still looking, and the longest never waiting, against half as many and only without
            // a queue: 1037, 1264, 1303 and 1059, 1245, 1238, bfloat16 mode 777, 846, 843 and 768, 836, 834, 57 with e4m3 weights 644 and 635, 128 utterances
            // 3807 and 3721.  Whoever has the most frames left: bfloat16 mode up to 4 % and the multi-blank model up to 3.5 % slower than
            // with a step at every label.)
            int most = w.len - w.t;
            const int rest = most;
            if constexpr (R == 8) asm("s_nop 1\n\tv_max_i32_dpp %0, %0, %0 row_ror:2 row_mask:0xf bank_mask:0xf" : "+v"(most));
            asm("s_nop 1\n\tv_max_i32_dpp %0, %0, %0 row_ror:4 row_mask:0xf bank_mask:0xf\n\t"
                "s_nop 1\n\tv_max_i32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf" : "+v"(most));
            const unsigned longest = (unsigned)__ballot(rest == most) & active;
            need_pred = n_moved != 0 && (NT < NMT || n_moved > 2 * n_search || (!queued && (longest & ~moved) == 0u));
            const unsigned next = need_pred || n_moved == 0 ? active : active & ~moved;
            if (next != part_rows && any_active) {
                // (a row has ended for good, or some go on looking alone: its samples go to the others)
                lay_out(nt_, lane, next);
            }
            if (lead) rows.s[r] = w;
            if (need_pred) row_steps += n_moved;
            if constexpr (HALVES && NT == NMT) {
                // every so many steps: have all rows in work gone on by less than one and a half frames a step?
                // (No lane condition around the store: `change` would count as different from lane to lane.)
                if ((jn & (kResCalm - 1)) == 0) {
                    const int from = rows.since[r], on = w.t < from ? w.t : w.t - from;
                    change = __ballot(w.t < w.len && on > kResCalm * 3 / 2) == 0ull;
                    rows.since[r] = w.t;
                }
            }
            if constexpr (NT < NMT) change = __ballot(left > 0 && !found && !ended) != 0ull;      // a row's next label is further away
            // Before a prediction step the waves with cells do it when they have published theirs: it is off the chain there.
            // (32 utterances 1308, 1321, 1151 us with it here, 1291, 1305, 1142 there, bfloat16 mode 836, 941, 892 and 812, 918, 869.
            // One or two rows a team: 530 and 538 us for one utterance, the polls are later there than the words.)
            later = NMT == 2 && need_pred && has_cells && !change;
            if (!change && !later) set_up_samples(lane, w.t, b, w.len);
        }
        ok = rc.ok != 0;
        RES_MARK(17);
    }
    };
    if constexpr (!HALVES) {
        steps(all_tiles);
    } else {
        // Where the rows go on by less than one and a half frames a step (ten labels on every frame, say), the second
        // tile of samples is computed for nothing: then the team goes on with half the frames per row, until
        // a row's next label is not among them.  128 utterances of ten labels on every frame: 8.4 us a step with two
        // tiles, 7.7 with one (100.7 and 92.1 ms a call), and with ten labels on every other frame 50.5 and 46.2 ms a
        // call.  At 0.7 labels a frame the two are even; below, a team hardly ever
        // gets here, and what looking out for it costs is within 0.6 % of a call.
        // Two-layer fp32 models only: the others were faster than the streaming kernel on such input as well, and
        // their second loop costs more registers than there are (bfloat16 mode: twelve spilled, 4 to 6 % of a call).
        std::integral_constant<int, 1> one_tile;
        auto changed_to = [&](auto nt_) {
            const int lane = lane_id(), r = (int)((unsigned)lane / LR) & (R - 1);
            const RRow w = rows.s[r];
            lay_out(nt_, lane, part_rows);
            if (lane < 16 && (lane & (LR - 1)) == 0) rows.since[r] = -0x10000000;      // (not after less than kResCalm steps)
            set_up_samples(lane, w.t, rows.b[r], w.len);
        };
        for (;;) {
            steps(all_tiles);
            if (!ok || !any_active) break;
            changed_to(one_tile);
            steps(one_tile);
            if (!ok || !any_active) break;
            changed_to(all_tiles);
        }
    }
    __syncthreads();
    if (PAIR && rc.ok) {
        // the helpers wait for the next candidate vectors: tell them that there are none
        const unsigned o = slot_at(n_pred + 1, VSLOT);
        for (int i = threadIdx.x; i < p.slots * nu; i += kResThreads) {
            const int r = i / nu, u = i - r * nu;
            put_far(x, (unsigned)r * VROW + (unsigned)(u0 + u) * 4u, bo.hr[0] + o, kStop);
            put_far(x, (unsigned)r * VROW + (unsigned)(u0 + u) * 4u, bo.hr[1] + o, kStop);
        }
    }
    if (threadIdx.x == 0) {
        int st = 0;
        if (x.rank == 0) st = (rc.st_clamped ? 1 : 0) | (rc.st_overflow ? 2 : 0);
        if (!rc.ok) st |= 4;
        if (st) __hip_atomic_fetch_or(p.status, st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (x.rank == 0) {
            long long *sp = p.stats + (long long)team * kStatStride;
            if (p.zero_stats) { sp[kStatPred] = 0; sp[kStatJoint] = 0; sp[kStatSamples] = 0; sp[kStatPolls] = 0; }
            sp[kStatPred] += p.count_rows ? row_steps : (int)n_pred; sp[kStatJoint] += n_joint; sp[kStatSamples] += n_samples; sp[kStatPolls] += x.polls;
            atomicMax(reinterpret_cast<unsigned long long *>(p.stats + kStatDecodeEnd), (unsigned long long)wall_clock64());
#ifdef RNNT_PROFILE
            for (int i = 0; i < 24; ++i) sp[kStatCount + i] = res_prof[i];
#endif
        }
    }
}

template <int KIND, bool BF, int CLS, int NMT, int R, bool ONE = false>
hipError_t launch_resident_one(const ResidentParams &p, bool plain, hipStream_t stream, hipEvent_t end)
{
    const void *fn = reinterpret_cast<const void *>(&resident_kernel<KIND, BF, CLS, NMT, R, ONE>);
    constexpr unsigned lds = (unsigned)resident_lds(KIND, BF, CLS, NMT, R).bytes;
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ResidentParams pc = p;
    void *args[] = {&pc};
    const dim3 grid(p.pl.n_xcd * 32), block(kResThreads);
    if (plain) return launch_ending(fn, grid, block, args, lds, stream, end);
    return hipLaunchCooperativeKernel(fn, grid, block, args, lds, stream);
}

}  // namespace
}  // namespace rnnt
