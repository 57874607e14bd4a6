// Decode kernel with register-resident weights (device code, instantiated by resident_inst.hip).
//
// The step chain of a decode (a prediction step, a joint step, and again) is bound by latency:
// three dense stages and four hand-overs between work-groups per label.  Two things make it
// short here.  (1) Every weight of the step is held in the registers of one compute unit for the
// whole launch: eight waves of 256 registers, of which up to 196 hold weights, so a stage reads
// nothing but its input vector (streamed out of L2, the weights took 5 to 27 us of a step).  (2) A team
// of work-groups sits inside one XCD, so its hand-overs go through that XCD's L2: a store that stays
// in the L2 and a load that passes by the L1 hand 640 floats to 32 work-groups in 0.70 us, where
// stores and loads through the memory side take 1.3 us (4 x 640 floats: 0.88 against 1.4 us).
// 32 utterances of a two-layer model of 640 units: 4.35 to 2.06 ms, one of 500 frames 1.63 to 0.53 ms.
//
// Work split inside a team of `ts` work-groups: LSTM units, projection columns and output columns
// in contiguous ranges.  LSTM stages and the projection run on v_mfma 4x4 (16 blocks): the rows of a
// block are four utterances, its columns the gates of a unit or four columns, K is split over the waves
// and the partial sums meet in LDS.  The joint output runs on v_mfma 16x16 (16 columns x 16 samples,
// two column tiles, K in eighths over the waves); its operand relu(P + q) is formed on the way from
// LDS to the matrix instruction.
//
// Two-layer fp32 models have more weights than one XCD's registers hold (24 MB against 12 + 4):
// there the teams' XCDs keep the input, projection and output matrices and run the whole step chain;
// the helpers' XCDs keep the recurrent matrices and compute W_hh h of the candidate states, which the
// chain needs only at the next label: their hand-overs across the XCDs run beside the rest of the
// step.  A helper is busy 3 us of a team's step and serves two teams: 128 utterances 7.7 ms with one team
// per helper, 6.5 with five teams on three XCDs of helpers, 7.1 with six on two.
//
// Utterances are decoded label-looping fashion: every utterance has its own frame index, a joint
// step examines `la` frames of every utterance (half as many in label-dense stretches of two-layer fp32
// models, see the end of the loop), and the next prediction step runs as soon as one
// of them has a label.  A team takes a list of utterances and decodes up to kResRows at a time;
// when one ends the next of the list takes its place.  (Eight rows of four frames took 15 us a step
// where four rows of eight take 10.)
//
// Exchange: a vector's buffer has four slots used in turn; words are 32-bit floats, all ones
// meaning "not there yet" (readers poll the data itself).  A work-group puts that mark back into
// slot n - 2 when it publishes step n: by then it has received something of step n - 1 from
// everyone, which everyone sent after reading step n - 2; and it waits for that store before it
// publishes step n + 1, so nobody can look for step n + 2's data in a slot that still holds old data.
//
// Registers decide what the code looks like: values that could be kept for the whole loop are worked out
// where they are used (lane_id), state that few waves need lies in LDS, arguments that few steps need are
// read again (args_again).  A spilled weight is a load from memory in the middle of a stage.
#pragma once
#include <type_traits>

#include "engine.h"
#include "gate.h"
#include "resident.h"

namespace rnnt {
namespace {

typedef float r4f __attribute__((ext_vector_type(4)));
typedef unsigned r4u __attribute__((ext_vector_type(4)));
typedef unsigned r2u __attribute__((ext_vector_type(2)));
typedef short r4s __attribute__((ext_vector_type(4)));
typedef __bf16 r8b __attribute__((ext_vector_type(8)));

constexpr unsigned kMark = 0xffffffffu;    // no data yet
constexpr unsigned kStop = 0xfffffffeu;    // to the helpers: the team is done

// Rows in work: every wave keeps a copy of its own and takes the same decisions from the same
// results, so loop control needs no work-group barrier.
struct __align__(16) RRow { int t, len, n, cnt; };       // frame, frames, labels of this frame, labels; t >= len: idle
struct RRows {
    RRow s[kResRows];
    int b[kResRows], m[kResRows];     // utterance; t modulo the frames of a joint step
    int since[kResRows], next;        // t some steps ago; first utterance of the list that no row has had
};

struct RCtl {
    RRows rows[kResWaves];
    int s_k[kResSamples], s_d[kResSamples];        // results of a joint step
    float s_v[kResSamples], s_lp[kResSamples];
    int n_list, ok, st_clamped, st_overflow;
    int dur[kMaxDur];
    unsigned seen[2][kResWaves];      // helpers: what a wave has seen of the teams' vectors
    int list_b[kResList], list_len[kResList];
    // this work-group's slices of the biases: second layer [unit][gate], projection, output and tail column
    float b1[kResUnits * 4], bp[20], bo[32], bt;
};
__shared__ RCtl rc;
static_assert(sizeof(RCtl) <= kResCtl, "the control block has its place");

// Phase timers (100 MHz wall clock), compiled in only for profiling builds.
#ifdef RNNT_PROFILE
__shared__ long long res_prof[24];
__shared__ long long res_prof_last;
#define RES_MARK(slot) do { __builtin_amdgcn_sched_barrier(0); if (threadIdx.x == 0) { long long t_ = wall_clock64(); res_prof[slot] += t_ - res_prof_last; res_prof_last = t_; } __builtin_amdgcn_sched_barrier(0); } while (0)
#else
#define RES_MARK(slot) do { } while (0)
#endif

template <int N> struct RegW { float w[N]; };

// Loads registers [first, first + N) of the wave's packed run.  The empty asm makes each value
// opaque, so that it stays in its register and is never read from memory again.
template <int N>
__device__ __forceinline__ void load_regs(RegW<N> &r, const float *src, int first, int lane)
{
#pragma unroll
    for (int i0 = 0; i0 < N; i0 += 32) {          // 32 loads in flight
#pragma unroll
        for (int i = i0; i < N && i < i0 + 32; ++i) r.w[i] = src[(first + i) * 64 + lane];
#pragma unroll
        for (int i = i0; i < N && i < i0 + 32; ++i) asm volatile("" : "+v"(r.w[i]));
    }
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
    const r2u mark = {kMark, kMark};
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
    const r2u mark = {kMark, kMark};
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
__device__ __forceinline__ void receive(const ResidentParams &p, RCtx &x, const unsigned (&off)[N], unsigned imm, r4u (&v)[N])
{
    unsigned spins = 0;
    for (;;) {
        bool missing = false;
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = get4(x, off[i], imm);
#pragma unroll
        for (int i = 0; i < N; ++i) missing = missing || has_mark(v[i]);
        if (__ballot(missing) == 0ull) break;
        if (wait_expired(p, spins)) { rc.ok = 0; break; }
    }
    x.polls += __builtin_amdgcn_readfirstlane((int)spins);
}

// two fp32 values as bf16 (ties to even), first in the low half
__device__ __forceinline__ unsigned bf16_pair(float a, float b)
{
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    const f2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, b2));
}

// Stores piece k4 (four values) of an activation row in LDS.
template <bool BF>
__device__ __forceinline__ void x_put(unsigned char *row, int k4, r4u v)
{
    if (BF) {
        uint2 o;
        o.x = bf16_pair(__uint_as_float(v.x), __uint_as_float(v.y));
        o.y = bf16_pair(__uint_as_float(v.z), __uint_as_float(v.w));
        *reinterpret_cast<uint2 *>(row + k4 * 8) = o;
    } else {
        *reinterpret_cast<r4u *>(row + k4 * 16) = v;
    }
}

// A piece of K of an activation row, and the matrix instructions that take it: four fp32 (e = 0 .. 3)
// or one bf16.
template <bool BF> struct Piece;
template <> struct Piece<false> {
    static constexpr int N = 4, B = 16;
    float4 v;
    __device__ __forceinline__ void load(const unsigned char *p) { v = *reinterpret_cast<const float4 *>(p); }
    // S, ID: the blocks form groups of 2^S that all take the operand of block ID of their group
    template <int S = 0, int ID = 0>
    __device__ __forceinline__ void mfma(int e, const float *w, r4f &acc) const
    {
        acc = __builtin_amdgcn_mfma_f32_4x4x1f32(e == 0 ? v.x : (e == 1 ? v.y : (e == 2 ? v.z : v.w)), w[e], acc, S, ID, 0);
    }
};
template <> struct Piece<true> {
    static constexpr int N = 1, B = 8;
    r4s v;
    __device__ __forceinline__ void load(const unsigned char *p) { v = *reinterpret_cast<const r4s *>(p); }
    template <int S = 0, int ID = 0>
    __device__ __forceinline__ void mfma(int, const float *w, r4f &acc) const
    {
        struct P { float a, b; };
        acc = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(v, __builtin_bit_cast(r4s, P{w[0], w[1]}), acc, S, ID, 0);
    }
};

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

__device__ __forceinline__ void swap32(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap16(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
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

// One LSTM stage over the wave's part of K: partial sums of the work-group's units for all rows go to
// LDS, [row group][wave][lane] with a lane's four rows; the readers add six or eight of them
// (stage_sum), so there are no sums across lanes.  The activation rows x are read once: lane 4 b + r
// fetches another piece of row r for every block b, and the matrix instruction's broadcast hands each of
// them to all blocks in turn (waves 6 and 7: to the four blocks of a slice of K).  Reading a piece
// once per block instead kept the LDS as busy as the matrix cores: 2.8 against 1.9 us for eight rows.
template <bool BF, int CLS>
__device__ __forceinline__ void lstm_stage(const RegW<res_lstm_regs(BF, CLS)> &w, const unsigned char *x, int h4, float *sums, int wave, int lane)
{
    constexpr int N = res_lstm_pieces(CLS), N8 = res_pieces(CLS) / 8, PR = res_piece_regs(BF), XROW = res_xrow(BF, CLS);
    typedef Piece<BF> Pc;
    r4f acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    const int b = lane >> 2;
    const unsigned char *xr = x + (lane & 3) * XROW;       // (pieces beyond the last have zero weights: the last will do)
    if (wave < 6) {
        constexpr int Q = (N + 15) / 16;
        Pc q[Q];
#pragma unroll
        for (int h = 0; h < Q; ++h) q[h].load(xr + min(wave * N + h * 16 + b, h4 - 1) * Pc::B);
        static_for<0, N>([&](auto i_) {
            constexpr int i = decltype(i_)::value;
#pragma unroll
            for (int e = 0; e < Pc::N; ++e) q[i / 16].template mfma<4, i % 16>(e, &w.w[i * PR], acc[(i * Pc::N + e) & 1]);
        });
    } else {
        constexpr int Q = (N8 + 3) / 4;
        Pc q[2];
        auto fetch = [&](int h) { q[h & 1].load(xr + min((h * 4 + (b & 3)) * 8 + (wave - 6) * 4 + (b >> 2), h4 - 1) * Pc::B); };
        fetch(0);
        static_for<0, Q>([&](auto h_) {
            constexpr int h = decltype(h_)::value;
            if constexpr (h + 1 < Q) fetch(h + 1);
            __builtin_amdgcn_sched_barrier(0);
            static_for<h * 4, (h * 4 + 4 < N8 ? h * 4 + 4 : N8)>([&](auto i_) {
                constexpr int i = decltype(i_)::value;
#pragma unroll
                for (int e = 0; e < Pc::N; ++e) q[h & 1].template mfma<2, i % 4>(e, &w.w[i * PR], acc[(i * Pc::N + e) & 1]);
            });
        });
    }
    *reinterpret_cast<r4f *>(sums + (wave * 64 + lane) * 4) = acc[0] + acc[1];
}

// The stage's sum for lane `lane` of wave `blk` < 5: unit 4 blk + lane / 16, row lane / 4 % 4, gate lane % 4.
__device__ __forceinline__ float stage_sum(const float *sums, int blk, int lane)
{
    const int uu = lane >> 4, row = (lane >> 2) & 3, j = lane & 3;
    const float *s = sums + row;
    if (blk < 4) {
        s += (4 * (blk * 4 + uu) + j) * 4;
        return (s[0] + (s[256] + s[512])) + (s[768] + (s[1024] + s[1280]));
    }
    s += 6 * 256 + (4 * uu + j) * 4;         // slices 64 floats apart
    return ((s[0] + s[64]) + (s[128] + s[192])) + ((s[256] + s[320]) + (s[384] + s[448]));
}

// LSTM cell on the four lanes of a block: lane j holds the pre-activation of gate j (i, f, g, o).
// Every lane of the block gets the results.
__device__ __forceinline__ void cell(float pre, int j, float c_old, float &c_new, float &h)
{
    const float act = gate_act(pre, j == 2);
    const float i_ = dppf<0x00>(act), f_ = dppf<0x55>(act), g_ = dppf<0xAA>(act), o_ = dppf<0xFF>(act);
    c_new = fmaf(f_, c_old, i_ * g_);
    h = o_ * gate_act(c_new, true);
}

// What the prediction step does with a row's candidate state: take it, or start afresh (else nothing).
constexpr int kTake = 1 << 30, kFresh = (int)(1u << 31);

#define RES_SLOT(n) ((unsigned)(n) & (kResSlots - 1))

// Receives a vector of `rows` rows of n4 16-byte pieces each (rows row_bytes apart from byte `base`
// of the exchange buffers on) and hands every piece to f(row, k4, words).
// (piece i of a thread: number piece_index, of row piece_row; threads beyond the vector read its last
// piece along)
__device__ __forceinline__ unsigned piece_index(unsigned tid, int i, int n) { return min(tid + (unsigned)(i * kResThreads), (unsigned)(n - 1)); }
__device__ __forceinline__ unsigned piece_inverse(int n4) { return ((1u << 20) + (unsigned)n4 - 1u) / (unsigned)n4; }     // idx / n4 for idx * n4 < 2^20, idx < 2^11
__device__ __forceinline__ unsigned piece_row(unsigned idx, unsigned inv) { return __umul24(idx, inv) >> 20; }
template <int WIDTH>
__device__ __forceinline__ unsigned piece_offset(unsigned idx, unsigned inv, int n4)
{
    return __umul24(piece_row(idx, inv), WIDTH * 4u - (unsigned)n4 * 16u) + idx * 16u;
}
template <int WIDTH, class F>
__device__ __forceinline__ void receive_rows(const ResidentParams &p, RCtx &x, unsigned base, int rows, int n4, F f)
{
    constexpr int N = (kResRows * (WIDTH / 4) + kResThreads - 1) / kResThreads;
    unsigned off[N];
    r4u v[N];
    const unsigned tid = (unsigned)(x.wave * 64 + lane_id()), inv = piece_inverse(n4);
#pragma unroll
    for (int i = 0; i < N; ++i) off[i] = piece_offset<WIDTH>(piece_index(tid, i, rows * n4), inv, n4);
    receive<N>(p, x, off, base, v);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const unsigned idx = piece_index(tid, i, rows * n4), r = piece_row(idx, inv);
        f((int)r, (int)(idx - __umul24(r, (unsigned)n4)), v[i]);
    }
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

// Loads row `row` of the projected frames into sample s's place in LDS, straight from memory.  The
// 16-byte piece k4 goes to position (k4 with its low four bits xored with s), so that sixteen samples'
// pieces of the same k sit in different banks.  (The instruction's offset counts on both sides.)
template <int ROW>
__device__ __forceinline__ void load_frame(const ResidentParams &p, const RCtx &x, unsigned lds_p, int row, int s)
{
    const int lane = lane_id(), j4 = p.J >> 2, k4 = lane ^ (s & 15);
    const char *src = reinterpret_cast<const char *>(p.P + (long long)row * p.J);
    const unsigned m = (unsigned)__builtin_amdgcn_readfirstlane((int)(lds_p + (unsigned)(s * ROW * 4)));
    static_for<0, (ROW / 4 + 63) / 64>([&](auto u_) {
        constexpr int u = decltype(u_)::value;
        const char *from = src;
        const unsigned to = m, off = (unsigned)k4 * 16u;
        if (((u + 1) * 64 <= ROW / 4 || lane < ROW / 4 - u * 64) && (j4 == ROW / 4 || u * 64 + k4 < j4))
            asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2 offset:%3"
                         :: "v"(off), "s"(to), "s"(from), "n"(u * 1024) : "memory");
    });
}

__device__ __forceinline__ int from_lane(int v, int lane) { return __builtin_amdgcn_ds_bpermute(lane << 2, v); }

// KIND: ResidentKind; BF: bfloat16 mode; CLS: size class; NMT: tiles of 16 samples of a joint step
template <int KIND, bool BF, int CLS, int NMT>
__global__ void __launch_bounds__(kResThreads, 1) resident_kernel(const ResidentParams p)
{
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int NL = KIND == kResident1 ? 1 : 2;
    constexpr bool PAIR = KIND == kResident2Pair;
    constexpr int W = res_width(CLS), ROW = res_row(CLS), TS = res_team(CLS), XROW = res_xrow(BF, CLS);
    constexpr int NI = res_joint_steps(CLS), PR = res_piece_regs(BF), LREGS = res_lstm_regs(BF, CLS);
    typedef Piece<BF> Pc;
    constexpr bool HALVES = PAIR && NMT == 2;     // steps with one tile of samples as well, see after the loop
    constexpr int NREC = PAIR ? 0 : NL;          // recurrent matrices the chain's work-groups hold
    constexpr ResidentBuf bo = resident_buf(CLS);
    constexpr ResidentLds lo = resident_lds(KIND, BF, CLS, NMT);
    constexpr unsigned VROW = W * 4u, VSLOT = kResRows * VROW;                      // h and q rows
    constexpr unsigned KSLOT = kResSamples * TS * 8u, DSLOT = kResSamples * kMaxDur * 4u;
    constexpr unsigned PSLOT = TS * 5u * 64u * 4u;

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
    // this work-group's team; a helper's first, and every helper_xcds-th one of the same place after it
    const int team = (helper ? xcd - chain_xcds : xcd) + chain_xcds * (place / TS);
    auto serves = [&](int i) { return team % chain_xcds + i * helper_xcds < chain_xcds && list_of(team + i * helper_xcds) > 0; };
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
        put_marks(0u, PAIR ? bo.pre : bo.hr[0]);
    } else {
        bool any = false;
        for (int i = 0; i < kResServed; ++i)
            if (serves(i)) { x.buf = buffers_of(team + i * helper_xcds); put_marks(bo.pre, bo.bytes); any = true; }
        if (!any) return;
    }
    if (tid0 == 0) { rc.ok = 1; rc.n_list = 0; rc.st_clamped = 0; rc.st_overflow = 0; }
    if (tid0 < kResSamples) { rc.s_k[tid0] = p.blank; rc.s_d[tid0] = 0; }
    if (tid0 < kMaxDur) rc.dur[tid0] = p.durations[tid0];
    if (lane0 < kResRows) {
        RRows &w = rc.rows[x.wave];
        w.s[lane0] = RRow{0, 0, 0, 0}; w.b[lane0] = w.m[lane0] = w.since[lane0] = w.next = 0;
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
    // Waits for team t in the first wave, lanes 0 .. TS-1 for the chain's work-groups and (both) lanes 32 .. for
    // its helpers; true when the chain's all sit on one XCD.
    auto meet = [&](int t, bool both) {
        const int side = lane0 >> 5, r = lane0 & 31;
        const bool mine = x.wave == 0 && r < TS && (side == 0 || both);
        unsigned v = 1;
        if (mine) {
            const int on = t % chain_xcds, at = side ? chain_xcds + on % helper_xcds : on;
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
    const bool has_cells = x.wave < 5;          // finishes 16 (unit, row) pairs of the LSTM stages, see stage_sum
    auto prelane = [&]() { return (((unsigned)x.rank * 5u + (unsigned)x.wave) * 64u + (unsigned)lane_id()) * 4u; };
    const int h4 = p.H >> 2;

    if (PAIR && helper) {
        // ---- helpers: W_hh of both layers times the candidate vectors ------------------------
        RegW<LREGS> w0, w1;
        const float *src = p.w_help + (long long)(x.rank * kResWaves + x.wave) * (2 * LREGS) * 64;
        load_regs(w0, src, 0, lane0);
        load_regs(w1, src, LREGS, lane0);
        announce();
        // A helper XCD works for kResServed teams, in the order in which their vectors come: it needs 3 us for
        // both layers of a step that takes the chain 7 to 10.
        __amdgpu_buffer_rsrc_t bufs[kResServed];
        unsigned step[2 * kResServed];             // of team i: step number, and the layer that comes next
        unsigned live = 0;
#pragma unroll
        for (int i = 0; i < kResServed; ++i) {
            step[2 * i] = 1; step[2 * i + 1] = 0;
            bufs[i] = buffers_of(serves(i) ? team + i * helper_xcds : team);
            if (serves(i)) { (void)meet(team + i * helper_xcds, false); live |= 1u << i; }
        }
        __syncthreads();
        constexpr int N = (kResRows * (W / 4) + kResThreads - 1) / kResThreads;
        const unsigned inv = piece_inverse(h4);
        // LDS: partial sums of the teams' stages, then the rows of their vectors
        constexpr int XR = kResServed * kResWaves * 1024;
        static_assert(XR + kResServed * kResRows * XROW <= lo.bytes, "the helpers' layout fits");
        unsigned spins = 0, par = 0;
        while (live != 0u && rc.ok) {
            r4u v[kResServed][N];
            const unsigned tid = (unsigned)(x.wave * 64 + lane_id());
            unsigned f = 0;                        // bits 0 ..: team i's vector is complete; bits 8 ..: it says stop
#pragma unroll
            for (int i = 0; i < kResServed; ++i)
                if (live >> i & 1u) {
                    x.buf = bufs[i];
                    const unsigned at = bo.hr[0] + step[2 * i + 1] * (bo.hr[1] - bo.hr[0]) + RES_SLOT(step[2 * i]) * VSLOT;
                    bool missing = false;
#pragma unroll
                    for (int k = 0; k < N; ++k) v[i][k] = get4(x, piece_offset<W>(piece_index(tid, k, p.slots * h4), inv, h4), at);
#pragma unroll
                    for (int k = 0; k < N; ++k) missing = missing || has_mark(v[i][k]);
                    if (__ballot(missing) == 0ull) f |= 1u << i | (__ballot(v[i][0].x == kStop) != 0ull ? 256u << i : 0u);
                }
            if (lane_id() == 0) rc.seen[par][x.wave] = f;
            __syncthreads();
            unsigned all = ~0u, any = 0;
#pragma unroll
            for (int w = 0; w < kResWaves; ++w) { all &= rc.seen[par][w]; any |= rc.seen[par][w]; }
            all = (unsigned)__builtin_amdgcn_readfirstlane((int)all) & live;
            any = (unsigned)__builtin_amdgcn_readfirstlane((int)any);
            par ^= 1u;
            if (all == 0u) {
                if (wait_expired(p, spins)) rc.ok = 0;
                continue;
            }
            spins = 0;
            unsigned todo = all & ~(any >> 8);
            live &= ~(all & (any >> 8));
            // the vectors that are here go to LDS; the second layers' first, which are needed sooner
            unsigned second = 0;
#pragma unroll
            for (int i = 0; i < kResServed; ++i)
                if (todo >> i & 1u) {
                    second |= step[2 * i + 1] << i;
#pragma unroll
                    for (int k = 0; k < N; ++k) {
                        const unsigned idx = piece_index(tid, k, p.slots * h4), r = piece_row(idx, inv);
                        x_put<BF>(lds + XR + (i * kResRows + r) * XROW, (int)(idx - __umul24(r, (unsigned)h4)), v[i][k]);
                    }
                }
            __syncthreads();
            while (todo != 0u) {
                const unsigned t = (unsigned)__builtin_ctz(second & todo ? second & todo : todo);
                todo &= ~(1u << t);
                unsigned n = 0, layer = 0;
#pragma unroll
                for (unsigned i = 0; i < kResServed; ++i)
                    if (t == i) {
                        x.buf = bufs[i];
                        n = step[2 * i]; layer = step[2 * i + 1];
                        step[2 * i] += layer; step[2 * i + 1] = layer ^ 1u;
                    }
                const unsigned char *xr = lds + XR + t * kResRows * XROW;
                float *sums = reinterpret_cast<float *>(lds) + t * kResWaves * 256;
                if (layer == 0) lstm_stage<BF, CLS>(w0, xr, h4, sums, x.wave, lane_id());
                else lstm_stage<BF, CLS>(w1, xr, h4, sums, x.wave, lane_id());
                __syncthreads();
                if (has_cells) {
                    put_far(x, prelane(), bo.pre + (layer * kResSlots + RES_SLOT(n)) * PSLOT, word_of(stage_sum(sums, x.wave, lane_id())));
                    put_far(x, prelane(), bo.pre + (layer * kResSlots + RES_SLOT(n + 2)) * PSLOT, kMark);
                }
            }
        }
        if (!rc.ok && threadIdx.x == 0) __hip_atomic_fetch_or(p.status, 4, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }

    // ---- the chain's work-groups ---------------------------------------------------------------
    RegW<LREGS> w_hh[NREC > 0 ? NREC : 1], w_ih;
    RegW<res_pred_regs(BF, CLS)> w_pr;
    RegW<res_joint_regs(BF, CLS)> w_ou;
    {
        const float *src = p.w + (long long)(x.rank * kResWaves + x.wave) * res_main_regs(KIND, BF, CLS) * 64;
        int first = 0;
#pragma unroll
        for (int l = 0; l < NREC; ++l) { load_regs(w_hh[l], src, first, lane0); first += LREGS; }
        if (NL > 1) { load_regs(w_ih, src, first, lane0); first += LREGS; }
        load_regs(w_pr, src, first, lane0); first += res_pred_regs(BF, CLS);
        load_regs(w_ou, src, first, lane0);
    }
    // utterances of the team: ranked by length (longest first, ties by index), dealt in serpentine
    // order; empty ones are complete from the start
    for (int b = tid0; b < p.B; b += kResThreads) {
        const int raw = p.enc_len[b];
        if (raw < 0 || raw > p.T) rc.st_clamped = 1;
        const int len = min(max(raw, 0), p.T);
        int pos = 0;
        for (int o = 0; o < p.B; ++o) {
            const int l2 = min(max(p.enc_len[o], 0), p.T);
            pos += (l2 > len || (l2 == len && o < b)) ? 1 : 0;
        }
        const int q = pos / n_teams, m = pos - q * n_teams;
        if (((q & 1) ? n_teams - 1 - m : m) == team) {
            rc.list_b[q] = b; rc.list_len[q] = len;
            if (len > 0) atomicAdd(&rc.n_list, 1);       // the empty ones are the last of the list
            else if (x.rank == 0) res_finish_row(b, 0);
        }
    }
    const int u0 = x.rank * p.pl.units, nu = max(0, min(p.pl.units, p.H - u0));
    const int g0 = x.rank * p.pl.jgroups, njg = max(0, min(p.pl.jgroups, (p.J >> 2) - g0));
    const bool has_tail = x.rank < p.pl.n_tail;      // a column of the tail, with column tile 0
    const int tcol = p.pl.nout_m + x.rank;
    const int n_tok = min(p.VT, p.pl.nout_m) - x.rank * 32;      // token columns of this work-group's tiles
    const bool dur_cols = p.tdt && p.VT < p.pl.nout_m && x.rank * 32 + 32 > p.VT;      // they hold duration columns
    if (tid0 < kResUnits * 4) rc.b1[tid0] = (NL > 1 && tid0 < nu * 4) ? p.bias_l[((long long)p.H + u0) * 4 + tid0] : 0.f;
    if (tid0 < 20) rc.bp[tid0] = tid0 < njg * 4 ? p.b_pred[g0 * 4 + tid0] : 0.f;
    if (tid0 < 32) rc.bo[tid0] = x.rank * 32 + tid0 < p.pl.nout_m ? p.b_out[x.rank * 32 + tid0] : 0.f;
    if (tid0 == 0) rc.bt = has_tail ? p.b_out[tcol] : 0.f;
    if (has_tail)
        for (int i = tid0; i < ROW; i += kResThreads) {
            const float w = p.w_tail[(long long)x.rank * ROW + i];
            // (bfloat16 mode: bf16 values, followed by as many zeros)
            if (BF) reinterpret_cast<unsigned short *>(lds + lo.tail)[i] = (unsigned short)(__float_as_uint(w) >> 16);
            else reinterpret_cast<float *>(lds + lo.tail)[i] = w;
        }
    // What a lane finishes in the LSTM stages, see stage_sum: a row of the team, a unit and a gate.  Worked
    // out where it is used: kept for the whole loop, values like these take the registers that the
    // weights need.
    struct Place { int row, j, lu, gu; bool ok; };
    auto place_of = [&](int lane) {
        Place l;
        l.row = (lane >> 2) & 3; l.j = lane & 3;
        l.lu = x.wave * 4 + (lane >> 4);
        l.ok = l.lu < nu && l.j == 0 && l.row < p.slots;      // the lanes that publish it
        l.gu = min(u0 + l.lu, p.H - 1);
        return l;
    };
    // (joint output: a wave takes every eighth step of K for both column tiles)
    // Frames per row and samples of a joint step with NT tiles of samples: p.la, or half of it with one tile instead
    // of two.  (That is read and worked out anew, or it and all that follows from it takes scalar registers in the
    // steps with two.)
    struct Frames {
        int la, ns;
        unsigned inv_la, inv_t;
        __device__ __forceinline__ int row_of(int s) const { return (int)(((unsigned)s * inv_la) >> 10); }      // s / la for s < 32, la <= 16
        __device__ __forceinline__ int mod_la(int t) const { return t - (int)__umulhi((unsigned)t, inv_t) * la; }      // t % la for t < 2^24
    };
    auto frames_of = [&](auto nt_) {
        Frames f;
        if constexpr (HALVES) {
            const Args a = args_again();
            f.la = decltype(nt_)::value < NMT ? a->la >> 1 : a->la;
            f.ns = a->slots * f.la;
        } else {
            f.la = p.la;
            f.ns = p.slots * f.la;
        }
        f.inv_la = (1024u + (unsigned)f.la - 1u) / (unsigned)f.la;
        f.inv_t = 0xffffffffu / (unsigned)f.la + 1u;
        return f;
    };
    constexpr int QS = ROW + 16;                     // floats per q row
    float *lq = reinterpret_cast<float *>(lds + lo.q);
    const unsigned lds_p = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)(lds + lo.p);
    float *part = reinterpret_cast<float *>(lds + lo.part);          // joint sums, see there
    float *tpart = reinterpret_cast<float *>(lds + lo.tpart);        // [wave][tile][16]
    float *g4 = reinterpret_cast<float *>(lds + lo.g4);              // [row group][wave][lane][row]

    announce();
    x.local = meet(team, PAIR);
    bool ok = rc.ok != 0;

    // state of the lane's cell, [layer]: committed and candidate cell value, recurrent pre-activation
    // W_hh h of the committed vector (that of the candidate is in the stage's sums, or comes from the helpers)
    float cs[NL], cc[NL], ps[NL];
#pragma unroll
    for (int l = 0; l < NL; ++l) cs[l] = cc[l] = ps[l] = 0.f;
    float *sums_ih = reinterpret_cast<float *>(lds + lo.ih), *sums_rec = reinterpret_cast<float *>(lds + lo.rec), *sums_rec2 = sums_rec + (NREC - 1) * kResWaves * 256;     // (the top layer's)
    unsigned n_pred = 0, n_joint = 0;

    RRows &rows = rc.rows[x.wave];
    int n_samples = 0, row_steps = 0;
    // What the loop control leaves for the steps: of the row that the lane finishes cells of, the last label
    // (and, in lane_const, what the prediction step does with the candidate state); of sample `lane`, its row
    // of the projected frames, -1 for none.
    int last = p.blank, pidx = -1;
    // What a lane needs of the loop control's tables, packed (a register each would be one too many): the
    // sample's row (2 bits) and place (4), its own row's first sample (5), the word of a row of T0 that
    // its cell takes (12); kTake and kFresh.
    int lane_const = kFresh;
    auto pack_lane = [&](const Frames &f, int lane) {
        const int srow = min(f.row_of(lane & (kResSamples - 1)), kResRows - 1), si = (lane - srow * f.la) & 15;
        const Place l = place_of(lane);
        lane_const = srow | si << 2 | (l.row * f.la) << 6 | (l.gu * 4 + l.j) << 11 | (lane_const & (kTake | kFresh));
    };
    std::integral_constant<int, NMT> all_tiles;
    const Frames f_all = frames_of(all_tiles);
    pack_lane(f_all, lane0);
    // Samples of the next joint step: `la` frames of every row in work, frame f in the row's place f % la,
    // so that a frame stays where it is until the row has passed it.  fresh: the samples to load.
    unsigned long long fresh = 0;
    auto set_up_samples = [&](const Frames &f, int lane, int t, int m, int b, int len) {
        const int la = f.la, ns = f.ns;
        const int from = (lane_const & 3) << 4;                                     // (bytes: four lanes per row)
        const int base = __builtin_amdgcn_ds_bpermute(from, b * p.T + t);
        const int info = __builtin_amdgcn_ds_bpermute(from, max(0, min(len - t, la)) | m << 8);
        int off = ((lane_const >> 2) & 15) - (info >> 8);
        if (off < 0) off += la;
        const int was = pidx;
        pidx = (lane < ns && off < (info & 255)) ? base + off : -1;
        fresh = __ballot(pidx >= 0 && pidx != was);
        n_samples += __popcll(__ballot(pidx >= 0));
    };
    // Rows that want one get the next utterances of the list.  (Control state is by row: every lane works on
    // row lane / 4 % 4, and lanes 0, 4, 8, 12 stand for the rows in ballots.)
    auto refill = [&](int lane, bool want, int &b, int &len) {
        const unsigned long long m = __ballot(want) & 0x1111ull;
        if (m == 0ull) return false;
        const int next = rows.next, at = next + __popcll(m & ((1ull << (lane & 12)) - 1ull));
        const bool got = want && at < rc.n_list;
        if (got) { b = rc.list_b[at]; len = rc.list_len[at]; }
        rows.next = next + __popcll(m);
        return got;
    };
    __syncthreads();                  // the list is complete
    bool any_active, need_pred;
    {
        int b = 0, len = 0;
        const int r = (lane0 >> 2) & 3;
        const bool got = refill(lane0, r < p.slots, b, len);
        if (got) { rows.b[r] = b; rows.s[r].len = len; }
        const unsigned long long m = __ballot(got) & 0x1111ull;
        any_active = need_pred = m != 0ull;
        row_steps = __popcll(m);
        set_up_samples(f_all, lane0, 0, 0, b, len);
    }
    // the row of the embedding table (folded into the first layer) that the next prediction step adds
    float t0 = 0.f;
    const unsigned t0_row = (unsigned)p.H * 16u;
    auto load_t0 = [&]() {
        t0 = 0.f;
        if (has_cells) t0 = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(p.T0) + (__umul24((unsigned)last, t0_row) + ((unsigned)lane_const >> 9 & 0x3ffcu)));
    };
    // kResident2Pair: W_hh h of the last step's candidates as far as it is there, kMark where not
    unsigned pre[2] = {0u, 0u};
    auto load_pre = [&](unsigned n, unsigned (&to)[2]) {
        const unsigned slot = bo.pre + RES_SLOT(n) * PSLOT;
#pragma unroll
        for (int l = 0; l < 2; ++l) to[l] = !has_cells ? 0u : get1(x, prelane(), slot + (unsigned)l * kResSlots * PSLOT);
    };
    if (need_pred) load_t0();
#ifdef RNNT_PROFILE
    if (tid0 == 0) { for (int i = 0; i < 24; ++i) res_prof[i] = 0; res_prof_last = wall_clock64(); }
#endif

    // Steps with NT tiles of samples: until the team is done, or the other number of tiles suits its rows better.
    auto steps = [&](auto nt_) {
    constexpr int NT = decltype(nt_)::value;
    const Frames f = HALVES ? frames_of(nt_) : f_all;
    const int la = f.la, ns = f.ns;
    bool change = false;
    // (Two teams of short steps keep their helpers busy: half the results come after the control's start has
    // asked for them, and one more round trip costs 1.3 us; asked for again at its end, 0.16 us a step less.)
    unsigned later[2] = {kMark, kMark};
    while (ok && any_active && !change) {
        if (!need_pred)
            for (int s = x.wave; s < ns; s += kResWaves)
                if (fresh >> s & 1) load_frame<ROW>(p, x, lds_p, __builtin_amdgcn_readlane(pidx, s), s);
        if (need_pred) {
            // ---- prediction step -----------------------------------------------------------------
            ++n_pred;
            const unsigned n = n_pred;
            if (PAIR && n > 1) {
                unsigned spins = 0;
                if (NT < NMT && __ballot(pre[0] == kMark || pre[1] == kMark) != 0ull) { pre[0] = later[0]; pre[1] = later[1]; }
                while (__ballot(pre[0] == kMark || pre[1] == kMark) != 0ull) {
                    if (wait_expired(p, spins)) { rc.ok = 0; break; }
                    load_pre(n - 1, pre);
                }
                x.polls += __builtin_amdgcn_readfirstlane((int)spins);
            }
            RES_MARK(0);
            // rows that emitted take their candidate state, fresh rows start from zero (kResident2: the second
            // layer's while the first one's vector is on its way)
            auto commit = [&](int l) {
                float pc = 0.f;
                if (PAIR) pc = __uint_as_float(pre[l]);
                else if (has_cells) pc = stage_sum(l == NL - 1 ? sums_rec2 : sums_rec, x.wave, lane_id());
                const bool take = lane_const & kTake, fresh_row = lane_const & kFresh;       // (bits: as a chain of comparisons it became branches)
                cs[l] = take ? cc[l] : cs[l]; cs[l] = fresh_row ? 0.f : cs[l];
                ps[l] = take ? pc : ps[l]; ps[l] = fresh_row ? 0.f : ps[l];
            };
            commit(0);
            if constexpr (PAIR) commit(1);       // (here: its load came before the stores below, and waits end in order)
            // publishes the lane's hidden value of a layer and clears the slot of two steps ago
            auto publish_h = [&](int layer, const Place &l, float h) {
                if (l.ok) {
                    const unsigned o = (unsigned)l.row * VROW + (unsigned)l.gu * 4u;
                    const unsigned s1 = RES_SLOT(n) * VSLOT, s2 = RES_SLOT(n + 2) * VSLOT;
                    put(x, o, bo.h[layer] + s1, bo.h[layer] + s2, word_of(h));
                    if (PAIR) { put_far(x, o, bo.hr[layer] + s1, word_of(h)); put_far(x, o, bo.hr[layer] + s2, kMark); }
                }
            };
            if (has_cells) {
                const Place l = place_of(lane_id());
                float h;
                cell(ps[0] + t0, l.j, cs[0], cc[0], h);
                publish_h(0, l, h);
            }
            if constexpr (NREC > 1) commit(1);
            // The frames of the joint step, by the waves that have the least to do here.  A wave's loads return in
            // order, so these waves see the hidden vector when their frames are there: at about the time it comes.
            if (x.wave >= 5)
                for (int s = x.wave - 5; s < ns; s += kResWaves - 5)
                    if (fresh >> s & 1) load_frame<ROW>(p, x, lds_p, __builtin_amdgcn_readlane(pidx, s), s);
            RES_MARK(1);
            unsigned char *x0 = lds + lo.xh, *x1 = lds + lo.xh + (NL - 1) * kResRows * XROW;
            receive_rows<W>(p, x, bo.h[0] + RES_SLOT(n) * VSLOT, p.slots, h4, [&](int r, int k4, r4u v) { x_put<BF>(x0 + r * XROW, k4, v); });
            __syncthreads();
            RES_MARK(2);
            if constexpr (NL > 1) {
                lstm_stage<BF, CLS>(w_ih, x0, h4, sums_ih, x.wave, lane_id());
                __syncthreads();
                RES_MARK(3);
                if (has_cells) {
                    const int lane = lane_id();
                    const Place l = place_of(lane);
                    float h;
                    cell(stage_sum(sums_ih, x.wave, lane) + (ps[1] + rc.b1[l.lu * 4 + l.j]), l.j, cs[1], cc[1], h);
                    publish_h(1, l, h);
                }
                RES_MARK(4);
                // (while the hand-over is on its way) the recurrent part of the next step's first layer
                if constexpr (NREC > 1) lstm_stage<BF, CLS>(w_hh[0], x0, h4, sums_rec, x.wave, lane_id());
                RES_MARK(5);
                receive_rows<W>(p, x, bo.h[1] + RES_SLOT(n) * VSLOT, p.slots, h4, [&](int r, int k4, r4u v) { x_put<BF>(x1 + r * XROW, k4, v); });
                __syncthreads();
            }
            RES_MARK(6);
            // prediction-side joint projection: a wave's blocks are five groups of four columns times three slices of K;
            // partial sums through LDS
            {
                constexpr int NP = res_pred_pieces(CLS);
                {
                    const int lane = lane_id(), sl = ((lane >> 2) * 13) >> 6;        // block / 5
                    const unsigned char *xl = x1 + (lane & 3) * XROW;
                    Pc v[NP];
#pragma unroll
                    for (int i = 0; i < NP; ++i) v[i].load(xl + min(i * 24 + x.wave * 3 + sl, h4 - 1) * Pc::B);
                    r4f a[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                    for (int i = 0; i < NP; ++i)
#pragma unroll
                        for (int e = 0; e < Pc::N; ++e) v[i].mfma(e, &w_pr.w[i * PR], a[(i * Pc::N + e) & 1]);
                    if (lane < 60) *reinterpret_cast<r4f *>(g4 + (x.wave * 60 + lane) * 4) = a[0] + a[1];
                }
                __syncthreads();
                // four adjacent threads per value (group, column, row), two waves' sums each
                const int tid = (x.wave * 64 + lane_id()), g = tid >> 6, j = (tid >> 4) & 3, r = (tid >> 2) & 3;
                if (g < njg) {
                    const float *v = g4 + ((tid & 3) * 120 + g * 4 + j) * 4 + r;
                    const float bias = rc.bp[g * 4 + j];
                    const float s = lane_sum<4>(((v[0] + v[80]) + v[160]) + ((v[240] + v[320]) + v[400]));
                    if ((tid & 3) == 0 && r < p.slots)
                        put(x, (unsigned)r * VROW + (unsigned)((g0 + g) * 4 + j) * 4u, bo.q + RES_SLOT(n) * VSLOT, bo.q + RES_SLOT(n + 2) * VSLOT, word_of(s + bias));
                }
            }
            RES_MARK(7);
            // (while q is on its way) the recurrent part of the top layer's next step
            if constexpr (NREC > 0) lstm_stage<BF, CLS>(w_hh[NREC - 1], x1, h4, sums_rec2, x.wave, lane_id());
            RES_MARK(8);
            receive_rows<W>(p, x, bo.q + RES_SLOT(n) * VSLOT, p.slots, p.J >> 2, [&](int r, int k4, r4u v) {
                *reinterpret_cast<r4u *>(lq + r * QS + k4 * 4) = v;
            });
            RES_MARK(9);
        }
        // ---- joint step ----------------------------------------------------------------------------
        ++n_joint;
        const unsigned jn = n_joint;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the frames of this wave's samples are in LDS
        __syncthreads();
        RES_MARK(10);
        {
            r4f acc[NT][2];                 // [tile of samples][column tile]
            const int lane = lane_id(), m16 = lane & 15, kq = lane >> 4;
            // Piece k4 = 32 ii + 4 wave + kq of sample m16: its low bits are the same for all steps.  The operand
            // relu(P + q) is formed on the way: K is split over the waves, so nobody else needs it.  The
            // vector instructions of a step come in one run before its matrix instructions: the fp32 ones share
            // the vector pipe with them, and every change between the two costs some ten cycles.
            const int k40 = x.wave * 4 + kq;
            const unsigned char *pr = lds + lo.p + m16 * ROW * 4 + ((k40 & 16) | ((k40 ^ m16) & 15)) * 16;
            const float *q[NT];
#pragma unroll
            for (int mt = 0; mt < NT; ++mt) {
                acc[mt][0] = acc[mt][1] = (r4f){0.f, 0.f, 0.f, 0.f};
                q[mt] = lq + min(f.row_of(mt * 16 + m16), kResRows - 1) * QS + k40 * 4;
            }
            auto fetch = [&](int ii, int mt, float4 &pv, float4 &qv) {
                pv = *reinterpret_cast<const float4 *>(pr + mt * 16 * ROW * 4 + ii * 512);
                qv = *reinterpret_cast<const float4 *>(q[mt] + ii * 128);
            };
            if constexpr (BF) {
                float4 pv, qv;
                fetch(0, 0, pv, qv);
                struct Q { float a, b; };
                struct U { unsigned a, b; };
                // the tail column as an operand of its own: its row mt is the weights for tile mt, the others are zeros
                const unsigned char *wt = lds + lo.tail + k40 * 8;
                r4f tacc = (r4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < NI * NT; ++i) {
                    const int ii = i / NT, mt = i % NT;
                    const r4s z = __builtin_bit_cast(r4s, U{bf16_pair(fmaxf(pv.x + qv.x, 0.f), fmaxf(pv.y + qv.y, 0.f)),
                                                            bf16_pair(fmaxf(pv.z + qv.z, 0.f), fmaxf(pv.w + qv.w, 0.f))});
                    if (i + 1 < NI * NT) fetch((i + 1) / NT, (i + 1) % NT, pv, qv);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const float *w = &w_ou.w[(ii * 2 + c) * PR];
                        acc[mt][c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(r4s, Q{w[0], w[1]}), z, acc[mt][c], 0, 0, 0);
                    }
                    if (has_tail) tacc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const r4s *>(wt + (m16 == mt ? 0 : ROW * 2) + ii * 256), z, tacc, 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (has_tail) {
#pragma unroll
                    for (int mt = 0; mt < NT; ++mt)
                        if (kq == 0) tpart[(x.wave * 2 + mt) * 16 + m16] = tacc[mt];
                }
            } else {
                const float *wt = reinterpret_cast<const float *>(lds + lo.tail) + k40 * 4;
                float tl[NT];
#pragma unroll
                for (int mt = 0; mt < NT; ++mt) tl[mt] = 0.f;
                float4 wv = *reinterpret_cast<const float4 *>(wt), pv[NT], qv[NT];
#pragma unroll
                for (int mt = 0; mt < NT; ++mt) fetch(0, mt, pv[mt], qv[mt]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int ii = 0; ii < NI; ++ii) {
                    float z[NT][4];
#pragma unroll
                    for (int mt = 0; mt < NT; ++mt) {
                        z[mt][0] = fmaxf(pv[mt].x + qv[mt].x, 0.f); z[mt][1] = fmaxf(pv[mt].y + qv[mt].y, 0.f);
                        z[mt][2] = fmaxf(pv[mt].z + qv[mt].z, 0.f); z[mt][3] = fmaxf(pv[mt].w + qv[mt].w, 0.f);
                        tl[mt] = fmaf(z[mt][3], wv.w, fmaf(z[mt][2], wv.z, fmaf(z[mt][1], wv.y, fmaf(z[mt][0], wv.x, tl[mt]))));
                        // (the sums are opaque here: otherwise they move behind the loop, under the condition they are used
                        // under, with every z kept in a register till then)
                        asm volatile("" : "+v"(tl[mt]));
                    }
                    if (ii + 1 < NI) {
#pragma unroll
                        for (int mt = 0; mt < NT; ++mt) fetch(ii + 1, mt, pv[mt], qv[mt]);
                        wv = *reinterpret_cast<const float4 *>(wt + (ii + 1) * 128);
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int mt = 0; mt < NT; ++mt)
#pragma unroll
                            for (int c = 0; c < 2; ++c)
                                acc[mt][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(w_ou.w[(ii * 2 + c) * 4 + e], z[mt][e], acc[mt][c], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (has_tail) {
#pragma unroll
                    for (int mt = 0; mt < NT; ++mt) {
                        float a = tl[mt], b = tl[mt];
                        swap32(a, b); a += b; b = a;
                        swap16(a, b); a += b;
                        if (lane < 16) tpart[(x.wave * 2 + mt) * 16 + lane] = a;
                    }
                }
            }
            RES_MARK(11);
            // every wave's sums to LDS, [wave][sample][column]; then sixteen lanes per sample, two columns each
#pragma unroll
            for (int mt = 0; mt < NT; ++mt)
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    *reinterpret_cast<r4f *>(part + ((x.wave * NT + mt) * 16 + m16) * kResSumRow + c * 16 + kq * 4) = acc[mt][c];
            __syncthreads();
            const int tid = (x.wave * 64 + lane_id());
            if (tid < 16 * NT * 16) {
                const int s = tid >> 4, col = (tid & 15) * 2, gcol = x.rank * 32 + col;
                float2 o[kResWaves];
#pragma unroll
                for (int w = 0; w < kResWaves; ++w)
                    o[w] = *reinterpret_cast<const float2 *>(part + (w * NT * 16 + s) * kResSumRow + col);
                const float2 bias = *reinterpret_cast<const float2 *>(&rc.bo[col]);
                static_assert(kResWaves == 8, "eight lanes add the waves' sums of the tail column");
                float tw = 0.f;
                if (has_tail) tw = tpart[((tid & 7) * 2 + (s >> 4)) * 16 + (s & 15)];
                const float l0 = (((o[0].x + o[1].x) + (o[2].x + o[3].x)) + ((o[4].x + o[5].x) + (o[6].x + o[7].x))) + bias.x;
                const float l1 = (((o[0].y + o[1].y) + (o[2].y + o[3].y)) + ((o[4].y + o[5].y) + (o[6].y + o[7].y))) + bias.y;
                const float m0 = col < n_tok ? l0 : -INFINITY, m1 = col + 1 < n_tok ? l1 : -INFINITY;
                const float mine = fmaxf(m0, m1);
                float m = lane_max<16>(mine);
                // the first lane of the sixteen that holds the maximum publishes (without a token column: lane 0)
                const unsigned hit = (unsigned)(__ballot(mine == m && col < n_tok) >> (tid & 48)) & 0xffffu;
                const int first = hit ? __builtin_ctz(hit) : 0;
                int ix = hit ? (m0 == m ? gcol : gcol + 1) : 0x7fffffff;
                float tail = -INFINITY;
                if (has_tail) {
                    tail = lane_sum<8>(tw) + rc.bt;
                    if (tcol >= p.VT) {
                        if ((tid & 15) == 0 && s < ns) {
                            const unsigned d = ((unsigned)s * kMaxDur + (unsigned)(tcol - p.VT)) * 4u;
                            put(x, d, bo.dur + RES_SLOT(jn) * DSLOT, bo.dur + RES_SLOT(jn + 2) * DSLOT, word_of(tail));
                        }
                        tail = -INFINITY;
                    } else if (tail > m) {
                        m = tail; ix = tcol;
                    }
                }
                if (dur_cols && s < ns) {
                    // duration columns inside the column tiles
#pragma unroll
                    for (int c = 0; c < 2; ++c)
                        if (gcol + c >= p.VT && gcol + c < p.pl.nout_m) {
                            const unsigned d = ((unsigned)s * kMaxDur + (unsigned)(gcol + c - p.VT)) * 4u;
                            put(x, d, bo.dur + RES_SLOT(jn) * DSLOT, bo.dur + RES_SLOT(jn + 2) * DSLOT, word_of(c ? l1 : l0));
                        }
                }
                const unsigned ko = ((unsigned)s * TS + (unsigned)x.rank) * 8u;
                if ((tid & 15) == first && s < ns)
                    put2(x, ko, bo.key + RES_SLOT(jn) * KSLOT, bo.key + RES_SLOT(jn + 2) * KSLOT, (r2u){word_of(m), (unsigned)ix});
                if (p.logps) {
                    float e = (m0 > -INFINITY ? expf(m0 - m) : 0.f) + (m1 > -INFINITY ? expf(m1 - m) : 0.f);
                    e = lane_sum<16>(e);
                    if (tail > -INFINITY) e += expf(tail - m);
                    if ((tid & 15) == 0 && s < ns)
                        put(x, ko / 2, bo.lse + RES_SLOT(jn) * (KSLOT / 2), bo.lse + RES_SLOT(jn + 2) * (KSLOT / 2), word_of(e));
                }
            }
        }
        if constexpr (NT < NMT) {
            // the samples that this step does not have: the marks that their words of step jn + 2 need
            const int tid = x.wave * 64 + lane_id(), s = tid >> 4;
            if (s >= ns && s < ns * 2) {
                const int gcol = x.rank * 32 + (tid & 15) * 2;
                const unsigned ko = ((unsigned)s * TS + (unsigned)x.rank) * 8u, ds = (unsigned)s * kMaxDur * 4u;
                const bool lead = (tid & 15) == 0;
                if (lead) put_mark2(x, ko, bo.key + RES_SLOT(jn + 2) * KSLOT);
                if (lead && p.logps) put_mark(x, ko / 2, bo.lse + RES_SLOT(jn + 2) * (KSLOT / 2));
                if (lead && has_tail && tcol >= p.VT) put_mark(x, ds + (unsigned)(tcol - p.VT) * 4u, bo.dur + RES_SLOT(jn + 2) * DSLOT);
                if (dur_cols) {
#pragma unroll
                    for (int c = 0; c < 2; ++c)
                        if (gcol + c >= p.VT && gcol + c < p.pl.nout_m)
                            put_mark(x, ds + (unsigned)(gcol + c - p.VT) * 4u, bo.dur + RES_SLOT(jn + 2) * DSLOT);
                }
            }
        }
        RES_MARK(12);
        // ---- argmax over the team: TS / 2 adjacent lanes per sample, two candidates per lane --------
        {
            const int tid = (x.wave * 64 + lane_id()), lane = tid & 63;
            constexpr int L = TS / 2;
            static_assert(16 * NT * L <= kResThreads, "one piece per thread");
            const int s = tid / L;
            if ((x.wave * 64) / L < ns) {
                const unsigned off[1] = {(unsigned)min(tid, ns * L - 1) * 16u};
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
                        v[0] = get4(x, off[0], bo.key + RES_SLOT(jn) * KSLOT);
                        bool missing = false;
#pragma unroll
                        for (int i = 0; i < ND; ++i) dv[i] = get1(x, o + i * 4u, bo.dur + RES_SLOT(jn) * DSLOT);
#pragma unroll
                        for (int i = 0; i < ND; ++i) missing = missing || (di + i < p.D && dv[i] == kMark);
                        if (__ballot(missing || has_mark(v[0])) == 0ull) break;
                        if (wait_expired(p, spins)) { rc.ok = 0; break; }
                    }
                    x.polls += __builtin_amdgcn_readfirstlane((int)spins);
                    // best duration, the lowest index on ties
                    const float d0 = di < p.D ? __uint_as_float(dv[0]) : -INFINITY, d1 = ND > 1 && di + 1 < p.D ? __uint_as_float(dv[ND - 1]) : -INFINITY;
                    const float dl = fmaxf(d0, d1), dm = lane_max<L>(dl);
                    const unsigned hit = (unsigned)(__ballot(dl == dm && di < p.D) >> (lane & ~(L - 1))) & ((1u << L) - 1u);
                    if (li == (hit ? __builtin_ctz(hit) : 0) && s < ns) rc.s_d[s] = d0 == dm || ND == 1 ? v0 : v1;
                } else {
                    receive<1>(p, x, off, bo.key + RES_SLOT(jn) * KSLOT, v);
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
                        e0 = get1(x, off[0] >> 1, bo.lse + RES_SLOT(jn) * (KSLOT / 2));
                        e1 = get1(x, (off[0] >> 1) + 4u, bo.lse + RES_SLOT(jn) * (KSLOT / 2));
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
                if (win && s < ns) {
                    rc.s_k[s] = (unsigned)bi < (unsigned)p.VT ? bi : p.blank;
                    rc.s_v[s] = m + 0.0f;
                    if (p.logps) rc.s_lp[s] = lp2;
                }
            }
            RES_MARK(13);
        }
        // ---- loop control: every wave for itself, lane = row (outputs: the last wave, which has the least to do next) ------
        {
            const int lane = lane_id(), r = (lane >> 2) & 3;
            RRow w = rows.s[r];
            int b = rows.b[r], m = rows.m[r];
            __syncthreads();
            RES_MARK(14);
            if (PAIR) load_pre(n_pred, pre);       // (on its way during the rest)
            const int mine = rc.s_k[lane & (kResSamples - 1)], row0 = (lane_const >> 6) & 31, left = w.len - w.t;
            const bool lead = lane < 16 && (lane & 3) == 0;     // stands for its row
            const bool writer = x.rank == 0 && x.wave == kResWaves - 1 && lead;
            const bool walk = p.tdt || p.VT != p.V1;
            int pos, dval = 0;
            bool found;
            if (!walk) {
                // a blank moves on by one frame: the first label among the frames the row still has
                const unsigned labels = (unsigned)__ballot(mine != p.blank);
                const unsigned at = (labels >> row0) & ((1u << la) - 1u), avail = (unsigned)max(0, min(la, left));     // by place
                pos = __builtin_ctz(((at >> m) | (at << (la - m))) | (1u << avail));                                  // by frame
                found = pos < (int)avail;
            } else {
                // lane = sample: the offset (from the row's frame) that the walk goes to from it, its own for a label
                // or beyond the row's frames, and the lane of that offset, its own where the walk leaves the step;
                // then the hops are doubled until every one reaches its end
                const int sr = lane_const & 3, ms = from_lane(m, sr * 4);
                int to = ((lane_const >> 2) & 15) - ms;
                if (to < 0) to += la;
                int d = 0;
                if (mine >= p.V1) d = max(rc.dur[(mine - p.V1) & (kMaxDur - 1)], 1);            // big blank: its span of frames
                else if (mine == p.blank) d = p.tdt ? max(rc.s_d[lane & (kResSamples - 1)], 1) : 1;
                if (pidx < 0) d = 0;
                to += d;
                int at = ms + to;
                if (at >= la) at -= la;
                int hop = (d > 0 && to < la ? (int)__umul24((unsigned)sr, (unsigned)la) + at : lane) << 2;
                for (int i = 1; i < la; i *= 2) hop = __builtin_amdgcn_ds_bpermute(hop, hop);
                hop = __builtin_amdgcn_ds_bpermute((row0 + m) << 2, hop);
                pos = __builtin_amdgcn_ds_bpermute(hop, to);
                found = pos < la && pos < left;
            }
            int at = m + pos;
            if (at >= la) at -= la;
            const int s = max(0, min(row0 + at, kResSamples - 1));
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
                if (p.tdt && dval > 0) { adv += dval; w.n = 0; }
                else if (++w.n == p.S) { ++adv; w.n = 0; }
            }
            w.t += adv;
            const bool ended = left > 0 && adv >= left;
            int action = found && !ended ? kTake : 0;
            if (walk) {
                m = f.mod_la(w.t);
            } else {
                m += adv;                               // (at most la + 1)
                if (m >= la) m -= la;
                if (m >= la) m -= la;
            }
            if (__ballot(ended) != 0ull) {
                if (writer && ended) res_finish_row(b, w.cnt);
                const bool got = refill(lane, ended, b, w.len);
                if (got) { w.t = w.n = w.cnt = m = 0; action = kFresh; last = p.blank; }
                if (lead) rows.b[r] = b;
                load_t0();
            }
            lane_const = (lane_const & ~(kTake | kFresh)) | action;
            if (lead) { rows.s[r] = w; rows.m[r] = m; }

            const unsigned long long moved = __ballot(action != 0) & 0x1111ull;      // rows whose next step has new inputs
            any_active = __ballot(w.t < w.len) != 0ull;
            need_pred = moved != 0ull;
            row_steps += __popcll(moved);
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
            if (!change) set_up_samples(f, lane, w.t, m, b, w.len);
            if (PAIR && NT < NMT) load_pre(n_pred, later);
        }
        ok = rc.ok != 0;
        RES_MARK(15);
    }
    };
    if constexpr (!HALVES) {
        steps(all_tiles);
    } else {
        // Where the rows go on by less than one and a half frames a step (ten labels on every frame, say), the second
        // tile of samples is computed for nothing: then the team goes on with half the frames per row, until
        // a row's next label is not among them.  128 utterances of ten labels on every frame: 9.7 us a step with two
        // tiles, 8.8 with one (136.4 and 123.6 ms a call; the streaming kernel: 125.8), and with ten labels on every
        // other frame 68.5 and 61.7 ms (62.7).  At 0.7 labels a frame the two are even; below, a team hardly ever
        // gets here, and what looking out for it costs is within 0.6 % of a call.
        // Two-layer fp32 models only: the others were faster than the streaming kernel on such input as well, and
        // their second loop costs more registers than there are (bfloat16 mode: twelve spilled, 4 to 6 % of a call).
        std::integral_constant<int, 1> one_tile;
        auto changed_to = [&](auto nt_) {
            const int lane = lane_id(), r = (lane >> 2) & 3;
            const RRow w = rows.s[r];
            const Frames f = frames_of(nt_);
            const int m = f.mod_la(w.t);
            pack_lane(f, lane);
            if (lane < 16 && (lane & 3) == 0) {
                rows.m[r] = m;
                rows.since[r] = -0x10000000;      // (not after less than kResCalm steps)
            }
            pidx = -1;                // every frame has another place
            set_up_samples(f, lane, w.t, m, rows.b[r], w.len);
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
        // the helpers wait for the next candidate vector: tell them that there is none
        const unsigned o = bo.hr[0] + RES_SLOT(n_pred + 1) * VSLOT;
        for (int i = threadIdx.x; i < p.slots * nu; i += kResThreads) {
            const int r = i / nu, u = i - r * nu;
            put_far(x, (unsigned)r * VROW + (unsigned)(u0 + u) * 4u, o, kStop);
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

template <int KIND, bool BF, int CLS, int NMT>
hipError_t launch_resident_one(const ResidentParams &p, bool plain, hipStream_t stream)
{
    const void *fn = reinterpret_cast<const void *>(&resident_kernel<KIND, BF, CLS, NMT>);
    constexpr unsigned lds = (unsigned)resident_lds(KIND, BF, CLS, NMT).bytes;
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ResidentParams pc = p;
    void *args[] = {&pc};
    const dim3 grid(p.pl.n_xcd * 32), block(kResThreads);
    if (plain) return hipLaunchKernel(fn, grid, block, args, lds, stream);
    return hipLaunchCooperativeKernel(fn, grid, block, args, lds, stream);
}

}  // namespace
}  // namespace rnnt
