// Decode kernel with register-resident weights (device code, instantiated by resident_inst.hip).
//
// The step chain of a decode (a prediction step, a joint step, and again) is bound by latency:
// three dense stages and four hand-overs between work-groups per label.  Two things make it
// short here.  (1) Every weight of the step is held in the registers of one compute unit for the
// whole launch: four waves of 512 registers keep up to 368 weight registers per lane, 92 K fp32
// values per compute unit, so a stage reads nothing but its input vector.  (2) A team of
// work-groups sits inside one XCD, so its hand-overs go through that XCD's L2: a store that stays
// in the L2 and a load that passes by the L1 hand 640 floats to 32 work-groups in 0.97 us, where
// stores and loads through the memory side take 1.76 us (4 x 640 floats: 1.2 against 1.95 us).
//
// Work split inside a team of `ts` work-groups: LSTM units, projection columns and output columns
// in contiguous ranges.  LSTM stages run on v_mfma 4x4 (16 blocks): a wave owns five units (the
// four gates of a unit are a block's four columns) and its 16 blocks are 16 slices of K, so the
// sums of a unit meet inside one wave (permlane swaps and DPP adds) and the pointwise part follows
// without a barrier.  The joint output runs on v_mfma 16x16 (16 samples x 16 columns, two column
// tiles x two halves of K over the four waves); its operand relu(P + q) is formed on the way from
// LDS to the matrix instruction.
//
// Two-layer fp32 models have more weights than one XCD's registers hold (24 MB against 12 + 4):
// there a team owns two XCDs.  The work-groups of the first run the whole step chain and keep the
// input, projection and output matrices; those of the second keep the recurrent matrices and
// compute W_hh h of the candidate state, which the chain needs only at the next label: their
// hand-overs across the XCDs (1.8 us each way) run beside the rest of the step.
//
// Utterances are decoded label-looping fashion: every utterance has its own frame index, a joint
// step examines `la` frames of every utterance, and the next prediction step runs as soon as one
// of them has a label.  A team takes a list of utterances and decodes up to kResRows at a time;
// when one ends the next of the list takes its place.
//
// Exchange: a vector's buffer has four slots used in turn; words are 32-bit floats, all ones
// meaning "not there yet" (readers poll the data itself).  A work-group puts that mark back into
// slot n - 2 when it publishes step n: by then it has received something of step n - 1 from
// everyone, which everyone sent after reading step n - 2; and it waits for that store before it
// publishes step n + 1, so nobody can look for step n + 2's data in a slot that still holds old data.
#pragma once
#include "engine.h"
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
struct RRows { int b[kResRows], len[kResRows], t[kResRows], n[kResRows], cnt[kResRows], active[kResRows]; };

struct RCtl {
    RRows rows[kResWaves];
    int s_k[kResSamples], s_d[kResSamples];        // results of a joint step
    float s_v[kResSamples], s_lp[kResSamples];
    int n_list, ok, st_clamped, st_overflow;
    int list_b[kResList], list_len[kResList];
    // this work-group's slices of the biases: second layer [unit][gate], projection, output and tail column
    float b1[kResUnits * 4], bp[20], bo[32], bt;
};
__shared__ RCtl rc;

// Phase timers (100 MHz wall clock), compiled in only for profiling builds.
#ifdef RNNT_PROFILE
__shared__ long long res_prof[24];
__shared__ long long res_prof_last;
#define RES_MARK(slot) do { __builtin_amdgcn_sched_barrier(0); if (x.tid == 0) { long long t_ = wall_clock64(); res_prof[slot] += t_ - res_prof_last; res_prof_last = t_; } __builtin_amdgcn_sched_barrier(0); } while (0)
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

struct RCtx {
    int tid, lane, wave, rank;
    bool local;                       // every work-group of the team sits on the same XCD
    __amdgpu_buffer_rsrc_t buf;       // the team's exchange buffers
    int polls;
};

// stores that stay in the XCD's L2 / that go through to the memory side (sc1)
__device__ __forceinline__ void put(const RCtx &x, unsigned off, unsigned imm, unsigned v)
{
    if (x.local) __builtin_amdgcn_raw_buffer_store_b32(v, x.buf, (int)off, (int)imm, 0);
    else __builtin_amdgcn_raw_buffer_store_b32(v, x.buf, (int)off, (int)imm, 16);
}
__device__ __forceinline__ void put2(const RCtx &x, unsigned off, unsigned imm, r2u v)
{
    if (x.local) __builtin_amdgcn_raw_buffer_store_b64(v, x.buf, (int)off, (int)imm, 0);
    else __builtin_amdgcn_raw_buffer_store_b64(v, x.buf, (int)off, (int)imm, 16);
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

__device__ __forceinline__ int again(int v) { asm volatile("" : "+v"(v)); return v; }

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
    x.polls += spins;
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
    __device__ __forceinline__ void mfma(int e, const float *w, r4f &acc) const
    {
        acc = __builtin_amdgcn_mfma_f32_4x4x1f32(e == 0 ? v.x : (e == 1 ? v.y : (e == 2 ? v.z : v.w)), w[e], acc, 0, 0, 0);
    }
};
template <> struct Piece<true> {
    static constexpr int N = 1, B = 8;
    r4s v;
    __device__ __forceinline__ void load(const unsigned char *p) { v = *reinterpret_cast<const r4s *>(p); }
    __device__ __forceinline__ void mfma(int, const float *w, r4f &acc) const
    {
        struct P { float a, b; };
        acc = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(v, __builtin_bit_cast(r4s, P{w[0], w[1]}), acc, 0, 0, 0);
    }
};

template <int CTRL>
__device__ __forceinline__ float dppf(float v)
{
    const int i = (int)__float_as_uint(v);
    return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(i, i, CTRL, 0xf, 0xf, false));
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

// Sum of a group's partial sums over the wave's 16 blocks: lane l gets the one of row l / 16,
// column l % 4 (the same in the four blocks of a 16-lane row).
__device__ __forceinline__ float sum_blocks(r4f v)
{
    float a = v[0], b = v[1], c = v[2], d = v[3];
    swap32(a, c); a += c;             // rows 0 and 2
    swap32(b, d); b += d;             // rows 1 and 3
    swap16(a, b); a += b;             // rows 0, 1, 2, 3 by 16-lane row
    a += dppf<0x124>(a);              // row_ror 4
    a += dppf<0x128>(a);              // row_ror 8
    return a;
}

// One LSTM stage over the wave's part of K: partial sums of the work-group's units for all rows go to
// LDS, [row group][wave][lane] with a lane's four rows.  x: the lane's first piece of row lane % 4 (waves
// 0 .. 5: the same for all blocks, so a read is a broadcast), `step` bytes from piece to piece.  No
// sums across lanes: the readers of the partial sums add six or eight of them (stage_sum).
template <bool BF, int CLS, int RG>
__device__ __forceinline__ void lstm_stage(const RegW<res_lstm_regs(BF, CLS)> &w, const unsigned char *x, int step, float *sums, int wave, int lane)
{
    constexpr int N = res_lstm_pieces(CLS), PR = res_piece_regs(BF), XR = 4 * res_xrow(BF, CLS);
    typedef Piece<BF> Pc;
    constexpr int C = RG == 1 ? 2 : 1;  // chains of sums per row group
    r4f acc[RG][C];
#pragma unroll
    for (int rg = 0; rg < RG; ++rg)
#pragma unroll
        for (int i = 0; i < C; ++i) acc[rg][i] = (r4f){0.f, 0.f, 0.f, 0.f};
    constexpr int D = BF ? 3 : (RG == 1 ? 2 : 1);         // pieces on their way ahead of the matrix instructions
    constexpr int N8 = res_pieces(CLS) / 8;               // pieces of a block of waves 6 and 7
    Pc q[D][RG];
#pragma unroll
    for (int i = 0; i < D && i < N8; ++i)
#pragma unroll
        for (int rg = 0; rg < RG; ++rg) q[i][rg].load(x + i * step + rg * XR);
    auto run = [&](int i, bool more) {
        Pc v[RG];
#pragma unroll
        for (int rg = 0; rg < RG; ++rg) {
            v[rg] = q[i % D][rg];
            if (more) q[i % D][rg].load(x + (i + D) * step + rg * XR);
        }
#pragma unroll
        for (int e = 0; e < Pc::N; ++e)
#pragma unroll
            for (int rg = 0; rg < RG; ++rg) v[rg].mfma(e, &w.w[i * PR], acc[rg][(i * Pc::N + e) % C]);
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int i = 0; i < N8; ++i) run(i, i + D < N8);
    if (wave < 6) {                     // (uniform; a read beyond a block's pieces would leave the row)
#pragma unroll
        for (int i = N8; i < N8 + D && i < N; ++i)
#pragma unroll
            for (int rg = 0; rg < RG; ++rg) q[i % D][rg].load(x + i * step + rg * XR);
#pragma unroll
        for (int i = N8; i < N; ++i) run(i, i + D < N);
    }
#pragma unroll
    for (int rg = 0; rg < RG; ++rg)
        *reinterpret_cast<r4f *>(sums + ((rg * kResWaves + wave) * 64 + lane) * 4) = C == 1 ? acc[rg][0] : acc[rg][0] + acc[rg][C - 1];
}

// The stage's sum for lane `lane` of block `blk` of sixteen (unit, row) pairs: row group blk / 5, unit
// 4 (blk % 5) + lane / 16, row lane / 4 % 4, gate lane % 4.
__device__ __forceinline__ float stage_sum(const float *sums, int blk, int lane)
{
    const int rg = blk >= 5 ? 1 : 0, ub = blk - 5 * rg, uu = lane >> 4, row = (lane >> 2) & 3, j = lane & 3;
    const float *s = sums + rg * kResWaves * 256 + row;
    if (ub < 4) {
        s += (4 * (ub * 4 + uu) + j) * 4;
        return ((s[0] + s[256]) + (s[512] + s[768])) + (s[1024] + s[1280]);
    }
    s += 6 * 256 + (4 * uu + j) * 4;         // slices 64 floats apart
    return ((s[0] + s[64]) + (s[128] + s[192])) + ((s[256] + s[320]) + (s[384] + s[448]));
}

// sigmoid(x), or tanh(x) where th: both are N / (1 + e) with e = exp(-x) or exp(-2x); tanh below
// 0.55, where 1 - e would cancel, is Lambert's continued fraction to x^5 / x^4.  The exponential is
// the hardware's exp2 with the rounding of x log2(e) carried along, the quotient the hardware's
// reciprocal with two Newton steps; at most 3 units in the last place over the whole range.
__device__ __forceinline__ float gate_act(float x, bool th)
{
    const float y = fminf(fmaxf(th ? x + x : x, -80.f), 80.f);
    const float kL = 1.44269504f, kLo = 1.92596303e-8f;          // log2(e)
    const float t = -y * kL;
    const float lo = fmaf(-y, kL, -t) - y * kLo;
    float e = __builtin_amdgcn_exp2f(t);
    e = fmaf(e, lo * 0.693147182f, e);
    const float q = x * x;
    const bool small = th && fabsf(x) < 0.55f;
    float n = th ? 1.f - e : 1.f, d = 1.f + e;
    n = small ? x * fmaf(q, 105.f + q, 945.f) : n;
    d = small ? fmaf(q, fmaf(q, 15.f, 420.f), 945.f) : d;
    float r = __builtin_amdgcn_rcpf(d);
    r = fmaf(fmaf(-d, r, 1.f), r, r);
    const float v = n * r;
    return fmaf(fmaf(-d, v, n), r, v);
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

#define RES_SLOT(n) ((unsigned)(n) & (kResSlots - 1))

// Receives a vector of `rows` rows of n4 16-byte pieces each (rows row_bytes apart from byte `base`
// of the exchange buffers on) and hands every piece to f(row, k4, words).
template <int RG, int WIDTH, class F>
__device__ __forceinline__ void receive_rows(const ResidentParams &p, RCtx &x, unsigned base, int rows, int n4, F f)
{
    constexpr int N = (4 * RG * (WIDTH / 4) + kResThreads - 1) / kResThreads;
    unsigned off[N];
    r4u v[N];
    const unsigned tid = (unsigned)again(x.tid), last = (unsigned)(rows * n4 - 1);
    const unsigned inv = ((1u << 20) + (unsigned)n4 - 1u) / (unsigned)n4;   // idx / n4 for idx * n4 < 2^20, idx < 2^11
#pragma unroll
    for (int i = 0; i < N; ++i) {
        // (threads beyond the vector read its last piece along)
        const unsigned idx = min(tid + (unsigned)(i * kResThreads), last), r = (idx * inv) >> 20;
        off[i] = r * (WIDTH * 4u) + (idx - r * (unsigned)n4) * 16u;
    }
    receive<N>(p, x, off, base, v);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const unsigned r = off[i] / (WIDTH * 4u);
        f((int)r, (int)((off[i] - r * (WIDTH * 4u)) >> 4), v[i]);
    }
}

// End of a row: outputs are written by one work-group of the team.
__device__ __forceinline__ void res_finish_row(const ResidentParams &p, int b, int cnt)
{
    p.tok_len[b] = cnt;
    if (p.done) __hip_atomic_store(p.done + b, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Loads the projected frames of the next joint step's samples into LDS, straight from memory.
// Sample s's 16-byte piece k4 goes to position (k4 with its low four bits xored with s), so that
// sixteen samples' pieces of the same k sit in different banks.  Wave v takes samples v, v + 4, ...
// pidx: the frame row of sample `lane`, -1 for none.
template <int ROW, int NMT>
__device__ __forceinline__ void prefetch_frames(const ResidentParams &p, const RCtx &x, unsigned lds_p, int pidx)
{
    const int lane = again(x.lane);
    const int j4 = p.J >> 2;
#pragma unroll
    for (int i = 0; i < 16 * NMT / kResWaves; ++i) {
        const int s = x.wave + i * kResWaves;
        const int row = __builtin_amdgcn_readlane(pidx, s);
        if (row >= 0) {
            const char *src = reinterpret_cast<const char *>(p.P + (long long)row * p.J);
            const int l16 = lane ^ (s & 15);
            auto load = [&](int u) {
                const unsigned m = lds_p + (unsigned)(s * ROW * 4 + u * 1024);
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2"
                             :: "v"(l16 * 16 + u * 1024), "s"(__builtin_amdgcn_readfirstlane((int)m)), "s"(src) : "memory");
            };
            constexpr int U = ROW / 256;                  // whole runs of 64 pieces
            if (j4 == ROW / 4) {
#pragma unroll
                for (int u = 0; u < U; ++u) load(u);
                if (ROW / 4 > 64 * U && lane < ROW / 4 - 64 * U) load(U);
            } else {
#pragma unroll
                for (int u = 0; u < (ROW / 4 + 63) / 64; ++u)
                    if (u * 64 + lane < ROW / 4 && u * 64 + l16 < j4) load(u);
            }
        }
    }
}

__device__ __forceinline__ int from_lane(int v, int lane) { return __builtin_amdgcn_ds_bpermute(lane << 2, v); }

// KIND: ResidentKind; BF: bfloat16 mode; CLS: size class; RG: row groups (of 4 utterances) decoded
// at a time; NMT: tiles of 16 samples of a joint step
template <int KIND, bool BF, int CLS, int RG, int NMT>
__global__ void __launch_bounds__(kResThreads, 1) resident_kernel(const ResidentParams p)
{
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int NL = KIND == kResident1 ? 1 : 2;
    constexpr bool PAIR = KIND == kResident2Pair;
    constexpr int W = res_width(CLS), ROW = res_row(CLS), TS = res_team(CLS), XROW = res_xrow(BF, CLS);
    constexpr int NI = res_joint_steps(CLS), PR = res_piece_regs(BF), LREGS = res_lstm_regs(BF, CLS);
    constexpr int NB = (5 * RG + kResWaves - 1) / kResWaves;     // blocks of 16 (unit, row) pairs a wave finishes at most
    typedef Piece<BF> Pc;
    constexpr int NREC = PAIR ? 0 : NL;          // recurrent matrices the chain's work-groups hold
    constexpr ResidentBuf bo = resident_buf(CLS);
    constexpr ResidentLds lo = resident_lds(KIND, BF, CLS, RG, NMT);
    constexpr unsigned VROW = W * 4u, VSLOT = kResRows * VROW;                      // h and q rows
    constexpr unsigned KSLOT = kResSamples * TS * 8u, DSLOT = kResSamples * kMaxDur * 4u;
    constexpr unsigned PSLOT = TS * 10u * 64u * 4u;

    RCtx x;
    x.tid = threadIdx.x; x.lane = x.tid & 63;
    x.wave = __builtin_amdgcn_readfirstlane(x.tid >> 6);
    x.polls = 0;
    // Work-groups go to the XCDs round-robin: index % n_xcd is the XCD, index / n_xcd the place on it.
    const int n_xcd = p.pl.n_xcd, xcd = blockIdx.x % n_xcd, place = blockIdx.x / n_xcd;
    const int chain_xcds = PAIR ? n_xcd / 2 : n_xcd;
    const bool helper = PAIR && xcd >= chain_xcds;
    const int team = (xcd % chain_xcds) + chain_xcds * (place / TS);
    x.rank = place % TS;
    const int n_teams = p.pl.n_teams;
    int n_list = 0;
    for (int q = 0; q * n_teams < p.B; ++q) n_list += q * n_teams + ((q & 1) ? n_teams - 1 - team : team) < p.B;
    if (n_list == 0) {
        if (p.zero_stats && !helper && x.rank == 0 && x.tid < kStatCount) p.stats[(long long)team * kStatStride + x.tid] = 0;
        return;
    }
    x.buf = __builtin_amdgcn_make_buffer_rsrc(p.xbuf + (size_t)team * bo.bytes, 0, (int)bo.bytes, 0x00020000);

    // ---- put the mark into this work-group's share of every buffer -----------------------------
    {
        // (through to the memory side: whether the team may keep its words in the L2 is known below)
        const unsigned lo_b = helper ? bo.pre : 0u, hi_b = helper ? bo.bytes : (PAIR ? bo.pre : bo.hr[0]);
        const r4u mark = {kMark, kMark, kMark, kMark};
        for (unsigned o = lo_b + ((unsigned)x.rank * kResThreads + (unsigned)x.tid) * 16u; o < hi_b; o += TS * kResThreads * 16u)
            __builtin_amdgcn_raw_buffer_store_b128(mark, x.buf, (int)o, 0, 16);
    }
    if (x.tid == 0) { rc.ok = 1; rc.n_list = 0; rc.st_clamped = 0; rc.st_overflow = 0; }
    if (x.tid < kResSamples) { rc.s_k[x.tid] = p.blank; rc.s_d[x.tid] = 0; }
    if (x.lane < kResRows) {
        RRows &w = rc.rows[x.wave];
        w.b[x.lane] = 0; w.len[x.lane] = 0; w.t[x.lane] = 0; w.n[x.lane] = 0; w.cnt[x.lane] = 0; w.active[x.lane] = 0;
    }
    for (int i = x.tid * 16; i < lo.bytes; i += kResThreads * 16) *reinterpret_cast<r4u *>(lds + i) = (r4u){0, 0, 0, 0};
    // the marks have to be in memory before this work-group says that it is there
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    // ---- the team meets: everyone announces the XCD it runs on --------------------------------
    auto meet = [&]() {
        if (x.tid == 0) {
            const unsigned id = (__builtin_amdgcn_s_getreg((3 << 11) | 20) & 0xfu) + 1u;
            __hip_atomic_store(p.form + blockIdx.x, id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // lanes 0 .. TS-1 of the first wave: the chain's work-groups, lanes 32 ..: the helpers
        const int side = x.lane >> 5, r = x.lane & 31;
        const bool mine = x.wave == 0 && r < TS && (side == 0 || PAIR);
        unsigned v = 1;
        if (mine) {
            const unsigned *slot = p.form + (((team / chain_xcds) * TS + r) * n_xcd + team % chain_xcds + side * chain_xcds);
            unsigned spins = 0;
            v = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            while (v == 0u) {
                if (wait_expired(p, spins)) { rc.ok = 0; break; }
                v = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            x.polls += spins;
        }
        const unsigned first = (unsigned)__builtin_amdgcn_readlane((int)v, helper ? 32 : 0);
        const int same = !(mine && (side == 1) == helper && v != first);
        x.local = __syncthreads_and(same) != 0;
    };
    const unsigned prelane = ((unsigned)x.rank * 10u * 64u + (unsigned)x.lane) * 4u;     // + 256 per block
    // the lane's first piece of an activation row in the LSTM stages, and the distance of the following
    const int lane_x = (x.lane & 3) * XROW + (x.wave < 6 ? x.wave * res_lstm_pieces(CLS) : (x.wave - 6) * 4 + (x.lane >> 4)) * Pc::B;
    const int step_x = x.wave < 6 ? Pc::B : 8 * Pc::B;
    const int h4 = p.H >> 2;

    if (PAIR && helper) {
        // ---- helpers: W_hh of both layers times the candidate vectors ------------------------
        RegW<LREGS> w0, w1;
        const float *src = p.w_help + (long long)(x.rank * kResWaves + x.wave) * (2 * LREGS) * 64;
        load_regs(w0, src, 0, x.lane);
        load_regs(w1, src, LREGS, x.lane);
        meet();
        bool go = rc.ok != 0;
        for (unsigned n = 1; go; ++n) {
#pragma unroll
            for (int layer = 0; layer < 2; ++layer) {
                unsigned char *xr = lds + lo.xh + layer * 4 * RG * XROW;
                float *sums = reinterpret_cast<float *>(lds + lo.p);
                int seen = 0;
                receive_rows<RG, W>(p, x, bo.hr[layer] + RES_SLOT(n) * VSLOT, p.slots, h4, [&](int r, int k4, r4u v) {
                    if (v.x == kStop) seen = 1;
                    x_put<BF>(xr + r * XROW, k4, v);
                });
                if (__syncthreads_or(seen) || !rc.ok) { go = false; break; }
                lstm_stage<BF, CLS, RG>(layer == 0 ? w0 : w1, xr + lane_x, step_x, sums, x.wave, x.lane);
                __syncthreads();
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    const int blk = x.wave + i * kResWaves;
                    if (blk >= 5 * RG) break;
                    const unsigned o = prelane + (unsigned)blk * 256u;
                    put_far(x, o, bo.pre + ((unsigned)layer * kResSlots + RES_SLOT(n)) * PSLOT, word_of(stage_sum(sums, blk, x.lane)));
                    put_far(x, o, bo.pre + ((unsigned)layer * kResSlots + RES_SLOT(n + 2)) * PSLOT, kMark);
                }
            }
        }
        if (!rc.ok && x.tid == 0) __hip_atomic_fetch_or(p.status, 4, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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
        for (int l = 0; l < NREC; ++l) { load_regs(w_hh[l], src, first, x.lane); first += LREGS; }
        if (NL > 1) { load_regs(w_ih, src, first, x.lane); first += LREGS; }
        load_regs(w_pr, src, first, x.lane); first += res_pred_regs(BF, CLS);
        load_regs(w_ou, src, first, x.lane);
    }
    // utterances of the team: ranked by length (longest first, ties by index), dealt in serpentine
    // order; empty ones are complete from the start
    for (int b = x.tid; b < p.B; b += kResThreads) {
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
            else if (x.rank == 0) res_finish_row(p, b, 0);
        }
    }
    const int u0 = x.rank * p.pl.units, nu = max(0, min(p.pl.units, p.H - u0));
    const int g0 = x.rank * p.pl.jgroups, njg = max(0, min(p.pl.jgroups, (p.J >> 2) - g0));
    const bool has_tail = x.rank < p.pl.n_tail;      // a column of the tail, with column tile 0
    const int tcol = p.pl.nout_m + x.rank;
    if (x.tid < kResUnits * 4) rc.b1[x.tid] = (NL > 1 && x.tid < nu * 4) ? p.bias_l[((long long)p.H + u0) * 4 + x.tid] : 0.f;
    if (x.tid < 20) rc.bp[x.tid] = x.tid < njg * 4 ? p.b_pred[g0 * 4 + x.tid] : 0.f;
    if (x.tid < 32) rc.bo[x.tid] = x.rank * 32 + x.tid < p.pl.nout_m ? p.b_out[x.rank * 32 + x.tid] : 0.f;
    if (x.tid == 0) rc.bt = has_tail ? p.b_out[tcol] : 0.f;
    if (has_tail)
        for (int i = x.tid; i < ROW; i += kResThreads) {
            const float w = p.w_tail[(long long)x.rank * ROW + i];
            // (bfloat16 mode: bf16 values, followed by as many zeros)
            if (BF) reinterpret_cast<unsigned short *>(lds + lo.tail)[i] = (unsigned short)(__float_as_uint(w) >> 16);
            else reinterpret_cast<float *>(lds + lo.tail)[i] = w;
        }
    // What a lane finishes in the LSTM stages, see stage_sum: a row of the team, a unit and a gate.  Worked
    // out where it is used: kept for the whole loop, values like these take the registers that the
    // weights need.
    struct Place { int row, j, lu, gu; bool ok; };
    auto place_of = [&](int blk, int lane) {
        Place l;
        const int rg = blk >= 5 ? 1 : 0;
        l.row = rg * 4 + ((lane >> 2) & 3); l.j = lane & 3;
        l.lu = (blk - 5 * rg) * 4 + (lane >> 4);
        l.ok = l.lu < nu && l.j == 0 && l.row < p.slots;      // the lanes that publish it
        l.gu = min(u0 + l.lu, p.H - 1);
        return l;
    };
    const int n_blk = x.wave < 5 * RG ? (x.wave + kResWaves < 5 * RG ? 2 : 1) : 0;    // blocks this wave finishes
    // (joint output: a wave takes every eighth step of K for both column tiles)
    const int la = p.la, ns = p.slots * la;
    const unsigned inv_la = (1024u + (unsigned)la - 1u) / (unsigned)la;             // s / la for s < 32, la <= 16
    auto row_of = [&](int s) { return (int)(((unsigned)s * inv_la) >> 10); };
    constexpr int QS = ROW + 16;                     // floats per q row
    float *lq = reinterpret_cast<float *>(lds + lo.q);
    const unsigned lds_p = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)(lds + lo.p);
    float *part = reinterpret_cast<float *>(lds + lo.p);             // joint sums, see there
    float *tpart = reinterpret_cast<float *>(lds + lo.tpart);        // [wave][tile][16]
    float *g4 = reinterpret_cast<float *>(lds + lo.g4);              // [own, fifth group][wave][row group][16]

    meet();
    bool ok = rc.ok != 0;

    // state of the lane's cells, [layer][block]: committed and candidate cell value, recurrent
    // pre-activation W_hh h of the committed and of the candidate vector
    float cs[NL][NB], cc[NL][NB], ps[NL][NB], pc[NL][NB];
#pragma unroll
    for (int l = 0; l < NL; ++l)
#pragma unroll
        for (int i = 0; i < NB; ++i) { cs[l][i] = cc[l][i] = ps[l][i] = pc[l][i] = 0.f; }
    float *sums_ih = lq, *sums_rec = reinterpret_cast<float *>(lds + lo.rec);
    unsigned n_pred = 0, n_joint = 0;

    RRows &rows = rc.rows[x.wave];
    int next = 0;                     // first utterance of the list that no row has had
    int n_samples = 0, row_steps = 0;
    // What the loop control leaves for the steps, lane = row: last label, and what the prediction step
    // does with the row's candidate state (0 nothing, 1 take it, 2 start afresh); lane = sample:
    // the sample's row of the projected frames, -1 for none.
    int last = p.blank, action = 2, pidx = -1;
    // samples of the next joint step: `la` frames of every row in work
    auto set_up_samples = [&](int lane, int t, int b, int len, bool active) {
        const int r = min(row_of(lane & (kResSamples - 1)), kResRows - 1);
        const int fr = from_lane(t, r) + (lane - r * la), br = from_lane(b, r), lr = from_lane(active ? len : 0, r);
        pidx = (lane < ns && fr < lr) ? br * p.T + fr : -1;
        n_samples += __popcll(__ballot(pidx >= 0));
    };
    // rows that want one get the next utterances of the list
    auto refill = [&](int lane, bool want, int &b, int &len) {
        const unsigned long long m = __ballot(want);
        if (m == 0ull) return false;
        const int at = next + __popcll(m & ((1ull << lane) - 1ull));
        const bool got = want && at < rc.n_list;
        if (got) { b = rc.list_b[at]; len = rc.list_len[at]; }
        next += __popcll(m);
        return got;
    };
    __syncthreads();                  // the list is complete
    bool any_active, need_pred;
    {
        int b = 0, len = 0;
        const bool got = refill(x.lane, x.lane < p.slots, b, len);
        if (got) { rows.b[x.lane] = b; rows.len[x.lane] = len; rows.active[x.lane] = 1; }
        any_active = need_pred = __ballot(got) != 0ull;
        row_steps = __popcll(__ballot(got));
        set_up_samples(x.lane, 0, b, len, got);
    }
    // the rows of the embedding table (folded into the first layer) that the next prediction step adds
    float t0[NB];
    auto load_t0 = [&](int lane, int label) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
            if (i < n_blk) {
                const Place l = place_of(x.wave + i * kResWaves, lane);
                t0[i] = p.T0[((unsigned)from_lane(label, l.row) * (unsigned)p.H + (unsigned)l.gu) * 4u + (unsigned)l.j];
            }
    };
#pragma unroll
    for (int i = 0; i < NB; ++i) t0[i] = 0.f;
    if (need_pred) load_t0(x.lane, last);
#ifdef RNNT_PROFILE
    if (x.tid == 0) { for (int i = 0; i < 24; ++i) res_prof[i] = 0; res_prof_last = wall_clock64(); }
#endif

    while (ok && any_active) {
        if (!need_pred) prefetch_frames<ROW, NMT>(p, x, lds_p, pidx);
        if (need_pred) {
            // ---- prediction step -----------------------------------------------------------------
            ++n_pred;
            const unsigned n = n_pred;
            if (PAIR && n > 1) {
                // W_hh h of the last step's candidates
                unsigned v[2][NB], spins = 0;
                const unsigned s1 = bo.pre + RES_SLOT(n - 1) * PSLOT;
                for (;;) {
                    bool missing = false;
#pragma unroll
                    for (int l = 0; l < 2; ++l)
#pragma unroll
                        for (int i = 0; i < NB; ++i) {
                            v[l][i] = 0u;
                            if (i < n_blk) v[l][i] = get1(x, prelane + (unsigned)(x.wave + i * kResWaves) * 256u, s1 + (unsigned)l * kResSlots * PSLOT);
                        }
#pragma unroll
                    for (int l = 0; l < 2; ++l)
#pragma unroll
                        for (int i = 0; i < NB; ++i) missing = missing || v[l][i] == kMark;
                    if (__ballot(missing) == 0ull) break;
                    if (wait_expired(p, spins)) { rc.ok = 0; break; }
                }
                x.polls += spins;
#pragma unroll
                for (int l = 0; l < 2; ++l)
#pragma unroll
                    for (int i = 0; i < NB; ++i) pc[l][i] = __uint_as_float(v[l][i]);
            }
            RES_MARK(0);
            // rows that emitted take their candidate state, fresh rows start from zero
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                if (i >= n_blk) break;
                const int act = from_lane(action, place_of(x.wave + i * kResWaves, again(x.lane)).row);
#pragma unroll
                for (int l = 0; l < NL; ++l) {
                    cs[l][i] = act == 1 ? cc[l][i] : (act == 2 ? 0.f : cs[l][i]);
                    ps[l][i] = act == 1 ? pc[l][i] : (act == 2 ? 0.f : ps[l][i]);
                }
            }
            // publishes the lane's hidden value of a layer and clears the slot of two steps ago
            auto publish_h = [&](int layer, const Place &l, float h) {
                if (l.ok) {
                    const unsigned o = (unsigned)l.row * VROW + (unsigned)l.gu * 4u;
                    const unsigned s1 = RES_SLOT(n) * VSLOT, s2 = RES_SLOT(n + 2) * VSLOT;
                    put(x, o, bo.h[layer] + s1, word_of(h));
                    if (PAIR) { put_far(x, o, bo.hr[layer] + s1, word_of(h)); put_far(x, o, bo.hr[layer] + s2, kMark); }
                    put(x, o, bo.h[layer] + s2, kMark);
                }
            };
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                if (i >= n_blk) break;
                const Place l = place_of(x.wave + i * kResWaves, again(x.lane));
                float h;
                cell(ps[0][i] + t0[i], l.j, cs[0][i], cc[0][i], h);
                publish_h(0, l, h);
            }
            RES_MARK(1);
            unsigned char *x0 = lds + lo.xh, *x1 = lds + lo.xh + (NL - 1) * 4 * RG * XROW;
            receive_rows<RG, W>(p, x, bo.h[0] + RES_SLOT(n) * VSLOT, p.slots, h4, [&](int r, int k4, r4u v) { x_put<BF>(x0 + r * XROW, k4, v); });
            __syncthreads();
            // (here, and not earlier: a wave's loads return in order, and nothing waits for one of its
            // loads before the next vector arrives)
            prefetch_frames<ROW, NMT>(p, x, lds_p, pidx);
            RES_MARK(2);
            if constexpr (NL > 1) {
                lstm_stage<BF, CLS, RG>(w_ih, x0 + lane_x, step_x, sums_ih, x.wave, x.lane);
                __syncthreads();
                RES_MARK(3);
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    if (i >= n_blk) break;
                    const int lane = again(x.lane);
                    const Place l = place_of(x.wave + i * kResWaves, lane);
                    float h;
                    cell(stage_sum(sums_ih, x.wave + i * kResWaves, lane) + (ps[1][i] + rc.b1[l.lu * 4 + l.j]), l.j, cs[1][i], cc[1][i], h);
                    publish_h(1, l, h);
                }
                RES_MARK(4);
                // (while the hand-over is on its way) the recurrent part of the next step's first layer
                if constexpr (NREC > 1) lstm_stage<BF, CLS, RG>(w_hh[0], x0 + lane_x, step_x, sums_rec, x.wave, x.lane);
                RES_MARK(5);
                receive_rows<RG, W>(p, x, bo.h[1] + RES_SLOT(n) * VSLOT, p.slots, h4, [&](int r, int k4, r4u v) { x_put<BF>(x1 + r * XROW, k4, v); });
                __syncthreads();
                if constexpr (NREC > 1) {
#pragma unroll
                    for (int i = 0; i < NB; ++i)
                        if (i < n_blk) pc[0][i] = stage_sum(sums_rec, x.wave + i * kResWaves, again(x.lane));
                }
            }
            RES_MARK(6);
            // prediction-side joint projection: a group per pair of waves, and a fifth one in eighths of K
            {
                constexpr int NO = res_pred_own(CLS), NF = res_pred_fifth(CLS);
                const int lane = again(x.lane), q16 = lane >> 4, cb = (lane >> 2) & 3, j = lane & 3;
                const unsigned char *xl = x1 + j * XROW + (lane >> 2) * Pc::B;
#pragma unroll
                for (int rg = 0; rg < RG; ++rg) {
                    const unsigned char *xr = xl + rg * 4 * XROW;
                    Pc v[NO], v5[NF];
#pragma unroll
                    for (int i = 0; i < NO; ++i) v[i].load(xr + (2 * i + (x.wave >> 2)) * 16 * Pc::B);
                    // (pieces beyond the last one have zero weights: any piece will do)
#pragma unroll
                    for (int i = 0; i < NF; ++i) v5[i].load(x1 + j * XROW + rg * 4 * XROW + min(i * 128 + x.wave * 16 + (lane >> 2), W / 4 - 1) * Pc::B);
                    r4f a[2], a5 = (r4f){0.f, 0.f, 0.f, 0.f};
                    a[0] = a[1] = a5;
#pragma unroll
                    for (int i = 0; i < NO; ++i)
#pragma unroll
                        for (int e = 0; e < Pc::N; ++e) {
                            v[i].mfma(e, &w_pr.w[i * PR], a[(i * Pc::N + e) & 1]);
                            if (i < NF) v5[i < NF ? i : 0].mfma(e, &w_pr.w[(NO + (i < NF ? i : 0)) * PR], a5);
                        }
                    const float s = sum_blocks(a[0] + a[1]), s5 = sum_blocks(a5);
                    if (cb == 0) {
                        g4[(x.wave * RG + rg) * 16 + q16 * 4 + j] = s;
                        g4[((kResWaves + x.wave) * RG + rg) * 16 + q16 * 4 + j] = s5;
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                __syncthreads();
                // one value per thread: column j of group g, row 4 rg + q
                const int tid = again(x.tid), o = tid & 15, gr = tid >> 4, rg = RG == 1 ? 0 : gr / 5, g = gr - rg * 5, r = rg * 4 + (o >> 2);
                if (gr < 5 * RG && g < njg && r < p.slots) {
                    float s;
                    if (g < 4) {
                        s = g4[(g * RG + rg) * 16 + o] + g4[((g + 4) * RG + rg) * 16 + o];
                    } else {
                        const float *f = g4 + (kResWaves * RG + rg) * 16 + o;
                        constexpr int st = RG * 16;
                        s = ((f[0] + f[st]) + (f[2 * st] + f[3 * st])) + ((f[4 * st] + f[5 * st]) + (f[6 * st] + f[7 * st]));
                    }
                    const unsigned at = (unsigned)r * VROW + (unsigned)((g0 + g) * 4 + (o & 3)) * 4u;
                    put(x, at, bo.q + RES_SLOT(n) * VSLOT, word_of(s + rc.bp[g * 4 + (o & 3)]));
                    put(x, at, bo.q + RES_SLOT(n + 2) * VSLOT, kMark);
                }
            }
            RES_MARK(7);
            // (while q is on its way) the recurrent part of the top layer's next step
            if constexpr (NREC > 0) lstm_stage<BF, CLS, RG>(w_hh[NREC - 1], x1 + lane_x, step_x, sums_rec, x.wave, x.lane);
            RES_MARK(8);
            receive_rows<RG, W>(p, x, bo.q + RES_SLOT(n) * VSLOT, p.slots, p.J >> 2, [&](int r, int k4, r4u v) {
                *reinterpret_cast<r4u *>(lq + r * QS + k4 * 4) = v;
            });
            RES_MARK(9);
        }
        // ---- joint step ----------------------------------------------------------------------------
        ++n_joint;
        const unsigned jn = n_joint;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the frames of this wave's samples are in LDS
        __syncthreads();
        if constexpr (NREC > 0) {
            if (need_pred) {
#pragma unroll
                for (int i = 0; i < NB; ++i)
                    if (i < n_blk) pc[NL - 1][i] = stage_sum(sums_rec, x.wave + i * kResWaves, again(x.lane));
            }
        }
        RES_MARK(10);
        {
            r4f acc[NMT][2];                 // [tile of samples][column tile]
            const int lane = again(x.lane), m16 = lane & 15, kq = lane >> 4;
            if constexpr (BF) {
                // relu(P + q) as bf16 in place: a 16-byte fp32 piece becomes an 8-byte one, in the first or the
                // second half of its place by the sample's parity (banks)
                const int tid = again(x.tid), sr = tid >> 5, pr = tid & 31;
#pragma unroll
                for (int mt = 0; mt < NMT; ++mt) {
                    const int s = mt * 16 + sr;
                    unsigned char *prow = lds + lo.p + s * ROW * 4 + (((pr & ~15) | ((pr ^ s) & 15)) * 16);
                    const float *q = lq + min(row_of(s), 4 * RG - 1) * QS + pr * 4;
#pragma unroll
                    for (int i = 0; i < ROW / 128; ++i) {
                        const float4 pa = *reinterpret_cast<const float4 *>(prow + i * 512), qa = *reinterpret_cast<const float4 *>(q + i * 128);
                        uint2 z;
                        z.x = bf16_pair(fmaxf(pa.x + qa.x, 0.f), fmaxf(pa.y + qa.y, 0.f));
                        z.y = bf16_pair(fmaxf(pa.z + qa.z, 0.f), fmaxf(pa.w + qa.w, 0.f));
                        *reinterpret_cast<uint2 *>(prow + i * 512 + (s & 1) * 8) = z;
                    }
                }
                __syncthreads();
            }
            // Piece k4 = 32 ii + 4 wave + kq of sample m16: its low bits are the same for all steps.  fp32: the
            // operand is formed on the way.
            const int k40 = x.wave * 4 + kq;
            const unsigned char *pr = lds + lo.p + m16 * ROW * 4 + ((k40 & 16) | ((k40 ^ m16) & 15)) * 16;
#pragma unroll
            for (int mt = 0; mt < NMT; ++mt) acc[mt][0] = acc[mt][1] = (r4f){0.f, 0.f, 0.f, 0.f};
            if constexpr (BF) {
                struct Q { float a, b; };
                r4f tacc[NMT];
                r4s z[NMT][NI];
#pragma unroll
                for (int mt = 0; mt < NMT; ++mt) {
                    tacc[mt] = (r4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ii = 0; ii < NI; ++ii) z[mt][ii] = *reinterpret_cast<const r4s *>(pr + mt * 16 * ROW * 4 + ii * 512 + (m16 & 1) * 8);
                }
#pragma unroll
                for (int ii = 0; ii < NI; ++ii)
#pragma unroll
                    for (int mt = 0; mt < NMT; ++mt)
#pragma unroll
                        for (int c = 0; c < 2; ++c) {
                            const float *w = &w_ou.w[(ii * 2 + c) * PR];
                            acc[mt][c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(z[mt][ii], __builtin_bit_cast(r4s, Q{w[0], w[1]}), acc[mt][c], 0, 0, 0);
                        }
                if (has_tail) {
                    // the tail column as an operand of its own: lane column 0 reads the weights, the others zeros
                    const unsigned char *wt = lds + lo.tail + (m16 == 0 ? 0 : ROW * 2) + k40 * 8;
#pragma unroll
                    for (int ii = 0; ii < NI; ++ii) {
                        const r4s w = *reinterpret_cast<const r4s *>(wt + ii * 256);
#pragma unroll
                        for (int mt = 0; mt < NMT; ++mt) tacc[mt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(z[mt][ii], w, tacc[mt], 0, 0, 0);
                    }
                    // lane 16 q holds column 0 of samples 4 q ..
#pragma unroll
                    for (int mt = 0; mt < NMT; ++mt)
                        if (m16 == 0) *reinterpret_cast<r4f *>(tpart + (x.wave * 2 + mt) * 16 + kq * 4) = tacc[mt];
                }
            } else {
                const float *wt = reinterpret_cast<const float *>(lds + lo.tail) + k40 * 4;
                const float *q[NMT];
                float tl[NMT];
#pragma unroll
                for (int mt = 0; mt < NMT; ++mt) {
                    q[mt] = lq + min(row_of(mt * 16 + m16), 4 * RG - 1) * QS + k40 * 4;
                    tl[mt] = 0.f;
                }
                // one step ahead of the matrix instructions, no further (registers)
                float4 pv[NMT], qv[NMT], wv;
                wv = *reinterpret_cast<const float4 *>(wt);
#pragma unroll
                for (int mt = 0; mt < NMT; ++mt) {
                    pv[mt] = *reinterpret_cast<const float4 *>(pr + mt * 16 * ROW * 4);
                    qv[mt] = *reinterpret_cast<const float4 *>(q[mt]);
                }
#pragma unroll
                for (int ii = 0; ii < NI; ++ii) {
                    float z[NMT][4];
                    float4 wn = wv;
#pragma unroll
                    for (int mt = 0; mt < NMT; ++mt) {
                        z[mt][0] = fmaxf(pv[mt].x + qv[mt].x, 0.f); z[mt][1] = fmaxf(pv[mt].y + qv[mt].y, 0.f);
                        z[mt][2] = fmaxf(pv[mt].z + qv[mt].z, 0.f); z[mt][3] = fmaxf(pv[mt].w + qv[mt].w, 0.f);
                        if (ii + 1 < NI) {
                            pv[mt] = *reinterpret_cast<const float4 *>(pr + mt * 16 * ROW * 4 + (ii + 1) * 512);
                            qv[mt] = *reinterpret_cast<const float4 *>(q[mt] + (ii + 1) * 128);
                        }
                    }
                    if (ii + 1 < NI) wn = *reinterpret_cast<const float4 *>(wt + (ii + 1) * 128);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int mt = 0; mt < NMT; ++mt) {
#pragma unroll
                            for (int c = 0; c < 2; ++c)
                                acc[mt][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(z[mt][e], w_ou.w[(ii * 2 + c) * 4 + e], acc[mt][c], 0, 0, 0);
                            tl[mt] = fmaf(z[mt][e], e == 0 ? wv.x : (e == 1 ? wv.y : (e == 2 ? wv.z : wv.w)), tl[mt]);
                        }
                    wv = wn;
                    // (the sums are opaque here: otherwise they move behind the loop, under the
                    // condition they are used under, with every z kept in a register till then)
#pragma unroll
                    for (int mt = 0; mt < NMT; ++mt) asm volatile("" : "+v"(tl[mt]));
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (has_tail) {
#pragma unroll
                    for (int mt = 0; mt < NMT; ++mt) {
                        float a = tl[mt], b = tl[mt];
                        swap32(a, b); a += b; b = a;
                        swap16(a, b); a += b;
                        if (lane < 16) tpart[(x.wave * 2 + mt) * 16 + lane] = a;
                    }
                }
            }
            __syncthreads();                  // the frames' place is free for the sums
            RES_MARK(11);
            // every wave's sums to LDS, [wave][sample][column]; then sixteen lanes per sample, two columns each
#pragma unroll
            for (int mt = 0; mt < NMT; ++mt)
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        part[((x.wave * NMT + mt) * 16 + kq * 4 + v) * kResSumRow + c * 16 + m16] = acc[mt][c][v];
            __syncthreads();
            const int tid = again(x.tid);
            if (tid < 16 * NMT * 16) {
                const int s = tid >> 4, col = (tid & 15) * 2, gcol = x.rank * 32 + col;
                float2 o[kResWaves];
#pragma unroll
                for (int w = 0; w < kResWaves; ++w)
                    o[w] = *reinterpret_cast<const float2 *>(part + (w * NMT * 16 + s) * kResSumRow + col);
                const float2 bias = *reinterpret_cast<const float2 *>(&rc.bo[col]);
                const float l0 = (((o[0].x + o[1].x) + (o[2].x + o[3].x)) + ((o[4].x + o[5].x) + (o[6].x + o[7].x))) + bias.x;
                const float l1 = (((o[0].y + o[1].y) + (o[2].y + o[3].y)) + ((o[4].y + o[5].y) + (o[6].y + o[7].y))) + bias.y;
                const int n_tok = min(p.VT, p.pl.nout_m);
                const float m0 = gcol < n_tok ? l0 : -INFINITY, m1 = gcol + 1 < n_tok ? l1 : -INFINITY;
                const float mine = fmaxf(m0, m1);
                float m = fmaxf(mine, dppf<0xB1>(mine));
                m = fmaxf(m, dppf<0x4E>(m)); m = fmaxf(m, dppf<0x141>(m)); m = fmaxf(m, dppf<0x140>(m));
                // the first lane of the sixteen that holds the maximum publishes (without a token column: lane 0)
                const unsigned hit = (unsigned)(__ballot(mine == m && gcol < n_tok) >> (tid & 48)) & 0xffffu;
                const int first = hit ? __ffs((int)hit) - 1 : 0;
                int ix = hit ? (m0 == m ? gcol : gcol + 1) : 0x7fffffff;
                float tail = -INFINITY;
                if (has_tail) {
                    float t[kResWaves];
#pragma unroll
                    for (int w = 0; w < kResWaves; ++w) t[w] = tpart[(w * 2 + (s >> 4)) * 16 + (s & 15)];
                    tail = (((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]))) + rc.bt;
                    if (tcol >= p.VT) {
                        if ((tid & 15) == 0 && s < ns) {
                            const unsigned d = ((unsigned)s * kMaxDur + (unsigned)(tcol - p.VT)) * 4u;
                            put(x, d, bo.dur + RES_SLOT(jn) * DSLOT, word_of(tail));
                            put(x, d, bo.dur + RES_SLOT(jn + 2) * DSLOT, kMark);
                        }
                        tail = -INFINITY;
                    } else if (tail > m) {
                        m = tail; ix = tcol;
                    }
                }
                if (p.tdt && gcol + 1 >= p.VT && gcol < p.pl.nout_m && s < ns) {
                    // duration columns inside the column tiles
#pragma unroll
                    for (int c = 0; c < 2; ++c)
                        if (gcol + c >= p.VT && gcol + c < p.pl.nout_m) {
                            const unsigned d = ((unsigned)s * kMaxDur + (unsigned)(gcol + c - p.VT)) * 4u;
                            put(x, d, bo.dur + RES_SLOT(jn) * DSLOT, word_of(c ? l1 : l0));
                            put(x, d, bo.dur + RES_SLOT(jn + 2) * DSLOT, kMark);
                        }
                }
                const unsigned ko = ((unsigned)s * TS + (unsigned)x.rank) * 8u;
                if ((tid & 15) == first && s < ns) {
                    put2(x, ko, bo.key + RES_SLOT(jn) * KSLOT, (r2u){word_of(m), (unsigned)ix});
                    put2(x, ko, bo.key + RES_SLOT(jn + 2) * KSLOT, (r2u){kMark, kMark});
                }
                if (p.logps) {
                    float e = (m0 > -INFINITY ? expf(m0 - m) : 0.f) + (m1 > -INFINITY ? expf(m1 - m) : 0.f);
                    e += dppf<0xB1>(e); e += dppf<0x4E>(e); e += dppf<0x141>(e); e += dppf<0x140>(e);
                    if (tail > -INFINITY) e += expf(tail - m);
                    if ((tid & 15) == 0 && s < ns) {
                        put(x, ko / 2, bo.lse + RES_SLOT(jn) * (KSLOT / 2), word_of(e));
                        put(x, ko / 2, bo.lse + RES_SLOT(jn + 2) * (KSLOT / 2), kMark);
                    }
                }
            }
        }
        RES_MARK(12);
        // ---- argmax over the team: TS / 2 adjacent lanes per sample, two candidates per lane --------
        {
            const int tid = again(x.tid), lane = tid & 63;
            constexpr int L = TS / 2;
            static_assert(16 * NMT * L <= kResThreads, "one piece per thread");
            const int s = tid / L;
            if ((x.wave * 64) / L < ns) {
                const unsigned off[1] = {(unsigned)min(tid, ns * L - 1) * 16u};
                r4u v[1];
                receive<1>(p, x, off, bo.key + RES_SLOT(jn) * KSLOT, v);
                const float va = __uint_as_float(v[0].x), vb = __uint_as_float(v[0].z);
                const int ia = (int)v[0].y, ib = (int)v[0].w;
                const bool second = vb > va || (vb == va && ib < ia);
                const float bv = second ? vb : va;
                const int bi = second ? ib : ia;
                float m = fmaxf(bv, dppf<0xB1>(bv));
                m = fmaxf(m, dppf<0x4E>(m));
                if (L > 4) m = fmaxf(m, dppf<0x141>(m));
                if (L > 8) m = fmaxf(m, dppf<0x140>(m));
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
                    t += dppf<0xB1>(t); t += dppf<0x4E>(t);
                    if (L > 4) t += dppf<0x141>(t);
                    if (L > 8) t += dppf<0x140>(t);
                    lp2 = -logf(t);
                }
                if (win && s < ns) {
                    rc.s_k[s] = (unsigned)bi < (unsigned)p.VT ? bi : p.blank;
                    rc.s_v[s] = m + 0.0f;
                    if (p.logps) rc.s_lp[s] = lp2;
                }
            }
            RES_MARK(13);
            if (p.tdt) {
                // one lane per sample (last wave): best duration, lowest index on ties
                const int s = tid - (kResThreads - 64);
                if (s >= 0 && s < ns) {
                    r4u d0, d1;
                    unsigned spins = 0;
                    const unsigned sl = bo.dur + RES_SLOT(jn) * DSLOT, o = (unsigned)s * kMaxDur * 4u;
                    for (;;) {
                        d0 = get4(x, o, sl); d1 = get4(x, o + 16u, sl);
                        bool all = true;
#pragma unroll
                        for (int i = 0; i < kMaxDur; ++i)
                            if (i < p.D) all = all && (i < 4 ? d0[i & 3] : d1[i & 3]) != kMark;
                        if (all) break;
                        if (wait_expired(p, spins)) { rc.ok = 0; break; }
                    }
                    x.polls += spins;
                    float best = -INFINITY; int bd = 0;
#pragma unroll
                    for (int i = 0; i < kMaxDur; ++i)
                        if (i < p.D) {
                            const float dv = __uint_as_float(i < 4 ? d0[i & 3] : d1[i & 3]);
                            if (i == 0 || dv > best) { best = dv; bd = i; }
                        }
                    rc.s_d[s] = bd;
                }
            }
        }
        __syncthreads();
        RES_MARK(14);
        // ---- loop control: every wave for itself, lane = row -----------------------------------------
        {
            const int lane = again(x.lane), r = lane & (kResRows - 1);
            const int mine = rc.s_k[lane & (kResSamples - 1)];
            int b = rows.b[r], len = rows.len[r], t = rows.t[r], nn = rows.n[r], cnt = rows.cnt[r];
            bool active = lane < p.slots && rows.active[r];
            int pos, found = 0, dval = 0;
            if (!p.tdt && p.VT == p.V1) {
                // a blank moves on by one frame: the first label among the frames the row still has
                const unsigned long long labels = __ballot(lane < ns && mine != p.blank);
                const int avail = min(la, len - t);
                const unsigned seg = (unsigned)(labels >> (r * la)) & ((1u << avail) - 1u);
                pos = seg ? __ffs((int)seg) - 1 : avail;
                found = seg != 0u;
            } else {
                // lane = sample: where the walk goes from it (nowhere from a label or beyond the row's
                // frames); then the steps are doubled until every one reaches its end
                const int sr = min(row_of(lane & (kResSamples - 1)), kResRows - 1), si = lane - sr * la;
                int to = si;
                const int d = p.tdt ? rc.s_d[lane & (kResSamples - 1)] & (kMaxDur - 1) : 0;
                if (mine >= p.V1) to += max(p.durations[mine - p.V1], 1);            // big blank: its span of frames
                else if (mine == p.blank) to += p.tdt ? max(p.durations[d], 1) : 1;
                if (pidx < 0) to = si;
#pragma unroll
                for (int i = 1; i < 16; i *= 2) {
                    const int on = from_lane(to, (sr * la + min(to, la - 1)) & 63);
                    if (to < la) to = on;
                }
                pos = from_lane(to, (r * la) & 63);
                found = pos < la && t + pos < len;
            }
            found = found && active;
            const int s = max(0, min(r * la + pos, kResSamples - 1));
            const int k = rc.s_k[s];
            if (p.tdt) dval = p.durations[rc.s_d[s] & (kMaxDur - 1)];
            // the label's row of the embedding table is what the next prediction step waits for
            if (found) last = k;
            load_t0(lane, last);
            const int t_emit = t + pos;
            bool ended = false;
            action = 0;
            if (active) {
                t += pos;
                if (pos > 0) nn = 0;
                if (found) {
                    if (x.rank == 0 && x.wave == 0) {
                        if (cnt < p.cap) {
                            const long long o = (long long)b * p.cap + cnt;
                            p.tokens[o] = k;
                            if (p.frames) p.frames[o] = t_emit;
                            if (p.logits) p.logits[o] = rc.s_v[s];
                            if (p.logps) p.logps[o] = rc.s_lp[s];
                            if (p.durs) p.durs[o] = dval;
                        } else {
                            rc.st_overflow = 1;
                        }
                    }
                    ++cnt;
                    action = 1;
                    if (p.tdt && dval > 0) { t += dval; nn = 0; }
                    else { ++nn; if (nn == p.S) { ++t; nn = 0; } }
                }
                if (t >= len) {
                    ended = true; active = false; action = 0;
                    if (x.rank == 0 && x.wave == 0) res_finish_row(p, b, cnt);
                }
            }
            if (__ballot(ended) != 0ull) {
                const bool got = refill(lane, ended, b, len);
                if (got) { t = 0; nn = 0; cnt = 0; active = true; action = 2; last = p.blank; rows.b[r] = b; rows.len[r] = len; }
                if (__ballot(got) != 0ull) load_t0(lane, last);
                if (lane < kResRows) rows.active[r] = active;
            }
            if (lane < kResRows) { rows.t[r] = t; rows.n[r] = nn; rows.cnt[r] = cnt; }
            const unsigned long long moved = __ballot(action != 0);      // rows whose next step has new inputs
            any_active = __ballot(active) != 0ull;
            need_pred = moved != 0ull;
            row_steps += __popcll(moved);
            set_up_samples(lane, t, b, len, active);
        }
        ok = rc.ok != 0;
        RES_MARK(15);
    }
    __syncthreads();
    if (PAIR && rc.ok) {
        // the helpers wait for the next candidate vector: tell them that there is none
        const unsigned o = bo.hr[0] + RES_SLOT(n_pred + 1) * VSLOT;
        for (int i = x.tid; i < p.slots * nu; i += kResThreads) {
            const int r = i / nu, u = i - r * nu;
            put_far(x, (unsigned)r * VROW + (unsigned)(u0 + u) * 4u, o, kStop);
        }
    }
    if (x.tid == 0) {
        int st = 0;
        if (x.rank == 0) st = (rc.st_clamped ? 1 : 0) | (rc.st_overflow ? 2 : 0);
        if (!rc.ok) st |= 4;
        if (st) __hip_atomic_fetch_or(p.status, st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (x.rank == 0) {
            long long *sp = p.stats + (long long)team * kStatStride;
            if (p.zero_stats) { sp[kStatPred] = 0; sp[kStatJoint] = 0; sp[kStatSamples] = 0; sp[kStatPolls] = 0; }
            sp[kStatPred] += p.count_rows ? row_steps : (int)n_pred; sp[kStatJoint] += n_joint; sp[kStatSamples] += n_samples; sp[kStatPolls] += x.polls;
sp[kStatPolls] += x.polls;
#ifdef RNNT_PROFILE
            for (int i = 0; i < 24; ++i) sp[kStatCount + i] = res_prof[i];
#endif
        }
    }
}

template <int KIND, bool BF, int CLS, int RG, int NMT>
hipError_t launch_resident_one(const ResidentParams &p, bool plain, hipStream_t stream)
{
    const void *fn = reinterpret_cast<const void *>(&resident_kernel<KIND, BF, CLS, RG, NMT>);
    constexpr unsigned lds = (unsigned)resident_lds(KIND, BF, CLS, RG, NMT).bytes;
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
