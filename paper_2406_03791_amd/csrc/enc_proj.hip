// Encoder-side joint projection  P[b, t, :] = W_enc x[b, t, :] + b_enc  for every
// valid frame, as one MFMA GEMM (fp32: v_mfma_f32_32x32x2_f32; bfloat16 mode:
// v_mfma_f32_32x32x16_bf16), and the one-time folding of the embedding table into the
// first LSTM layer's input term.
#include "engine.h"

namespace rnnt {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef __bf16 v4b __attribute__((ext_vector_type(4)));
typedef __bf16 v8b __attribute__((ext_vector_type(8)));

// nearest bfloat16 value (ties to even) of a float, as a float; NaN and infinities pass through
__device__ __forceinline__ float bf16_rne(float v)
{
    unsigned u = __float_as_uint(v);
    if ((u & 0x7f800000u) != 0x7f800000u) { u += 0x7fffu + ((u >> 16) & 1u); u &= 0xffff0000u; }
    return __uint_as_float(u);
}

// What a decode call needs cleared before its decode kernel starts, done by the blocks of the
// projection on the way (a kernel of its own would be one more launch in front of a decode of a
// few hundred microseconds): the synchronisation words, and the output rows' fill (-1 and 0).
__device__ __forceinline__ void init_call(const CallInit &ci, int B)
{
    if (blockIdx.x == 0) {
        for (int i = threadIdx.x; i < ci.n_form; i += blockDim.x) ci.form[i] = 0u;
        if (threadIdx.x == 0 && ci.abort_flag) { *ci.abort_flag = 0u; *ci.status = 0; }
        if (threadIdx.x == 0 && ci.stats) { ci.stats[kStatCallStart] = wall_clock64(); ci.stats[kStatDecodeEnd] = 0; }
    }
    if (!ci.tokens) return;
    const long long n = (long long)B * ci.cap, step = (long long)gridDim.x * blockDim.x;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) {
        ci.tokens[i] = -1;
        if (ci.frames) ci.frames[i] = -1;
        if (ci.logits) ci.logits[i] = 0.f;
        if (ci.logps) ci.logps[i] = 0.f;
        if (ci.durs) ci.durs[i] = -1;
    }
}

__device__ __forceinline__ const char *uniform(const char *p)
{
    const unsigned long long u = reinterpret_cast<unsigned long long>(p);
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)u), hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(u >> 32));
    return reinterpret_cast<const char *>((unsigned long long)hi << 32 | lo);
}

// One block (four waves) computes BM rows x BN columns: WM x WN waves, each its part, or WK > 1 waves
// with the whole tile and every WK-th slice of K each, summed at the end.  Blocks are numbered by
// valid row tile over all utterances, and the column tiles of a row tile follow each other on one XCD,
// whose L2 then holds the frames.  (Numbered by utterance and tile, padding included, the XCDs
// had up to a third more or less than the average to do.)
// K goes in slices of 32: both operands' rows are 128 bytes in LDS, loaded straight from memory
// into the other of two buffers while a slice is computed, 16-byte pieces xored with the row so
// that reads of 16 bytes by 8 rows meet different banks.  A lane reads four k's at once (K is the same
// permutation of itself in both operands), and the loop has next to no vector instructions, which
// the fp32 matrix instructions would share their pipe with.
// fp32, 1024 x 640, valid rows of ragged batches: 11300 rows 145 us (a grid over utterances and padded tiles
// took 195), 43100 rows 494 us (711), 500 rows 15 us (50); a dense batch of 45000 rows runs at 122 TFLOP/s,
// the library's product of that shape at 123.
// bfloat16 mode (BF): the frames are rounded to bfloat16 (ties to even) between LDS and the matrix
// instruction, W_enc holds bfloat16 values already (its low halves are zero), products are
// exact in fp32 and the sums are fp32: 11300 rows 55 us (64).
template <int BM, int BN, int WM, int WN, int WK, bool BF>
__global__ void __launch_bounds__(256)
enc_proj_kernel(const float *__restrict__ x, const int *__restrict__ enc_len, const float *__restrict__ w_enc,
                const float *__restrict__ b_enc, float *__restrict__ proj, int B, int T, int F, int J, const CallInit ci)
{
    static_assert(WM * WN * WK == 4, "four waves");
    constexpr int MI = BM / WM / 32, NI = BN / WN / 32;              // tiles of 32 x 32 of a wave
    constexpr int SLICE = (BM + BN) * 128, STAGE = SLICE * WK;       // bytes of a slice of K, of the slices in work
    constexpr int CNT = (BM + BN) / 8 * WK / 4;                      // loads (of 8 rows) of a wave per stage
    __shared__ __align__(16) unsigned char lds[2 * STAGE];
    init_call(ci, B);
    const TopWord call = !BF && ci.p_top ? ci.p_top[kTopWords * kTopStride] : 0;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ny = (J + BN - 1) / BN, slot = blockIdx.x >> 3, tile = (slot / ny) * 8 + (blockIdx.x & 7), n0 = slot % ny * BN;
    // the utterance and row that valid row tile number `tile` is of
    int b = -1, len = 0, m0 = 0;
    for (int b0 = 0, run = 0; b0 < B && b < 0; b0 += 64) {
        const int l = b0 + lane < B ? min(max(enc_len[b0 + lane], 0), T) : 0, t = (l + BM - 1) / BM;
        int p = t;
#pragma unroll
        for (int i = 1; i < 64; i *= 2) { const int o = __shfl_up(p, i); if (lane >= i) p += o; }
        const unsigned long long m = __ballot(run + p > tile);
        if (m != 0ull) {
            const int at = __builtin_ctzll(m);
            b = b0 + at;
            len = __builtin_amdgcn_readlane(l, at);
            m0 = (tile - run - __builtin_amdgcn_readlane(p - t, at)) * BM;
        }
        run += __builtin_amdgcn_readlane(p, 63);
    }
    if (b < 0) return;
    const int wk = wave % WK, wn = wave / WK % WN, wm = wave / WK / WN;
    const char *xa = reinterpret_cast<const char *>(x + ((long long)b * T + m0) * F), *wb = reinterpret_cast<const char *>(w_enc + (long long)n0 * F);
    // load i of this wave: rows 8 rb .. 8 rb + 7 of the frames, then of the weights; rows beyond the end
    // repeat the last one and are not stored
    auto block_of = [&](int i) { return WK == 1 ? wave * CNT + i : i; };
    const int r8 = lane >> 3, piece = (lane & 7) ^ r8;
    unsigned voff[CNT];
#pragma unroll
    for (int i = 0; i < CNT; ++i) {
        const int rb = block_of(i), row = rb < BM / 8 ? min(rb * 8 + r8, T - 1 - m0) : min((rb - BM / 8) * 8 + r8, J - 1 - n0);
        voff[i] = (unsigned)(row * F + piece * 4) * 4u;
    }
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
    auto k_of = [&](int s) { return (WK == 1 ? s : s * WK + wk) * 32; };
    auto load = [&](int s, int buf) {
        const int k0 = k_of(s);
        if (k0 >= F || (F - k0 < 32 && piece >= 4)) return;          // (F is a multiple of 16)
#pragma unroll
        for (int i = 0; i < CNT; ++i) {
            const int rb = block_of(i);
            const char *src = uniform((rb < BM / 8 ? xa : wb) + k0 * 4);
            const unsigned m = (unsigned)__builtin_amdgcn_readfirstlane((int)(lds0 + (unsigned)(buf * STAGE + wk * SLICE + rb * 1024)));
            asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2" :: "v"(voff[i]), "s"(m), "s"(src) : "memory");
        }
    };
    v16f acc[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;
    const int kh = lane >> 5, c = lane & 31;
    const unsigned char *la[4];              // the lane's row, its pieces 2 g + kh
#pragma unroll
    for (int g = 0; g < 4; ++g) la[g] = lds + wk * SLICE + c * 128 + (((2 * g + kh) ^ (c & 7)) << 4);
    auto read = [&](int g, int buf, v4f (&a)[MI], v4f (&w)[NI]) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) a[mi] = *reinterpret_cast<const v4f *>(la[g] + buf * STAGE + (wm * MI + mi) * 4096);
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) w[ni] = *reinterpret_cast<const v4f *>(la[g] + buf * STAGE + BM * 128 + (wn * NI + ni) * 4096);
    };
    auto compute = [&](int s, int buf) {
        const int k0 = k_of(s);
        if (WK > 1 && k0 >= F) return;
#pragma unroll
        for (int g = 0; g < 4; g += 2) {
            if (g == 2 && F - k0 < 32) break;
            v4f a[2][MI], w[2][NI];
            read(g, buf, a[0], w[0]);
            read(g + 1, buf, a[1], w[1]);
            if constexpr (BF) {
                v8b a8[MI], w8[NI];
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
                    a8[mi] = __builtin_shufflevector(__builtin_convertvector(a[0][mi], v4b), __builtin_convertvector(a[1][mi], v4b), 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) {
                    const v4u p = __builtin_bit_cast(v4u, w[0][ni]), q = __builtin_bit_cast(v4u, w[1][ni]);
                    v4u o;                   // the upper halves
                    o[0] = __builtin_amdgcn_perm(p[1], p[0], 0x07060302u); o[1] = __builtin_amdgcn_perm(p[3], p[2], 0x07060302u);
                    o[2] = __builtin_amdgcn_perm(q[1], q[0], 0x07060302u); o[3] = __builtin_amdgcn_perm(q[3], q[2], 0x07060302u);
                    w8[ni] = __builtin_bit_cast(v8b, o);
                }
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a8[mi], w8[ni], acc[mi][ni], 0, 0, 0);
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                            for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[h][mi][e], w[h][ni][e], acc[mi][ni], 0, 0, 0);
            }
        }
    };
    // a stage's loads have had the time of the stage before; with WK > 1 a wave's slices are its own
    auto step = [&](int s, int ns, int buf) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (WK == 1) __syncthreads();
        if (s + 1 < ns) load(s + 1, buf ^ 1);
        compute(s, buf);
        if (WK > 1) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
    const int ns = ((F + 31) / 32 + WK - 1) / WK;
    load(0, 0);
    for (int s = 0; s < ns; s += 2) {
        step(s, ns, 0);
        if (s + 1 < ns) step(s + 1, ns, 1);
    }
    // accumulator register v of lane l holds row 8*(v/4) + 4*(l/32) + v%4, column l%32
    float top = 0.f;                 // the largest finite value
    bool infinite = false;
    auto store = [&](int row, int col, float v) {
        if (row < len) {
            proj[((long long)b * T + row) * J + col] = v;
            if (!BF) { infinite = infinite || v == INFINITY; top = fmaxf(top, v == INFINITY ? 0.f : v); }
        }
    };
    if constexpr (WK == 1) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const int col = n0 + (wn * NI + ni) * 32 + c;
                if (col >= J) continue;
                const float bias = b_enc[col];
#pragma unroll
                for (int v = 0; v < 16; ++v) store(m0 + (wm * MI + mi) * 32 + 8 * (v >> 2) + 4 * kh + (v & 3), col, acc[mi][ni][v] + bias);
            }
    } else {
        static_assert(WK == 1 || (WK == 4 && MI == 1 && NI == 1), "one tile");
        float *red = reinterpret_cast<float *>(lds);
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 16; ++v) red[(wk * 16 + v) * 64 + lane] = acc[0][0][v];
        __syncthreads();
        const int col = n0 + c;
        if (col < J) {
            const float bias = b_enc[col];
#pragma unroll
            for (int v = wk * 4; v < wk * 4 + 4; ++v)
                store(m0 + 8 * (v >> 2) + 4 * kh + (v & 3), col,
                      ((red[v * 64 + lane] + red[(16 + v) * 64 + lane]) + (red[(32 + v) * 64 + lane] + red[(48 + v) * 64 + lane])) + bias);
        }
    }
    if (!BF && ci.p_top) {
#pragma unroll
        for (int i = 32; i; i >>= 1) top = fmaxf(top, __shfl_xor(top, i));
        TopWord *word = ci.p_top + (blockIdx.x % kTopWords) * kTopStride;
        const bool any = __ballot(infinite) != 0ull;
        if (lane == 0) {
            atomicMax(word, call << 16 | (__float_as_uint(top) + 0xffffu) >> 16);
            if (any) atomicMax(word + 1, call << 16 | 1u);
        }
    }
}

hipError_t launch_encoder_projection(const float *enc_out, const int *enc_len, const float *w_enc,
                                     const float *b_enc, float *proj, int B, int T, int F, int J,
                                     bool round_x, const CallInit &ci, hipStream_t stream)
{
    auto run = [&](auto kernel, int bm, int bn) {
        const long long tiles = (long long)B * ((T + bm - 1) / bm), ny = (J + bn - 1) / bn;
        hipLaunchKernelGGL(kernel, dim3((unsigned)((tiles + 7) / 8 * 8 * ny)), dim3(256), 0, stream, enc_out, enc_len, w_enc, b_enc,
                           proj, B, T, F, J, ci);
    };
    // Few rows: small tiles with K split over the waves, so that there are blocks for all compute units and the
    // chain of each is short (fp32, 500 rows: 15 against 28 us; even at 3700 rows in fp32, 2.4 blocks of 32 x 128
    // per unit; in the bfloat16 mode 10 against 17 and, at 3700 rows, 38 against 26).
    const long long blocks = (long long)B * ((T + 31) / 32) * ((J + 127) / 128);
    if (round_x) {
        if (blocks <= 512) run(enc_proj_kernel<32, 32, 1, 1, 4, true>, 32, 32);
        else run(enc_proj_kernel<64, 128, 2, 2, 1, true>, 64, 128);
    } else {
        // (32-row tiles waste the least on an utterance's last one: with 64 rows 5 % slower at 44700 rows)
        if (blocks <= 1024) run(enc_proj_kernel<32, 32, 1, 1, 4, false>, 32, 32);
        else run(enc_proj_kernel<32, 128, 1, 4, 1, false>, 32, 128);
    }
    return hipGetLastError();
}

__global__ void reset_resident_kernel(unsigned *form, int n_form, unsigned *abort_flag)
{
    for (int i = threadIdx.x; i < n_form; i += blockDim.x) form[i] = 0u;
    if (threadIdx.x == 0) *abort_flag = 0u;
}

hipError_t launch_reset_resident(unsigned *form, int n_form, unsigned *abort_flag, hipStream_t stream)
{
    hipLaunchKernelGGL(reset_resident_kernel, dim3(1), dim3(256), 0, stream, form, n_form, abort_flag);
    return hipGetLastError();
}

__global__ void round_bf16_kernel(float *v, long long n)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) v[i] = bf16_rne(v[i]);
}

hipError_t launch_round_bf16(float *v, long long n, hipStream_t stream)
{
    hipLaunchKernelGGL(round_bf16_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, v, n);
    return hipGetLastError();
}

// one thread per (label v, unit u, gate g)
__global__ void fold_embedding_kernel(const float *__restrict__ emb, const float *__restrict__ w_ih0,
                                      const float *__restrict__ b_ih0,
                                      const float *__restrict__ b_hh0, float *__restrict__ T0, int V1,
                                      int E, int H, int round_bf16)
{
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (long long)V1 * H * 4) return;
    const int g = (int)(idx & 3);
    const int u = (int)((idx >> 2) % H);
    const int v = (int)((idx >> 2) / H);
    const float *wr = w_ih0 + (long long)(g * H + u) * E;
    const float *er = emb + (long long)v * E;
    float s = 0.f;
    if (round_bf16) { for (int e = 0; e < E; ++e) s += bf16_rne(wr[e]) * bf16_rne(er[e]); }
    else { for (int e = 0; e < E; ++e) s += wr[e] * er[e]; }
    T0[idx] = s + b_ih0[g * H + u] + b_hh0[g * H + u];
}

hipError_t launch_fold_embedding(const float *emb, const float *w_ih0, const float *b_ih0,
                                 const float *b_hh0, float *T0, int V1, int E, int H,
                                 bool round_bf16, hipStream_t stream)
{
    const long long n = (long long)V1 * H * 4;
    hipLaunchKernelGGL(fold_embedding_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream,
                       emb, w_ih0, b_ih0, b_hh0, T0, V1, E, H, round_bf16 ? 1 : 0);
    return hipGetLastError();
}

}  // namespace rnnt
