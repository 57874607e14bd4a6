// Encoder-side joint projection  P[b, t, :] = W_enc x[b, t, :] + b_enc  for every
// valid frame, as one product on the 16-bit matrix instructions (fp32: two fp16 parts of every value), and the one-time folding of the embedding table into the
// first LSTM layer's input term.
#include "engine.h"
#include "parts.h"
#include <type_traits>

namespace rnnt {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef __bf16 v8b __attribute__((ext_vector_type(8)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

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

// A wave's 32 rows of frames: tile number `tile` of the valid rows of all utterances, in tiles of an utterance's own.
struct RowTile { int b, len, m0; };       // b < 0: there are fewer tiles
__device__ __forceinline__ RowTile row_tile(const int *__restrict__ enc_len, int B, int T, int tile, int lane)
{
    RowTile r{-1, 0, 0};
    for (int b0 = 0, run = 0; b0 < B && r.b < 0; b0 += 64) {
        const int l = b0 + lane < B ? min(max(enc_len[b0 + lane], 0), T) : 0, t = (l + 31) / 32;
        int p = t;
#pragma unroll
        for (int i = 1; i < 64; i *= 2) { const int o = __shfl_up(p, i); if (lane >= i) p += o; }
        const unsigned long long m = __ballot(run + p > tile);
        if (m != 0ull) {
            const int at = __builtin_ctzll(m);
            r.b = b0 + at;
            r.len = __builtin_amdgcn_readlane(l, at);
            r.m0 = (tile - run - __builtin_amdgcn_readlane(p - t, at)) * 32;
        }
        run += __builtin_amdgcn_readlane(p, 63);
    }
    return r;
}

// A wave computes 32 rows x NI tiles of 32 columns on v_mfma 32x32x16.  WK == 1: a block is four waves with a tile
// of rows each, the columns' weights are shared through LDS, and while a slice of K is multiplied the next one's
// frames are split and the loads after it are on their way.  WK == 4 or 8: a block is that many waves with the same tile and
// every WK-th slice each, summed at the end; the weights go straight to registers, and a wave has the loads of four
// slices in flight together.
// Tiles of rows are numbered over the valid rows of all utterances, and the column blocks of a group of tiles follow each
// other on one XCD, whose L2 then holds the frames.
//
// K goes in slices of 32: frames are loaded straight into LDS, rows of 128 bytes, 16-byte pieces xored with
// the row so that reads of 16 bytes by 8 rows meet different banks; weights lie in memory as the lanes take them.
// Bfloat16 mode (BF): frames are rounded to bfloat16 (ties to even) on their way from LDS, products are exact and the
// sums fp32.
//
// fp32: frames and weights are two fp16 parts each (22 bits and a sign), weights with a power of two for each column,
// frames with one for each row; three products (low times low is beyond what fp32 sums keep), those with a low part
// summed apart.  The row's power of two is that of its first slice, to 2^12 .. 2^13 with room for values eight times
// as large; a larger one later on lowers it, and the sums with it.  Infinite frames have no parts, and where sixteen values of a
// frame are all far below its largest (2^-14 to 2^-18 of it) theirs have too few bits: such a tile is computed
// once more from the fp32 values (as is everything for weights that are not finite).
// On the fp32 matrix instructions the product was bound by their rate, 154 TFLOP/s; these would do 59 us of it in 33.
// Against 64 bits, rms, frames of 1024 values: 4.1e-7 (WK > 1: 2.3e-7), on the fp32 instructions 1.06e-6 (5.4e-7).
//
// 1024 x 640, valid rows of ragged batches, us (before, on 32x32x2 and, in the bfloat16 mode, with weights of 32 bits
// in LDS and a rounding for each column tile):
//   rows               500   1757   3144   4350   7271  11800  45300
//   fp32               9.6   22.4   33.5   37.8   49.4   58.2    223
//     before          13.9   33.7   55.4   70.4   90.5    133    481
//   bfloat16 mode      7.8   13.7   19.6   24.4   26.7   28.4    128
//     before           8.5   21.6   25.2   26.3   32.7   53.5    218
template <int WK, int NI, bool BF>
__global__ void __launch_bounds__(WK == 8 ? 512 : 256, 2)
enc_proj_kernel(const float *__restrict__ x, const int *__restrict__ enc_len, const EncWeights w, float *__restrict__ proj, int B, int T, int F, int J,
                const CallInit ci)
{
    static_assert(WK == 1 || WK == 4 || WK == 8, "tiles or slices for the waves");
    constexpr int WAVES = WK == 8 ? 8 : 4, PL = BF ? 1 : 2;
    constexpr int DEPTH = WK == 1 ? 2 : 4;                           // slices of a wave in LDS
    constexpr int XBYTES = WAVES * DEPTH * 4096, WSLICE = NI * 2 * PL * 1024;
    constexpr int LDS = XBYTES + (WK == 1 ? 2 * WSLICE : 0);
    static_assert(WK == 1 || WAVES * NI * 4096 <= XBYTES, "the sums of the waves fit");
    __shared__ __align__(16) unsigned char lds[LDS];
    init_call(ci, B);
    const TopWord call = !BF && ci.p_top ? *ci.p_top : 0;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ny = (J + NI * 32 - 1) / (NI * 32), slot = blockIdx.x >> 3, group = (slot / ny) * 8 + (blockIdx.x & 7), n0 = slot % ny * (NI * 32);
    RowTile r = row_tile(enc_len, B, T, WK == 1 ? group * 4 + wave : group, lane);
    if (WK == 1) {
        if (__syncthreads_or(r.b >= 0) == 0) return;
        if (r.b < 0) r = RowTile{0, 0, 0};                           // (computes something and stores nothing)
    } else if (r.b < 0) return;
    const int kh = lane >> 5, c = lane & 31, r8 = lane >> 3, piece = (lane & 7) ^ r8;
    const int nks = F / 16, n_slices = (nks + 1) / 2;                // (F is a multiple of 16)
    const char *xa = reinterpret_cast<const char *>(x + ((long long)r.b * T + r.m0) * F);
    const char *wa = reinterpret_cast<const char *>(w.parts) + (long long)(n0 / 32) * nks * (PL * 1024);
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
    auto to_lds = [&](const char *from, unsigned off, unsigned to) {
        const char *src = uniform(from);
        const unsigned m = (unsigned)__builtin_amdgcn_readfirstlane((int)(lds0 + to));
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2" :: "v"(off), "s"(m), "s"(src) : "memory");
    };
    // rows beyond the end repeat the last one (what lies there may be anything) and are not stored
    unsigned voff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) voff[i] = (unsigned)(min(i * 8 + r8, max(r.len - 1 - r.m0, 0)) * F + piece * 4) * 4u;
    auto load_x = [&](int s, int buf) {
        if (s * 2 + 1 >= nks && piece >= 4) return;                  // half a slice
#pragma unroll
        for (int i = 0; i < 4; ++i) to_lds(xa + s * 128, voff[i], (unsigned)((wave * DEPTH + buf) * 4096 + i * 1024));
    };
    v16f big[NI], small[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int v = 0; v < 16; ++v) big[ni][v] = small[ni][v] = 0.f;
    float scale = 1.f, limit = -1.f;                                 // of row c; the largest value that it takes
    bool bad = false;
    // the scale of rows with a value above their limit
    auto rescale = [&](float m) {
        float o = m;
        const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(o), false, false);
        m = fmaxf(__uint_as_float(both[0]), __uint_as_float(both[1]));
        const int e = max((int)(__float_as_uint(m) >> 23) - 127, -100);
        bad = bad || m == INFINITY;
        const bool change = m > limit && m != INFINITY;
        const float next = change ? __uint_as_float((unsigned)(127 + 12 - e) << 23) : scale;
        const float f = limit < 0.f ? 1.f : next * __uint_as_float(0x7f000000u - __float_as_uint(scale));
        scale = next;
        limit = fminf(65000.f * __uint_as_float(0x7f000000u - __float_as_uint(scale)), 3.4e38f);        // (an infinity is above it)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) { big[ni] *= f; small[ni] *= f; }
    };
    // The lane's values of a slice in buffer buf, and their parts (half a slice: zeros, without an instruction on them)
    struct Slice { v4f a[4]; };
    struct Parts { v4u high[2], low[2]; };
    const unsigned char *xr = lds + wave * DEPTH * 4096 + c * 128;
    auto read = [&](int s, int buf) {
        Slice v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v.a[i] = *reinterpret_cast<const v4f *>(xr + buf * 4096 + (((i >> 1) * 4 + 2 * kh + (i & 1)) ^ (c & 7)) * 16);
        if (s * 2 + 1 >= nks) v.a[2] = v.a[3] = (v4f){0.f, 0.f, 0.f, 0.f};
        return v;
    };
    auto split = [&](const Slice &v) {
        Parts p;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (BF) {
                p.high[i >> 1][(i & 1) * 2] = bf16_pair(v.a[i].x, v.a[i].y); p.high[i >> 1][(i & 1) * 2 + 1] = bf16_pair(v.a[i].z, v.a[i].w);
            } else {
                const v4f o = v.a[i] * scale;
                unsigned h, l;
                f16_parts(o.x, o.y, h, l); p.high[i >> 1][(i & 1) * 2] = h; p.low[i >> 1][(i & 1) * 2] = l;
                f16_parts(o.z, o.w, h, l); p.high[i >> 1][(i & 1) * 2 + 1] = h; p.low[i >> 1][(i & 1) * 2 + 1] = l;
            }
        }
        return p;
    };
    auto largest = [&](const Slice &v) {
        float m = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) m = fmaxf(fmaxf(fmaxf(fabsf(v.a[i].x), fabsf(v.a[i].y)), m), fmaxf(fabsf(v.a[i].z), fabsf(v.a[i].w)));
        return m;
    };
    // Far below the row's largest value, parts have fewer bits than fp32: a lane's 16 values of a slice are off by 2^-25 of
    // the scaled range, more than 2^-23 of the largest of them from here on.
    auto lost = [&](float m) { return m > 0.f && m * scale < 0.25f; };
    // the parts of a slice, if need be with another scale
    auto parts_of = [&](const Slice &v) {
        if constexpr (!BF) {
            const float m = largest(v);
            if (__ballot(m > limit) != 0ull) rescale(m);
            bad = bad || lost(m);
        }
        return split(v);
    };
    auto multiply = [&](const Parts &p, bool both, auto weight) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (k == 1 && !both) continue;
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                if constexpr (BF) {
                    big[ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8b, weight(ni, k, 0)), __builtin_bit_cast(v8b, p.high[k]), big[ni], 0, 0, 0);
                } else {
                    const v8h wh = __builtin_bit_cast(v8h, weight(ni, k, 0)), wl = __builtin_bit_cast(v8h, weight(ni, k, 1));
                    const v8h high = __builtin_bit_cast(v8h, p.high[k]), low = __builtin_bit_cast(v8h, p.low[k]);
                    small[ni] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wh, low, small[ni], 0, 0, 0);
                    big[ni] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wh, high, big[ni], 0, 0, 0);
                    small[ni] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wl, high, small[ni], 0, 0, 0);
                }
            }
        }
    };
    if constexpr (WK == 1) {
        constexpr int CW = NI * 2 * PL / 4;                          // pieces of the weights' slice that a wave loads
        auto load_w = [&](int s) {
#pragma unroll
            for (int i = 0; i < CW; ++i) {
                const int q = wave * CW + i, ni = q / (2 * PL), k = q / PL % 2, pl = q % PL;
                if (s * 2 + k < nks)
                    to_lds(wa + (((long long)ni * nks + s * 2 + k) * PL + pl) * 1024, (unsigned)lane * 16u, (unsigned)(XBYTES + (s & 1) * WSLICE + q * 1024));
            }
        };
        // While a slice is multiplied, the next one's values are split, its weights and the frames after it are on their way.
        auto step = [&](int s, const Parts &p, Parts &next, auto more_) {
            constexpr bool MORE = decltype(more_)::value;
            const int buf = s & 1;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (MORE) load_w(s + 1);
            if (s + 2 < n_slices) load_x(s + 2, buf);
            const unsigned char *wl = lds + XBYTES + buf * WSLICE + lane * 16;
            auto weight = [&](int ni, int k, int pl) { return *reinterpret_cast<const v4u *>(wl + ((ni * 2 + k) * PL + pl) * 1024); };
            if constexpr (MORE) {
                const Slice v = read(s + 1, buf ^ 1);
                next = split(v);
                multiply(p, true, weight);
                if constexpr (!BF) {
                    const float m = largest(v);
                    if (__ballot(m > limit) != 0ull) { rescale(m); next = split(v); }
                    bad = bad || lost(m);
                }
            } else multiply(p, s * 2 + 1 < nks, weight);
        };
        load_w(0);
        load_x(0, 0);
        if (n_slices > 1) load_x(1, 1);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        Parts p = parts_of(read(0, 0)), next;
        for (int s = 0; s + 1 < n_slices; ++s) { step(s, p, next, std::true_type()); p = next; }
        step(n_slices - 1, p, next, std::false_type());
    } else {
        const auto wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(wa), 0, NI * nks * (PL * 1024), 0x00020000);
        // (four slices at a time, all their loads in flight together)
        for (int s0 = wave; s0 < n_slices; s0 += WK * DEPTH) {
            v4u wr[DEPTH][NI][2][PL];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // (read before it is written again)
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                const int s = s0 + d * WK;
                if (s < n_slices) load_x(s, d);
            }
#pragma unroll
            for (int d = 0; d < DEPTH; ++d)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                    for (int k = 0; k < 2; ++k)
#pragma unroll
                        for (int pl = 0; pl < PL; ++pl) {
                            const int ks = min((s0 + d * WK) * 2 + k, nks - 1);
                            wr[d][ni][k][pl] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(wbuf, lane * 16, ((ni * nks + ks) * PL + pl) * 1024, 0));
                        }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                const int s = s0 + d * WK;
                if (s < n_slices) multiply(parts_of(read(s, d)), s * 2 + 1 < nks, [&](int ni, int k, int pl) { return wr[d][ni][k][pl]; });
            }
        }
    }
    // Accumulator register v of lane l holds column 8 (v / 4) + 4 (l / 32) + v % 4 of a tile, row l % 32.
    // In four columns from `col` on: a sum's value less the scales and with the bias.
    float back = 1.f;
    bool plain = BF;                 // sums without scales
    if constexpr (!BF) {
        back = __uint_as_float(0x7f000000u - __float_as_uint(scale));
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) big[ni] += small[ni];
        if ((__ballot(bad) != 0ull && r.len > 0) || *w.not_finite != 0u) {
            plain = true;
            const float *row = x + ((long long)r.b * T + max(min(r.m0 + c, r.len - 1), 0)) * F + kh * 4;
            const float *col[NI];
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                col[ni] = w.plain + (long long)min(n0 + ni * 32 + c, J - 1) * F + kh * 4;
#pragma unroll
                for (int v = 0; v < 16; ++v) big[ni][v] = 0.f;
            }
            // (eight k's, four of either half of the lanes: which k an instruction takes does not matter, both operands take the same)
            for (int s = WK == 1 ? 0 : wave; s < n_slices; s += WK)
                for (int k = s * 32; k < min(s * 32 + 32, F); k += 8) {
                    const v4f xv = *reinterpret_cast<const v4f *>(row + k);
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) {
                        const v4f wv = *reinterpret_cast<const v4f *>(col[ni] + k);
#pragma unroll
                        for (int e = 0; e < 4; ++e) big[ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[e], xv[e], big[ni], 0, 0, 0);
                    }
                }
        }
    }
    auto value = [&](int ni, int j) {
        v4f o = {big[ni][j * 4], big[ni][j * 4 + 1], big[ni][j * 4 + 2], big[ni][j * 4 + 3]};
        if (!plain) o *= *reinterpret_cast<const v4f *>(w.inverse + n0 + ni * 32 + j * 8 + kh * 4) * back;
        return o;
    };
    float top = 0.f;                 // the largest finite value
    const bool wide = J % 4 == 0 && (reinterpret_cast<uintptr_t>(proj) & 15u) == 0;
    auto store = [&](int ni, int j, v4f v) {
        const int col = n0 + ni * 32 + j * 8 + kh * 4;
        v += *reinterpret_cast<const v4f *>(w.bias + col);
        if (r.m0 + c >= r.len || col >= J) return;
        float *to = proj + ((long long)r.b * T + r.m0 + c) * J + col;
        if (wide) *reinterpret_cast<v4f *>(to) = v;
        else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < J) to[e] = v[e];
        }
        if (!BF) {
#pragma unroll
            for (int e = 0; e < 4; ++e) top = fmaxf(top, v[e] == INFINITY ? 0.f : v[e]);
        }
    };
    if constexpr (WK == 1) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int j = 0; j < 4; ++j) store(ni, j, value(ni, j));
    } else {
        v4f *red = reinterpret_cast<v4f *>(lds);
        __syncthreads();
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int j = 0; j < 4; ++j) red[((ni * 4 + j) * WK + wave) * 64 + lane] = value(ni, j);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NI * 4 / WK; ++i) {
            const int at = wave * (NI * 4 / WK) + i;
            v4f o[WK];
#pragma unroll
            for (int q = 0; q < WK; ++q) o[q] = red[(at * WK + q) * 64 + lane];
#pragma unroll
            for (int q = WK / 2; q; q /= 2)
#pragma unroll
                for (int k = 0; k < q; ++k) o[k] += o[k + q];
            store(at >> 2, at & 3, o[0]);
        }
    }
    if (!BF && ci.p_top) {
#pragma unroll
        for (int i = 32; i; i >>= 1) top = fmaxf(top, __shfl_xor(top, i));
        if (lane == 0) atomicMax(ci.p_top + top_words(r.b) + blockIdx.x % kTopParts * kTopStride, call << 16 | (__float_as_uint(top) + 0xffffu) >> 16);
    }
}

hipError_t launch_encoder_projection(const float *enc_out, const int *enc_len, const EncWeights &w, float *proj, int B, int T, int F, int J,
                                     bool round_x, const CallInit &ci, hipStream_t stream)
{
    const long long tiles = (long long)B * ((T + 31) / 32);
    auto run = [&](auto kernel, long long groups, int columns, int threads) {
        const long long ny = (J + columns - 1) / columns;
        hipLaunchKernelGGL(kernel, dim3((unsigned)((groups + 7) / 8 * 8 * ny)), dim3((unsigned)threads), 0, stream, enc_out, enc_len, w, proj, B, T, F, J, ci);
    };
    // Few rows: K is split over the waves, so that there are blocks for all compute units and the chain of each is short.
    // The lines are drawn at blocks of the split form: up to one per compute unit, and K of more than 16 slices, eight
    // waves are better than four (500 rows of 1024: 9.6 against 10.9 us; 1000 rows 17.6 against 14.3); above
    // some five per unit whole K is (1024 x 640: at 1280 blocks 33.5 against 36.4 us, at 1920 38.3 against 37.8;
    // 256 x 320: at 960 12.7 against 16.7, at 1520 18.9 against 17.5).
    const long long blocks = tiles * ((J + 63) / 64);
    auto pick = [&](auto bf_) {
        constexpr bool BF = decltype(bf_)::value;
        if (blocks <= 256 && F > 512) run(enc_proj_kernel<8, 2, BF>, tiles, 64, 512);
        else if (blocks <= 1400) run(enc_proj_kernel<4, 2, BF>, tiles, 64, 256);
        else run(enc_proj_kernel<1, 4, BF>, (tiles + 3) / 4, 128, 256);
    };
    if (round_x) pick(std::true_type());
    else pick(std::false_type());
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

// T0 = emb W_ih0^T + b_ih0 + b_hh0, rows [unit][gate].  64 labels by 64 of a row's values per block, four by four of them per thread, one
// ascending sum each; 32 k's of both operands in LDS at a time.  Bound by its multiply-adds and LDS reads, about as long each.  (1025 labels, 640
// units, E 640: 6800 us with a thread per value that read both rows from memory, more than half of creating an engine; 98 us.)
constexpr int kFoldTile = 64, kFoldK = 32, kFoldRow = kFoldTile + 4;
template <bool BF>
__global__ void __launch_bounds__(256) fold_embedding_kernel(const float *__restrict__ emb, const float *__restrict__ w_ih0,
                                                             const float *__restrict__ b_ih0, const float *__restrict__ b_hh0,
                                                             float *__restrict__ T0, int V1, int E, int H)
{
    __shared__ __align__(16) float ev[kFoldK * kFoldRow], wv[kFoldK * kFoldRow];
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4, c0 = blockIdx.x * kFoldTile, v0 = blockIdx.y * kFoldTile;
    float s[4][4] = {};
    for (int k0 = 0; k0 < E; k0 += kFoldK) {
        const int k = tid & (kFoldK - 1), n = min(kFoldK, E - k0);
        if (k0) __syncthreads();
        // (rows beyond the last label or column: the last one's, not written below)
#pragma unroll
        for (int i = 0; i < kFoldTile * kFoldK / 256; ++i) {
            const int row = (tid / kFoldK) + i * (256 / kFoldK), c = min(c0 + row, 4 * H - 1), v = min(v0 + row, V1 - 1);
            if (k < n) {
                const float w = w_ih0[(long long)((c & 3) * H + (c >> 2)) * E + k0 + k], e = emb[(long long)v * E + k0 + k];
                wv[k * kFoldRow + row] = BF ? bf16_rne(w) : w;
                ev[k * kFoldRow + row] = BF ? bf16_rne(e) : e;
            }
        }
        __syncthreads();
#pragma unroll 8
        for (int kk = 0; kk < n; ++kk) {
            const float4 w = *reinterpret_cast<const float4 *>(wv + kk * kFoldRow + 4 * tx), e = *reinterpret_cast<const float4 *>(ev + kk * kFoldRow + 4 * ty);
            const float wa[4] = {w.x, w.y, w.z, w.w}, ea[4] = {e.x, e.y, e.z, e.w};
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) s[i][j] += wa[j] * ea[i];
        }
    }
    const int u = (c0 >> 2) + tx;
    if (u >= H) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int v = v0 + 4 * ty + i;
        if (v >= V1) break;
        float t[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) t[g] = s[i][g] + b_ih0[g * H + u] + b_hh0[g * H + u];
        reinterpret_cast<float4 *>(T0)[(long long)v * H + u] = make_float4(t[0], t[1], t[2], t[3]);
    }
}

hipError_t launch_fold_embedding(const float *emb, const float *w_ih0, const float *b_ih0,
                                 const float *b_hh0, float *T0, int V1, int E, int H,
                                 bool round_bf16, hipStream_t stream)
{
    const dim3 grid((unsigned)((4LL * H + kFoldTile - 1) / kFoldTile), (unsigned)((V1 + kFoldTile - 1) / kFoldTile));
    hipLaunchKernelGGL(round_bf16 ? fold_embedding_kernel<true> : fold_embedding_kernel<false>, grid, dim3(256), 0, stream,
                       emb, w_ih0, b_ih0, b_hh0, T0, V1, E, H);
    return hipGetLastError();
}

}  // namespace rnnt
