// Register images of the resident decode kernel's work-groups, the projection's weights as its matrix instructions
// take them, and the scales of fp32 weights, made on the device from the model's matrices (on the host, the parts of the Parakeet shape's 6.4 million weights took
// 33 of 55 ms of an engine's creation).
#include "engine.h"
#include "resident.h"

namespace rnnt {
namespace {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));

// bits of the nearest bf16 number (ties to even)
__device__ __forceinline__ unsigned bf16_of(float v)
{
    unsigned u = __float_as_uint(v);
    if ((u & 0x7f800000u) != 0x7f800000u) u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

// One wave per row of a matrix: 2^k with 2^14 <= 2^k max|row| < 2^15, as far as it and its inverse (times the scale of
// hidden values) are ordinary floats; check[0] is raised by a value that is not finite, check[1] is the largest row
// sum of magnitudes and `extra`, or zero, as a float's bits: what comes before the joint's relu is bounded from above, and
// a unit that its bias switches off, with -inf or -1e30, says nothing of the others.
__global__ void __launch_bounds__(256) row_scales_kernel(const float *__restrict__ w, int rows, int K, float *__restrict__ scale, const float *__restrict__ extra, unsigned *check)
{
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= rows) return;
    unsigned top = 0;
    float sum = 0.f;
    for (int k = lane; k < K; k += 64) {
        const float v = fabsf(w[(long long)row * K + k]);
        top = max(top, __float_as_uint(v));          // (NaN is the largest)
        sum += v;
    }
#pragma unroll
    for (int i = 32; i; i >>= 1) { top = max(top, (unsigned)__shfl_xor((int)top, i)); sum += __shfl_xor(sum, i); }
    if (lane) return;
    if (top >= 0x7f800000u) atomicOr(check, 1u);
    if (extra) atomicMax(check + 1, __float_as_uint(fminf(fmaxf((sum + extra[row]) * 1.001f, 0.f), kResHuge)));
    const float m = __uint_as_float(top);
    const int e = top >= 0x7f800000u ? 0 : (m > 0.f ? min(14 - ilogbf(m), 126 - kResHiddenExp) : 0);
    scale[row] = ldexpf(1.f, e);
}

// Which row of the matrix output o of a work-group is: gate o % 4 of its unit o / 4 (gates: rows of an LSTM matrix),
// or column first + o; -1 for none.
struct Rows { int gates, first, count, per_rank; };      // per_rank: units or columns of a work-group, count: all of them
__device__ __forceinline__ int row_of(const Rows &r, int rank, int o)
{
    const int at = r.gates ? o >> 2 : o, n = min(r.per_rank, r.count - rank * r.per_rank);
    if (at >= n) return -1;
    return r.gates ? (o & 3) * r.count + rank * r.per_rank + at : rank * r.per_rank + at;
}

// A wave's eighth of K of T tiles of 16 outputs, one thread per pair of values and work-group: lane l holds output
// l % 16 of a tile, of a block of 32 k's the eight from 8 (l / 16) on, of a half block four.  dst: the images
// [rank][wave][nreg][lane], a run of registers from `first` on (res_place).  scale (fp32): a row's, else bf16 values; whole: fp32
// values, four registers of a half block.
__global__ void __launch_bounds__(256) pack_tiles_kernel(unsigned *__restrict__ dst, int nreg, int first, const float *__restrict__ w, int K, const float *__restrict__ scale,
                                                         Rows rows, int T, int cls, int ts, bool whole)
{
    const int nh = res_halves(cls), nf = nh / 2, pairs = nh * 2;         // pairs of a lane per tile
    const int total = ts * kResWaves * T * pairs * 64;
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int lane = idx & 63, pair = (idx >> 6) % pairs, rest = (idx >> 6) / pairs;
    const int t = rest % T, wave = rest / T % kResWaves, rank = rest / T / kResWaves;
    const int kb = min(pair >> 2, nf), i = pair - kb * 4, g = lane >> 4;
    const int row = row_of(rows, rank, t * 16 + (lane & 15));
    const int k = wave * nh * 16 + kb * 32 + g * (kb < nf ? 8 : 4) + 2 * i;
    float v[2] = {0.f, 0.f};
    if (row >= 0)
        for (int e = 0; e < 2; ++e)
            if (k + e < K) v[e] = w[(long long)row * K + k + e];
    unsigned *to = dst + ((long long)(rank * kResWaves + wave) * nreg + first) * 64;
    const int n = res_tile_regs(!scale && !whole, cls, T);
    if (whole) {
        for (int e = 0; e < 2; ++e) to[res_place(n, t * 4 + 2 * i + e, lane)] = __float_as_uint(v[e]);
        return;
    }
    if (!scale) {
        unsigned u = 0;
        for (int e = 0; e < 2; ++e) u |= bf16_of(v[e]) << (16 * e);
        to[res_place(n, res_tile_at(true, cls, T, kb, t, 0) + i, lane)] = u;
        return;
    }
    const float s = row >= 0 ? scale[row] : 0.f;
    h2 high, low;
    for (int e = 0; e < 2; ++e) {
        const float a = v[e] * s;
        high[e] = (_Float16)a;
        low[e] = (_Float16)(a - (float)high[e]);
    }
    to[res_place(n, res_tile_at(false, cls, T, kb, t, 0) + i, lane)] = __builtin_bit_cast(unsigned, high);
    to[res_place(n, res_tile_at(false, cls, T, kb, t, 1) + i, lane)] = __builtin_bit_cast(unsigned, low);
}

// The helpers' image of a layer, one thread per pair of values: work-group `rank` has quarter rank % 4 of K and units 80 (rank / 4)
// .., a wave three tiles of four units, or two and zeros.
__global__ void __launch_bounds__(256) pack_helpers_kernel(unsigned *__restrict__ dst, const float *__restrict__ w, int H, const float *__restrict__ scale, int cls, int ts)
{
    const int hb = res_help_blocks(cls), nreg = res_help_regs(cls), pairs = nreg / 2;
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= ts * kResWaves * pairs * 64) return;
    const int lane = idx & 63, i = (idx >> 6) & 3, rest = (idx >> 6) % pairs >> 2, at = (idx >> 6) / pairs;
    const int t = rest % 3, kb = rest / 3, wave = at % kResWaves, rank = at / kResWaves;
    const int tile = wave < 4 ? wave * 3 + t : wave * 2 + 4 + t, unit = (rank >> 2) * 80 + tile * 4 + ((lane & 15) >> 2);
    const int k = ((rank & 3) * hb + kb) * 32 + (lane >> 4) * 8 + 2 * i;
    const int row = unit < H && (wave < 4 || t < 2) ? (lane & 3) * H + unit : -1;
    h2 high = {}, low = {};
    if (row >= 0)
        for (int e = 0; e < 2; ++e) {
            const float a = k + e < H ? w[(long long)row * H + k + e] * scale[row] : 0.f;
            high[e] = (_Float16)a;
            low[e] = (_Float16)(a - (float)high[e]);
        }
    unsigned *to = dst + (long long)at * nreg * 64;
    to[res_place(nreg, (kb * 3 + t) * 8 + i, lane)] = __builtin_bit_cast(unsigned, high);
    to[res_place(nreg, (kb * 3 + t) * 8 + 4 + i, lane)] = __builtin_bit_cast(unsigned, low);
}

// out[i] = 2^-down / scale of the row that entry i is: i, or (gates) gate i % 4 of unit i / 4
__global__ void inverse_scales_kernel(const float *__restrict__ scale, float *__restrict__ out, int n, int gates, int down)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = scale ? ldexpf(1.f / scale[gates ? (i & 3) * (n >> 2) + (i >> 2) : i], -down) : 1.f;
}

// rows `first` .. of the output matrix, scaled or rounded to bf16, padded to `width` values
__global__ void pack_tail_kernel(const float *__restrict__ w, const float *__restrict__ scale, float *__restrict__ out, int first, int J, int width, int n, bool whole)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n * width) return;
    const int row = first + i / width, k = i % width;
    const float v = k < J ? w[(long long)row * J + k] : 0.f;
    out[i] = scale ? v * scale[row] : whole ? v : __uint_as_float(bf16_of(v) << 16);
}

// W_enc as EncWeights::parts: one thread per tile of 32 columns, 16 k's and lane
__global__ void __launch_bounds__(256) pack_projection_kernel(const float *__restrict__ w, int F, int J, int tiles, const float *__restrict__ scale, unsigned *__restrict__ parts)
{
    const int nks = F / 16, lane = threadIdx.x & 63;
    const long long at = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (at >= (long long)tiles * nks) return;
    const int ks = (int)(at % nks), col = (int)(at / nks) * 32 + (lane & 31);
    const int planes = scale ? 2 : 1;
    unsigned *to = parts + (at * planes * 64 + lane) * 4;
    for (int i = 0; i < 4; ++i) {
        float v[2] = {0.f, 0.f};
        if (col < J)
            for (int e = 0; e < 2; ++e) v[e] = w[(long long)col * F + ks * 16 + (lane >> 5) * 8 + i * 2 + e];
        if (!scale) {
            to[i] = bf16_of(v[0]) | bf16_of(v[1]) << 16;
            continue;
        }
        const float s = col < J ? scale[col] : 0.f;
        h2 high, low;
        for (int e = 0; e < 2; ++e) {
            const float a = v[e] * s;
            high[e] = (_Float16)a;
            low[e] = (_Float16)(a - (float)high[e]);
        }
        to[i] = __builtin_bit_cast(unsigned, high);
        to[64 * 4 + i] = __builtin_bit_cast(unsigned, low);
    }
}

}  // namespace

hipError_t pack_projection(const float *w, int F, int J, bool bf16, unsigned *parts, float *inverse, unsigned *check, float *scratch, hipStream_t stream)
{
    const int tiles = enc_columns(J) / 32;
    if (!bf16) {
        hipLaunchKernelGGL(row_scales_kernel, dim3((unsigned)((J + 3) / 4)), dim3(256), 0, stream, w, J, F, scratch, nullptr, check);
        hipLaunchKernelGGL(inverse_scales_kernel, dim3((unsigned)((J + 255) / 256)), dim3(256), 0, stream, scratch, inverse, J, 0, 0);
    }
    hipLaunchKernelGGL(pack_projection_kernel, dim3((unsigned)(((long long)tiles * (F / 16) + 3) / 4)), dim3(256), 0, stream, w, F, J, tiles, bf16 ? nullptr : scratch, parts);
    return hipGetLastError();
}

hipError_t pack_resident(const ResidentPlan &pl, const ResidentWeights &rw, const ResidentImages &im, hipStream_t stream)
{
    const int H = rw.H, J = rw.J, nout = pl.nout_m + pl.n_tail, ts = res_team(pl.cls);
    const bool bf = pl.bf != 0, whole = res_whole(bf, pl.cls);
    const int main_regs = res_main_regs(pl.kind, bf, pl.cls), lstm = res_lstm_regs(bf, pl.cls);
    // row scales: outputs, projection columns, the second layer's input matrix, the recurrent ones
    float *s_out = nullptr, *s_pred = nullptr, *s_ih = nullptr, *s_hh[2] = {nullptr, nullptr};
    auto blocks = [](long long n) { return dim3((unsigned)((n + 255) / 256)); };
    if (!bf) {
        s_out = im.row_scales; s_pred = s_out + nout; s_ih = s_pred + J; s_hh[0] = s_ih + (rw.L > 1 ? 4 * H : 0); s_hh[1] = s_hh[0] + 4 * H;
        auto rows = [&](const float *w, int n, int K, float *s, const float *extra) {
            hipLaunchKernelGGL(row_scales_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, stream, w, n, K, s, extra, im.check);
        };
        if (whole) s_out = nullptr;
        else rows(rw.w_out, nout, J, s_out, nullptr);
        rows(rw.w_pred, J, H, s_pred, rw.b_pred);
        if (rw.L > 1) rows(rw.w_ih1, 4 * H, H, s_ih, nullptr);
        for (int l = 0; l < rw.L; ++l) rows(rw.w_hh[l], 4 * H, H, s_hh[l], nullptr);
    }
    auto tiles = [&](float *dst, int nreg, int first, const float *w, int K, const float *s, Rows r, int T, bool whole) {
        const long long n = (long long)ts * kResWaves * T * res_halves(pl.cls) * 2 * 64;
        hipLaunchKernelGGL(pack_tiles_kernel, blocks(n), dim3(256), 0, stream, reinterpret_cast<unsigned *>(dst), nreg, first, w, K, s, r, T, pl.cls, ts, whole);
    };
    const Rows gates{1, 0, H, pl.units};
    int at = 0;
    if (pl.kind != kResident2Pair)
        for (int l = 0; l < rw.L; ++l, at += lstm) tiles(im.w, main_regs, at, rw.w_hh[l], H, s_hh[l], gates, 5, false);
    if (rw.L > 1) { tiles(im.w, main_regs, at, rw.w_ih1, H, s_ih, gates, 5, false); at += lstm; }
    tiles(im.w, main_regs, at, rw.w_pred, H, s_pred, Rows{0, 0, J, pl.jgroups * 4}, 2, false);
    at += res_pred_regs(bf, pl.cls);
    tiles(im.w, main_regs, at, rw.w_out, J, s_out, Rows{0, 0, pl.nout_m, 32}, 2, whole);
    if (pl.kind == kResident2Pair)
        for (int l = 0; l < 2; ++l) {
            const long long regs = (long long)ts * kResWaves * res_help_regs(pl.cls), n = regs / 2 * 64;
            hipLaunchKernelGGL(pack_helpers_kernel, blocks(n), dim3(256), 0, stream, reinterpret_cast<unsigned *>(im.w_help) + l * regs * 64, rw.w_hh[l], H, s_hh[l], pl.cls, ts);
        }
    auto inverse = [&](const float *s, float *out, int n, int g, int down) {
        hipLaunchKernelGGL(inverse_scales_kernel, blocks(n), dim3(256), 0, stream, s, out, n, g, bf ? 0 : down);
    };
    inverse(s_out, im.s_out, nout, 0, 0);
    inverse(s_pred, im.s_pred, J, 0, kResHiddenExp);
    if (rw.L > 1) inverse(s_ih, im.s_ih, 4 * H, 1, kResHiddenExp);
    for (int l = 0; l < rw.L; ++l) inverse(s_hh[l], im.s_hh[l], 4 * H, 1, kResHiddenExp);
    if (pl.n_tail)
        hipLaunchKernelGGL(pack_tail_kernel, blocks((long long)pl.n_tail * res_row(pl.cls)), dim3(256), 0, stream, rw.w_out, s_out, im.w_tail, pl.nout_m, J, res_row(pl.cls), pl.n_tail, whole);
    return hipGetLastError();
}

}  // namespace rnnt
