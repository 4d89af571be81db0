// fp32 expert FFN (Appendix D, Eq. 10) over the real slots: the two grouped GEMMs of zeda_ffn.hip for fp32 layers.
//   gate/up:  act[r, i]  = silu(<x[tok(r)], W_gate[e][i]>) * <x[tok(r)], W_up[e][i]>
//   down:     y_slot[r,h] = <act[r], W_down[e][h]>
// A workgroup owns up to 32 rows of one expert and NA blocks of 16 weight rows (gate and up blocks alternate); its four waves
// split the reduction dimension, and their sums meet in LDS in wave order.  Any H and I that are multiples of 4.
// Bound by memory on paper (513 tokens, H=1024, I=512, 32 experts: 134 MB of gate/up weights); measured 60 us for gate/up and
// 34 us for down, 40 % of the HBM rate: fp32 products (20 us of matrix time), 64-byte row pieces and two waves per SIMD share
// the rest.  One workgroup per row, which re-read an expert's weights for every row, took 658 and 627 us.
#include "zeda_f32_tile.h"
#include "zeda_place.h"

namespace zeda {

constexpr int kF32Threads = 256;
constexpr int kF32Waves = kF32Threads / 64;
constexpr int kF32Rows = 32;  // token rows per workgroup: two blocks of 16
constexpr int kF32NB = kF32Rows / 16;
constexpr int kF32GridTiles = 1 << 14;  // token tiles along grid x (at most 512 feature tiles of 256 threads each: 2^31 work items), more along y

// this wave's slice of the sums of the first LIVE token blocks, left in part[2 (a * NB + b)][lane] and the row after it
template <int NA, int NB, int LIVE>
__device__ __forceinline__ void multiply_rows(f64x2 (*part)[64], const float *const (&pa)[NA], const float *const (&pb)[NB], int wave, int Kd)
{
    const int lane = threadIdx.x & 63;
    const float *p[LIVE];
#pragma unroll
    for (int b = 0; b < LIVE; ++b) p[b] = pb[b];
    F32Tile<NA, LIVE> t;
    t.run(pa, p, wave, kF32Waves, (int)blockIdx.x * 3, Kd);
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < LIVE; ++b) {
            part[2 * (a * NB + b)][lane] = t.acc[a][b][0];
            part[2 * (a * NB + b) + 1][lane] = t.acc[a][b][1];
        }
}

// GATEUP: tok = x[T,Kd], w0 = W_gate[N,F,Kd], w1 = W_up, out = act[S,F];  else tok = act[S,Kd], w0 = W_down[N,F,Kd],
// out = y_slot[S,F].  n_ft feature tiles per token tile; blocks past the last token tile return at once.
template <bool GATEUP, int NA>
__global__ __launch_bounds__(kF32Threads, 2) void ffn_f32_kernel(const float *__restrict__ tok, const float *__restrict__ w0,
                                                              const float *__restrict__ w1, const int32_t *__restrict__ offsets,
                                                              const int32_t *__restrict__ sorted_slot, float *__restrict__ out,
                                                              int N, int K, int Kd, int F, int n_ft, int T)
{
    constexpr int NB = kF32NB;
    constexpr int NO = (GATEUP ? NA / 2 : NA) * NB;  // output blocks
    __shared__ f64x2 s_part[kF32Waves][NA * NB * 2][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15;
    const int tile_x = blockIdx.x / n_ft, ft = blockIdx.x - tile_x * n_ft, tile = blockIdx.y * kF32GridTiles + tile_x;
    const int4 loc = locate_rows<kF32Rows>(offsets, N, tile);
    const int rows = loc.z;
    if (rows == 0) return;
    const int f0 = ft * 16 * (GATEUP ? NA / 2 : NA);

    const float *pa[NA], *pb[NB];
#pragma unroll
    for (int a = 0; a < NA; ++a) {
        const int f = min(f0 + 16 * (GATEUP ? a / 2 : a) + l16, F - 1);  // rows past F repeat the last one (never stored)
        pa[a] = ((GATEUP && (a & 1)) ? w1 : w0) + ((size_t)loc.x * F + f) * Kd;
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int r = loc.y + min(16 * b + l16, rows - 1);
        pb[b] = tok + (size_t)(GATEUP ? min(max(sorted_slot[r] / K, 0), T - 1) : r) * Kd;  // a bad index must not fault
    }
    // only the blocks that hold rows are fetched and multiplied
    if (rows > 16) multiply_rows<NA, NB, NB>(s_part[wave], pa, pb, wave, Kd);
    else multiply_rows<NA, NB, 1>(s_part[wave], pa, pb, wave, Kd);
    __syncthreads();

    // block (a, b): lane l holds features 4 (l / 16) .. + 3 of token l % 16
    for (int o = wave; o < NO; o += kF32Waves) {
        const int fb = o / NB, b = o - fb * NB, r = 16 * b + l16, f = f0 + 16 * fb + 4 * (lane >> 4);
        if (r >= rows || f >= F) continue;
        auto total = [&](int blk) {  // the waves' sums, in wave order, rounded once
            f32x4 r;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                double v = 0.0;
#pragma unroll
                for (int w = 0; w < kF32Waves; ++w) v += s_part[w][2 * blk + (k >> 1)][lane][k & 1];
                r[k] = (float)v;
            }
            return r;
        };
        f32x4 v;
        if (GATEUP) {
            const f32x4 g = total(2 * fb * NB + b), u = total((2 * fb + 1) * NB + b);
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = g[k] / (1.f + expf(-g[k])) * u[k];
        } else {
            v = total(fb * NB + b);
        }
        *reinterpret_cast<f32x4 *>(out + (size_t)(loc.y + r) * F + f) = v;
    }
}

template <bool GATEUP, int NA>
static int launch(const zeda_layer_desc *d, const float *tok, const float *w0, const float *w1, const int32_t *offsets,
                  const int32_t *sorted_slot, float *out, hipStream_t s)
{
    const int Kd = GATEUP ? d->H : d->I, F = GATEUP ? d->I : d->H;
    const int n_ft = ceil_div(F, 16 * (GATEUP ? NA / 2 : NA));
    const int S = d->T * d->K, tiles = (S < d->N ? S : d->N) + S / kF32Rows;  // at most this many token tiles
    const dim3 grid((unsigned)(tiles < kF32GridTiles ? tiles : kF32GridTiles) * n_ft, ceil_div(tiles, kF32GridTiles));
    ffn_f32_kernel<GATEUP, NA><<<grid, kF32Threads, 0, s>>>(tok, w0, w1, offsets, sorted_slot, out, d->N, d->K, Kd,
                                                                              F, n_ft, d->T);
    return last_launch_status();
}

// Four weight blocks per workgroup halve the token reads per weight byte; two make twice the workgroups, for layers whose
// experts are too few and too narrow to fill the device otherwise.
template <bool GATEUP>
static int launch_any(const zeda_layer_desc *d, const void *tok, const void *w0, const void *w1, const int32_t *offsets,
                      const int32_t *sorted_slot, void *out, hipStream_t s)
{
    const int F = GATEUP ? 2 * d->I : d->H;
    const bool wide = (int64_t)d->N * F >= 256 * 64;
    return wide ? launch<GATEUP, 4>(d, (const float *)tok, (const float *)w0, (const float *)w1, offsets, sorted_slot, (float *)out, s)
                : launch<GATEUP, 2>(d, (const float *)tok, (const float *)w0, (const float *)w1, offsets, sorted_slot, (float *)out, s);
}

int launch_gateup_f32(const zeda_layer_desc *d, const void *x, const void *wg, const void *wu, const int32_t *offsets,
                      const int32_t *sorted_slot, void *act, hipStream_t s)
{
    return launch_any<true>(d, x, wg, wu, offsets, sorted_slot, act, s);
}

int launch_down_f32(const zeda_layer_desc *d, const void *act, const void *wd, const int32_t *offsets, void *y_slot, hipStream_t s)
{
    return launch_any<false>(d, act, wd, nullptr, offsets, nullptr, y_slot, s);
}

}  // namespace zeda
