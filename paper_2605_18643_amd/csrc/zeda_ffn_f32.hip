// fp32 expert FFN (Appendix D, Eq. 10) over the real slots: the two grouped GEMMs of zeda_ffn.hip for fp32 layers.
//   gate/up:  act[r, i]  = silu(<x[tok(r)], W_gate[e][i]>) * <x[tok(r)], W_up[e][i]>
//   down:     y_slot[r,h] = <act[r], W_down[e][h]>
// A workgroup owns up to 32 rows of one expert and NA blocks of 16 weight rows (gate and up blocks alternate); its four waves
// split the reduction dimension, and their sums meet in LDS in wave order.  Any H and I that are multiples of 4.
// What bounds it: splitting the operands and adding up the chunks on the vector unit, then the weights (513 tokens, H=1024,
// I=512, 32 experts: 134 MB of gate/up weights).  There gate/up takes 48 us and down 27; with the fp32 matrix instruction and
// operands loaded straight into its registers 60 and 35.  Three workgroups per CU: with 48 and 64 rows a workgroup (two per CU) the
// last round is nearly empty or registers spill (53 + 31 and 41 + 26 us).
#include "zeda_f32_split.h"
#include "zeda_f32_tile.h"
#include "zeda_place.h"

namespace zeda {

constexpr int kF32Threads = 256;
constexpr int kF32Waves = kF32Threads / 64;
constexpr int kF32Rows = 32;  // token rows per workgroup: two blocks of 16
constexpr int kF32NB = kF32Rows / 16;
constexpr int kF32GridTiles = 1 << 14;  // token tiles along grid x (at most 512 feature tiles of 256 threads each: 2^31 work items), more along y

// where token tile `tile` is; PLACE: found from the ids of all slots, whose tables the first feature tiles write
template <bool PLACE>
__device__ __forceinline__ int4 locate_f32(const int32_t *offsets, int N, int K, int T, int tile, int ft, TilePlaceLds<PLACE ? kF32Rows : 1> &s, const TilePlace &tp)
{
    static_assert(kF32Threads == kTileThreads, "");
    if constexpr (PLACE) return place_tile<kF32Rows>([&](int slot) { return tp.ids[slot]; }, T * K, N, tile, ft == 0, tile == 0 && ft == 0, s, tp.out);
    else return locate_rows<kF32Rows>(offsets, N, tile);
}

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
// PLACE: the workgroup places the slots itself, from their ids (tp).
template <bool GATEUP, int NA, bool PLACE>
__global__ __launch_bounds__(kF32Threads, 2) void ffn_f32_kernel(const float *__restrict__ tok, const float *__restrict__ w0,
                                                              const float *__restrict__ w1, const int32_t *__restrict__ offsets,
                                                              const int32_t *__restrict__ sorted_slot, float *__restrict__ out,
                                                              int N, int K, int Kd, int F, int n_ft, int T, TilePlace tp)
{
    constexpr int NB = kF32NB;
    constexpr int NO = (GATEUP ? NA / 2 : NA) * NB;  // output blocks
    __shared__ f64x2 s_part[kF32Waves][NA * NB * 2][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15;
    const int tile_x = blockIdx.x / n_ft, ft = blockIdx.x - tile_x * n_ft, tile = blockIdx.y * kF32GridTiles + tile_x;
    __shared__ TilePlaceLds<PLACE ? kF32Rows : 1> s_place;
    const int4 loc = locate_f32<PLACE>(offsets, N, K, T, tile, ft, s_place, tp);
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
        const int row = min(16 * b + l16, rows - 1), slot = PLACE ? s_place.list[row] : GATEUP ? sorted_slot[loc.y + row] : 0;
        pb[b] = tok + (size_t)(GATEUP ? min(max(slot / K, 0), T - 1) : loc.y + row) * Kd;  // a bad index must not fault
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

constexpr int kF32Slots = 6;            // ring blocks a wave keeps in flight

// GATEUP: tok = x[T,Kd], w0 = W_gate[N,F,Kd], w1 = W_up, out = act[S,F];  else tok = act[S,Kd], w0 = W_down[N,F,Kd],
// out = y_slot[S,F].  n_ft feature tiles per token tile of up to 16 NB rows; blocks past the last token tile return at once.
template <bool GATEUP, int NA, int NB>
struct F32Ffn {
    static constexpr int NF = GATEUP ? NA / 2 : NA;  // feature blocks: gate and up blocks alternate
    static constexpr int RING = WaveRing<kF32Slots>::BYTES;
    static constexpr int PART = NA * 2 * 64 * (int)sizeof(f64x2);  // a wave's sums of one token block
    static constexpr int LDS_BYTES = kF32Waves * (RING > PART ? RING : PART);  // the rings, then the waves' sums
    typedef f64x2 (*Part)[NA * 2][64];

    // the tile's rows are out's rows first .. first + rows - 1, in LIVE blocks of 16; features f0 ..; tok_row(r): row r's token values
    template <int LIVE, typename TokRow>
    __device__ __forceinline__ static void run(unsigned char *lds, const float *w0, const float *w1, const uint32_t (&wo)[NA][2],
                                               const float *const (&pb)[NB][2], int Kd, float *__restrict__ out, int first, int rows, int f0, int F,
                                               const TokRow &tok_row)
    {
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15;
        const float *p[LIVE][2];
#pragma unroll
        for (int b = 0; b < LIVE; ++b) { p[b][0] = pb[b][0]; p[b][1] = pb[b][1]; }
        F32Split<NA, LIVE, kF32Slots> t;
        t.run(lds_addr(lds) + wave * RING, w0, w1, wo, p, wave, kF32Waves, (int)blockIdx.x * 3, Kd);
        Part part = reinterpret_cast<Part>(lds);
#pragma unroll
        for (int b = 0; b < LIVE; ++b) {
            __syncthreads();  // everyone is done with the rings, and with the sums of the block before
#pragma unroll
            for (int a = 0; a < NA; ++a) {
                part[wave][2 * a][lane] = t.acc[a][b][0];
                part[wave][2 * a + 1][lane] = t.acc[a][b][1];
            }
            const uint32_t odd_tok = (t.odd_tok >> (16 * b)) & 0xffffu;
            if (odd_tok || t.odd_w) multiply_odd(part[wave], odd_tok, t.odd_w, w0, w1, tok_row(min(16 * b + l16, rows - 1)), f0, F, wave, Kd);
            __syncthreads();
            // block (a, b): lane l holds features 4 (l / 16) .. + 3 of token l % 16
            const int r = 16 * b + l16;
            for (int fb = wave; fb < NF; fb += kF32Waves) {
                const int f = f0 + 16 * fb + 4 * (lane >> 4);
                if (r >= rows || f >= F) continue;
                auto total = [&](int a) {  // the waves' sums, in wave order, rounded once
                    f32x4 v;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        double sum = 0.0;
#pragma unroll
                        for (int w = 0; w < kF32Waves; ++w) sum += part[w][2 * a + (k >> 1)][lane][k & 1];
                        v[k] = (float)sum;
                    }
                    return v;
                };
                f32x4 v;
                if (GATEUP) {
                    const f32x4 g = total(2 * fb), u = total(2 * fb + 1);
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[k] = swiglu(g[k], u[k]);
                } else {
                    v = total(fb);
                }
                *reinterpret_cast<f32x4 *>(out + (size_t)(first + r) * F + f) = v;
            }
        }
    }
    // What rows outside the split's window contribute to one token block (row l % 16 of it: tok), in this wave's slice of the
    // reduction: their sums on the fp32 instruction take the place of the split's.  Ordinary pairs of rows keep theirs, so a
    // token's result does not depend on its neighbours.
    __device__ __forceinline__ static void multiply_odd(f64x2 (*part)[64], uint32_t odd_tok, uint64_t odd_w, const float *w0, const float *w1,
                                                        const float *tok, int f0, int F, int wave, int Kd)
    {
        const int lane = threadIdx.x & 63, l16 = lane & 15;
        static_assert(NA % 2 == 0, "two weight blocks at a time");
#pragma unroll 1
        for (int a0 = 0; a0 < NA; a0 += 2) {
            const uint32_t ow = (uint32_t)(odd_w >> (16 * a0));
            if (!(odd_tok | ow)) continue;
            const float *pa[2], *pb[1] = {tok};
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int f = min(f0 + 16 * (GATEUP ? a0 / 2 : a0 + i) + l16, F - 1);
                pa[i] = (GATEUP && i ? w1 : w0) + (size_t)f * Kd;
            }
            F32Tile<2, 1> t;
            t.run(pa, pb, wave, kF32Waves, (int)blockIdx.x * 3, Kd);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (((odd_tok >> l16) | (ow >> (16 * i + 4 * (lane >> 4) + k))) & 1)
                        part[2 * (a0 + i) + (k >> 1)][lane][k & 1] = t.acc[i][0][k >> 1][k & 1];
        }
    }
    __device__ __forceinline__ static float swiglu(float g, float u) { return g / (1.f + expf(-g)) * u; }
};

template <bool GATEUP, int NA, int NB, bool PLACE>
__global__ __launch_bounds__(kF32Threads, 3) void ffn_f32_split_kernel(const float *__restrict__ tok, const float *__restrict__ w0,
                                                              const float *__restrict__ w1, const int32_t *__restrict__ offsets,
                                                              const int32_t *__restrict__ sorted_slot, float *__restrict__ out,
                                                              int N, int K, int Kd, int F, int n_ft, int T, TilePlace tp)
{
    typedef F32Ffn<GATEUP, NA, NB> C;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[C::LDS_BYTES];
    const int lane = threadIdx.x & 63, r8 = lane >> 3;
    const int tile_x = blockIdx.x / n_ft, ft = blockIdx.x - tile_x * n_ft, tile = blockIdx.y * kF32GridTiles + tile_x;
    static_assert(16 * NB == kF32Rows, "");
    __shared__ TilePlaceLds<PLACE ? kF32Rows : 1> s_place;
    const int4 loc = locate_f32<PLACE>(offsets, N, K, T, tile, ft, s_place, tp);
    const int rows = loc.z;
    if (rows == 0) return;
    const int f0 = ft * 16 * C::NF;

    auto tok_row = [&](int row) {
        const int slot = PLACE ? s_place.list[row] : GATEUP ? sorted_slot[loc.y + row] : 0;
        return tok + (size_t)(GATEUP ? min(max(slot / K, 0), T - 1) : loc.y + row) * Kd;  // a bad index must not fault
    };
    const float *pb[NB][2];
    uint32_t wo[NA][2];  // (an expert's matrix has 604 MB at most)
    w0 += (size_t)loc.x * F * Kd;
    w1 = GATEUP ? w1 + (size_t)loc.x * F * Kd : w0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int a = 0; a < NA; ++a) {
            const int f = min(f0 + 16 * (GATEUP ? a / 2 : a) + 8 * h + r8, F - 1);  // rows past F repeat the last one (never stored)
            wo[a][h] = (uint32_t)f * Kd * 4;
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) pb[b][h] = tok_row(min(16 * b + 8 * h + r8, rows - 1));
    }
    // only the blocks that hold rows are fetched and multiplied
    if (rows > 16) C::template run<2>(lds, w0, w1, wo, pb, Kd, out, loc.y, rows, f0, F, tok_row);
    else C::template run<1>(lds, w0, w1, wo, pb, Kd, out, loc.y, rows, f0, F, tok_row);
}

// at most this many token tiles
static int f32_tiles(const zeda_layer_desc *d)
{
    const int S = d->T * d->K;
    return (S < d->N ? S : d->N) + S / kF32Rows;
}

// SPLIT: the kernel for many rows per expert
template <bool GATEUP, int NA, bool SPLIT>
static int launch(const zeda_layer_desc *d, const float *tok, const float *w0, const float *w1, const int32_t *offsets,
                  const int32_t *sorted_slot, float *out, const TilePlace *tp, hipStream_t s)
{
    const int Kd = GATEUP ? d->H : d->I, F = GATEUP ? d->I : d->H;
    const int n_ft = ceil_div(F, 16 * (GATEUP ? NA / 2 : NA)), tiles = f32_tiles(d);
    const dim3 grid((unsigned)(tiles < kF32GridTiles ? tiles : kF32GridTiles) * n_ft, ceil_div(tiles, kF32GridTiles));
    auto go = [&](auto *kernel) { kernel<<<grid, kF32Threads, 0, s>>>(tok, w0, w1, offsets, sorted_slot, out, d->N, d->K, Kd, F, n_ft, d->T, tp ? *tp : TilePlace{}); };
    if constexpr (GATEUP) {
        if (tp) {
            if constexpr (SPLIT) go(ffn_f32_split_kernel<GATEUP, NA, kF32NB, true>);
            else go(ffn_f32_kernel<GATEUP, NA, true>);
            return last_launch_status();
        }
    }
    if constexpr (SPLIT) go(ffn_f32_split_kernel<GATEUP, NA, kF32NB, false>);
    else go(ffn_f32_kernel<GATEUP, NA, false>);
    return last_launch_status();
}

// Where the split kernel is the faster one, by the slots per expert of the whole pool (whole layer, its time over the other's):
// H=1024, I=512, N=32, K=4: 4 slots 1.01, 8 0.98, 16 0.91, 32 0.76, 128 0.75; with Z=8: 6.4 1.01, 12.8 0.95, 51 0.86; H=2048, I=1024,
// N=16: 6.4 0.96, 19 0.88, 102 0.74; H=768, N=48: 9 0.96, 27 0.82; H=512, I=512, N=16: 8 0.99, 24 0.93, 128 0.88.  With a row or two per
// expert it is 3 us slower (one more turn through LDS before the first product; H=820, I=360, one token: 30 -> 35 us), as it is
// throughout for layers that are not wide.
static bool f32_many_rows(const zeda_layer_desc *d) { return (int64_t)d->T * d->K >= 8 * ((int64_t)d->N + d->Z); }

// Four weight blocks per workgroup halve the token reads per weight byte; two make twice the workgroups, for layers whose
// experts are too few and too narrow to fill the device otherwise.
static bool f32_wide(const zeda_layer_desc *d, int rows) { return (int64_t)d->N * rows >= 256 * 64; }  // rows: of an expert's weights

int64_t gateup_f32_workgroups(const zeda_layer_desc *d)
{
    return (int64_t)f32_tiles(d) * ceil_div(d->I, f32_wide(d, 2 * d->I) ? 32 : 16);
}

template <bool GATEUP>
static int launch_any(const zeda_layer_desc *d, const void *tok, const void *w0, const void *w1, const int32_t *offsets,
                      const int32_t *sorted_slot, void *out, const TilePlace *tp, hipStream_t s)
{
    const bool wide = f32_wide(d, GATEUP ? 2 * d->I : d->H);
    const float *t = (const float *)tok, *a = (const float *)w0, *b = (const float *)w1;
    if (wide && f32_many_rows(d)) return launch<GATEUP, 4, true>(d, t, a, b, offsets, sorted_slot, (float *)out, tp, s);
    return wide ? launch<GATEUP, 4, false>(d, t, a, b, offsets, sorted_slot, (float *)out, tp, s)
                : launch<GATEUP, 2, false>(d, t, a, b, offsets, sorted_slot, (float *)out, tp, s);
}

int launch_gateup_f32(const zeda_layer_desc *d, const void *x, const void *wg, const void *wu, const int32_t *offsets,
                      const int32_t *sorted_slot, void *act, const TilePlace *tp, hipStream_t s)
{
    return launch_any<true>(d, x, wg, wu, offsets, sorted_slot, act, tp, s);
}

int launch_down_f32(const zeda_layer_desc *d, const void *act, const void *wd, const int32_t *offsets, void *y_slot, hipStream_t s)
{
    return launch_any<false>(d, act, wd, nullptr, offsets, nullptr, y_slot, nullptr, s);
}

}  // namespace zeda
