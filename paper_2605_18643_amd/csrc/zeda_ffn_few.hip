// Expert FFN of small bf16 batches and small models (Appendix D, Eq. 10): the two grouped GEMMs of zeda_ffn.hip where the
// experts have a handful of rows each, so that nothing but the streaming of their weights counts, or where there are too
// few weight tiles to give every CU one.
//
// The tile kernel gives a workgroup 128 or 256 weight rows and all of the reduction dimension: one decoded token (8 slots,
// half of them real) makes 48 workgroups of 512 KiB each for gate/up on a chip with 256 CUs.  Here a workgroup owns NF
// blocks of 16 weight rows (of gate and of up) and up to 16 NB token rows, its four waves split the reduction dimension,
// and the weights go from memory straight into the registers that the 16x16x32 MFMA reads: a lane's operand is 16 bytes of
// one row, a tiled 32x32 unit is two such fragments of one contiguous KiB each.  No LDS and no barrier until the waves' sums
// meet; a wave keeps DEPTH chunks of 64 k in flight.  Bound by HBM: 64 tokens, 106 experts hit, 667 MB of gate/up weights
// in 107 us = 6.2 TB/s; one token, gate/up and down 23 + 13 -> 11 + 8 us (launch included).
#include "zeda_internal.h"

namespace zeda {

constexpr int kFewThreads = 256;
constexpr int kFewWaves = kFewThreads / 64;

// (expert, first row, rows) of token tile `tile`, or rows = 0 past the last one: lane l holds experts 4l..4l+3
template <int ROWS>
__device__ __forceinline__ int3 few_locate(const int32_t *__restrict__ offsets, int N, int tile)
{
    const int lane = threadIdx.x & 63;
    int off[5], nt[4], local = 0;
#pragma unroll
    for (int q = 0; q < 5; ++q) off[q] = offsets[min(4 * lane + q, N)];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        nt[q] = (off[q + 1] - off[q] + ROWS - 1) / ROWS;
        local += nt[q];
    }
    int incl = local;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
    int excl = incl - local, e = 0, row0 = 0, rows = 0;
    const unsigned long long mine = __ballot(tile >= excl && tile < incl);
    if (mine == 0) return make_int3(0, 0, 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (tile >= excl && tile < excl + nt[q]) {
            e = 4 * lane + q;
            row0 = off[q] + (tile - excl) * ROWS;
            rows = min(ROWS, off[q + 1] - row0);
        }
        excl += nt[q];
    }
    const int src = __ffsll((long long)mine) - 1;
    return make_int3(__builtin_amdgcn_readlane(e, src), __builtin_amdgcn_readlane(row0, src), __builtin_amdgcn_readlane(rows, src));
}

// this wave's share of the reduction for the first LIVE token blocks: part[a * NB + b][lane] of part
template <bool TILED, int NA, int NB, int LIVE, int DEPTH>
__device__ __forceinline__ void few_multiply(f32x4 (*part)[64], const bf16_t *const (&pa)[NA], const bf16_t *const (&pt)[NB], size_t wstep,
                                             int wave, int start, int Kd)
{
    const int lane = threadIdx.x & 63;
    f32x4 acc[NA][LIVE];
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < LIVE; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    // this wave's chunks of 64 k: wave, wave + 4, ..., from one that depends on `start` on
    const int n = (Kd / 64 - wave + kFewWaves - 1) / kFewWaves;
    int next = n > 0 ? (int)((unsigned)start % (unsigned)n) : 0;
    bf16x8 fa[DEPTH][2][NA], fb[DEPTH][2][LIVE];
    auto load = [&](int d) {
        const int kb = 2 * (wave + kFewWaves * next);
        next = next + 1 == n ? 0 : next + 1;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int a = 0; a < NA; ++a) fa[d][s][a] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8 *>(pa[a] + (kb + s) * wstep));
#pragma unroll
            for (int b = 0; b < LIVE; ++b) fb[d][s][b] = *reinterpret_cast<const bf16x8 *>(pt[b] + (kb + s) * 32);
        }
    };
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        if (d < n) load(d);
    for (int i = 0; i < n; i += DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            if (i + d < n) {
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int a = 0; a < NA; ++a)
#pragma unroll
                        for (int b = 0; b < LIVE; ++b)
                            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[d][s][a], fb[d][s][b], acc[a][b], 0, 0, 0);
                if (i + d + DEPTH < n) load(d);
            }
        }
    }
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < LIVE; ++b) part[a * NB + b][lane] = acc[a][b];
}

// GATEUP: tok = x[T,Kd], w0 = W_gate[N,F,Kd], w1 = W_up, out = act[S,F];  else tok = act[S,Kd], w0 = W_down[N,F,Kd],
// out = y_slot[S,F].  Kd a multiple of 64, F of 16 NF.  Up to 16 NB token rows.  Blocks past the last token tile return
// at once.
template <bool GATEUP, bool TILED, int NF, int NB, int DEPTH>
__global__ __launch_bounds__(kFewThreads) void ffn_few_kernel(const bf16_t *__restrict__ tok, const bf16_t *__restrict__ w0,
                                                              const bf16_t *__restrict__ w1, const int32_t *__restrict__ offsets,
                                                              const int32_t *__restrict__ sorted_slot, bf16_t *__restrict__ out,
                                                              int N, int K, int Kd, int F, int n_ft, int T)
{
    constexpr int NA = GATEUP ? 2 * NF : NF;  // weight blocks: gate and up blocks alternate
    __shared__ f32x4 s_part[kFewWaves][NA * NB][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, kq = lane >> 4;
    const int tile = blockIdx.x / n_ft, ft = blockIdx.x - tile * n_ft;
    const int3 loc = few_locate<16 * NB>(offsets, N, tile);
    if (loc.z == 0) return;
    const bf16_t *pt[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int r = loc.y + min(16 * b + l16, loc.z - 1);  // columns past the tile repeat its last row (never stored)
        pt[b] = tok + (size_t)(GATEUP ? min(max(sorted_slot[r] / K, 0), T - 1) : r) * Kd + kq * 8;  // a bad index must not fault
    }
    const bf16_t *pa[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) {
        const int f = (ft * NF + (GATEUP ? a / 2 : a)) * 16;
        const bf16_t *w = ((GATEUP && (a & 1)) ? w1 : w0) + (size_t)loc.x * F * Kd;
        const int row = (f & 31) + l16;  // of the stored unit
        pa[a] = TILED ? w + (size_t)(f >> 5) * 1024 + row * 32 + (kq ^ ((row >> 2) & 3)) * 8 : w + (size_t)(f + l16) * Kd + kq * 8;
    }
    const size_t wstep = TILED ? (size_t)F * 32 : 32;  // elements from one 32-wide k block to the next
    // An expert starts at a chunk of its own, so that not all workgroups stream the same columns: with few rows per expert
    // the same chunk of row-major rows, often a multiple of 4 KiB apart, sits on a few memory channels.  All feature tiles
    // of an expert start alike: neighbours then read neighbouring units of tiled weights at the same time.
    const int start = loc.x * 5;
    static_assert(NB == 2, "one or two live blocks");
    if (loc.z > 16) few_multiply<TILED, NA, NB, NB, DEPTH>(s_part[wave], pa, pt, wstep, wave, start, Kd);
    else few_multiply<TILED, NA, NB, 1, DEPTH>(s_part[wave], pa, pt, wstep, wave, start, Kd);
    __syncthreads();

    // a block's lane l holds features 4 (l / 16) .. + 3 of token l % 16
    for (int o = wave; o < NF * NB; o += kFewWaves) {
        const int fb = o / NB, b = o - fb * NB, r = 16 * b + l16;
        if (r >= loc.z) continue;
        auto total = [&](int a) {
            f32x4 v = s_part[0][a * NB + b][lane];
#pragma unroll
            for (int w = 1; w < kFewWaves; ++w) v += s_part[w][a * NB + b][lane];
            return v;
        };
        bf16x4 v;
        if (GATEUP) {
            const f32x4 g = total(2 * fb), u = total(2 * fb + 1);
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = (bf16_t)(g[k] * __builtin_amdgcn_rcpf(1.f + __expf(-g[k])) * u[k]);
        } else {
            const f32x4 y = total(fb);
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = (bf16_t)y[k];
        }
        *reinterpret_cast<bf16x4 *>(out + (size_t)(loc.y + r) * F + (ft * NF + fb) * 16 + 4 * kq) = v;
    }
}

// Where this kernel beats the tile kernel, by the rows an expert gets if the slots fall evenly on all N + Z experts (the
// real loads are only known on the device) and by the tile kernel's gate/up work items, one per 128 columns of I and expert:
//  - up to 5 rows both stream weights and nothing else; this one has more of them in flight (N=128, I=768, H=2048:
//    64 tokens 188 -> 177 us, row-major at 32 tokens 191 -> 168; level at 128 tokens, 3 % behind at 192);
//  - up to 64 tokens it also wins with more rows (N=8, K=2, I=3072: 75 -> 67 us; N=8, K=6, I=1024: 39 -> 38);
//  - up to 320 items the tile kernel fills little more than one round of 256 CUs or less (N=48, I=768, H=1536: 100 tokens
//    92 -> 73 us, 300 tokens row-major 138 -> 115; N=24, I=448, H=1152: 301 tokens 45 -> 40).  This kernel reads the token
//    rows once per 16 columns, so it falls behind once an expert has more rows than a workgroup: at 94 rows 49 -> 75 us;
//  - up to 40 items there is next to nothing to fill the chip with (N=16, I=256, H=512: 500 tokens 38 -> 23 us, 2000 tokens,
//    167 rows, 39 -> 30; level at 250 rows with N=32, I=128).
bool ffn_few_supported(const zeda_layer_desc *d)
{
    const int64_t slots = (int64_t)d->T * d->K, experts = d->N + d->Z, items = (int64_t)d->N * ceil_div(d->I, 128);
    return d->T <= 64 || slots <= 5 * experts || (items <= 320 && slots <= 40 * experts) || (items <= 40 && slots <= 170 * experts);
}

template <bool GATEUP, bool TILED>
static int launch(const zeda_layer_desc *d, const void *tok, const void *w0, const void *w1, const int32_t *offsets,
                  const int32_t *sorted_slot, void *out, hipStream_t s)
{
    // 16 gate and 16 up rows, or 32 rows of W_down (16 make twice the workgroups and token reads: 58 -> 61 us at 64 tokens);
    // two token blocks; three chunks of 64 k in flight (four leave fewer waves per SIMD: 177.5 -> 176.5 us)
    constexpr int NF = GATEUP ? 1 : 2, NB = 2, DEPTH = 3;
    const int Kd = GATEUP ? d->H : d->I, F = GATEUP ? d->I : d->H, n_ft = F / (16 * NF);
    const int S = d->T * d->K, tiles = (S < d->N ? S : d->N) + S / (16 * NB);  // at most this many token tiles
    ffn_few_kernel<GATEUP, TILED, NF, NB, DEPTH><<<(unsigned)tiles * n_ft, kFewThreads, 0, s>>>(
        (const bf16_t *)tok, (const bf16_t *)w0, (const bf16_t *)w1, offsets, sorted_slot, (bf16_t *)out, d->N, d->K, Kd, F, n_ft, d->T);
    return last_launch_status();
}

int launch_gateup_few(const zeda_layer_desc *d, const void *x, const void *wg, const void *wu, const int32_t *offsets,
                      const int32_t *sorted_slot, void *act, hipStream_t s)
{
    return d->weight_layout == ZEDA_WEIGHTS_TILED ? launch<true, true>(d, x, wg, wu, offsets, sorted_slot, act, s)
                                                  : launch<true, false>(d, x, wg, wu, offsets, sorted_slot, act, s);
}

int launch_down_few(const zeda_layer_desc *d, const void *act, const void *wd, const int32_t *offsets, void *y_slot, hipStream_t s)
{
    return d->weight_layout == ZEDA_WEIGHTS_TILED ? launch<false, true>(d, act, wd, nullptr, offsets, nullptr, y_slot, s)
                                                  : launch<false, false>(d, act, wd, nullptr, offsets, nullptr, y_slot, s);
}

}  // namespace zeda
