// Expert FFN of small bf16 batches (Appendix D, Eq. 10): the two grouped GEMMs of zeda_ffn.hip when the experts that were
// hit have a handful of rows each, so that nothing but the streaming of their weights counts and, with few experts hit,
// the number of workgroups that stream.
//
// The tile kernel gives a workgroup 128 weight rows and all of the reduction dimension: one decoded token (8 slots, half
// of them real) makes 48 workgroups of 512 KiB each for gate/up on a chip with 256 CUs.  Here a workgroup owns NF
// blocks of 16 weight rows (of gate and of up) and up to 16 token rows, its four waves split the reduction dimension, and
// the weights go from memory straight into the registers that the 16x16x32 MFMA reads: a lane's operand is 16 bytes of one
// row, a tiled 32x32 unit is two such fragments of one contiguous KiB each.  No LDS and no barrier until the waves' sums
// meet; a wave keeps DEPTH chunks of 64 k in flight.
#include "zeda_internal.h"

namespace zeda {

constexpr int kFewThreads = 256;
constexpr int kFewWaves = kFewThreads / 64;
constexpr int kFewRows = 16;  // token rows per workgroup

// (expert, first row, rows) of token tile `tile`, or rows = 0 past the last one: lane l holds experts 4l..4l+3
__device__ __forceinline__ int3 few_locate(const int32_t *__restrict__ offsets, int N, int tile)
{
    const int lane = threadIdx.x & 63;
    int off[5], nt[4], local = 0;
#pragma unroll
    for (int q = 0; q < 5; ++q) off[q] = offsets[min(4 * lane + q, N)];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        nt[q] = (off[q + 1] - off[q] + kFewRows - 1) / kFewRows;
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
            row0 = off[q] + (tile - excl) * kFewRows;
            rows = min(kFewRows, off[q + 1] - row0);
        }
        excl += nt[q];
    }
    const int src = __ffsll((long long)mine) - 1;
    return make_int3(__builtin_amdgcn_readlane(e, src), __builtin_amdgcn_readlane(row0, src), __builtin_amdgcn_readlane(rows, src));
}

// GATEUP: tok = x[T,Kd], w0 = W_gate[N,F,Kd], w1 = W_up, out = act[S,F];  else tok = act[S,Kd], w0 = W_down[N,F,Kd],
// out = y_slot[S,F].  Kd a multiple of 64, F of 16 NF.  Blocks past the last token tile return at once.
template <bool GATEUP, bool TILED, int NF, int DEPTH>
__global__ __launch_bounds__(kFewThreads) void ffn_few_kernel(const bf16_t *__restrict__ tok, const bf16_t *__restrict__ w0,
                                                              const bf16_t *__restrict__ w1, const int32_t *__restrict__ offsets,
                                                              const int32_t *__restrict__ sorted_slot, bf16_t *__restrict__ out,
                                                              int N, int K, int Kd, int F, int n_ft, int T)
{
    constexpr int NA = GATEUP ? 2 * NF : NF;  // weight blocks: gate and up blocks alternate
    __shared__ f32x4 s_part[kFewWaves][NA][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, kq = lane >> 4;
    const int tile = blockIdx.x / n_ft, ft = blockIdx.x - tile * n_ft;
    const int3 loc = few_locate(offsets, N, tile);
    if (loc.z == 0) return;
    const int r = loc.y + min(l16, loc.z - 1);  // columns past the tile repeat its last row (never stored)
    const bf16_t *pt = tok + (size_t)(GATEUP ? min(max(sorted_slot[r] / K, 0), T - 1) : r) * Kd + kq * 8;  // a bad index must not fault
    const bf16_t *pa[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) {
        const int f = (ft * NF + (GATEUP ? a / 2 : a)) * 16;
        const bf16_t *w = ((GATEUP && (a & 1)) ? w1 : w0) + (size_t)loc.x * F * Kd;
        const int row = (f & 31) + l16;  // of the stored unit
        pa[a] = TILED ? w + (size_t)(f >> 5) * 1024 + row * 32 + (kq ^ ((row >> 2) & 3)) * 8 : w + (size_t)(f + l16) * Kd + kq * 8;
    }
    const size_t wstep = TILED ? (size_t)F * 32 : 32;  // elements from one 32-wide k block to the next

    f32x4 acc[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[a] = f32x4{0.f, 0.f, 0.f, 0.f};
    // This wave's chunks of 64 k: wave, wave + 4, ...; a workgroup starts at a chunk of its own (rows are often a multiple
    // of 4 KiB apart, and the same chunk of every row would then sit on one L2 channel).
    const int n = (Kd / 64 - wave + kFewWaves - 1) / kFewWaves;
    int next = n > 0 ? (int)((unsigned)(loc.x * 5 + ft * 3) % (unsigned)n) : 0;
    bf16x8 fa[DEPTH][2][NA], fb[DEPTH][2];
    auto load = [&](int d) {
        const int kb = 2 * (wave + kFewWaves * next);
        next = next + 1 == n ? 0 : next + 1;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int a = 0; a < NA; ++a) fa[d][s][a] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8 *>(pa[a] + (kb + s) * wstep));
            fb[d][s] = *reinterpret_cast<const bf16x8 *>(pt + (kb + s) * 32);
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
                    for (int a = 0; a < NA; ++a) acc[a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[d][s][a], fb[d][s], acc[a], 0, 0, 0);
                if (i + d + DEPTH < n) load(d);
            }
        }
    }
#pragma unroll
    for (int a = 0; a < NA; ++a) s_part[wave][a][lane] = acc[a];
    __syncthreads();

    // a block's lane l holds features 4 (l / 16) .. + 3 of token l % 16
    for (int o = wave; o < NF; o += kFewWaves) {
        if (l16 >= loc.z) continue;
        auto total = [&](int a) {
            f32x4 v = s_part[0][a][lane];
#pragma unroll
            for (int w = 1; w < kFewWaves; ++w) v += s_part[w][a][lane];
            return v;
        };
        bf16x4 v;
        if (GATEUP) {
            const f32x4 g = total(2 * o), u = total(2 * o + 1);
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = (bf16_t)(g[k] * __builtin_amdgcn_rcpf(1.f + __expf(-g[k])) * u[k]);
        } else {
            const f32x4 y = total(o);
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = (bf16_t)y[k];
        }
        *reinterpret_cast<bf16x4 *>(out + (size_t)(loc.y + l16) * F + (ft * NF + o) * 16 + 4 * kq) = v;
    }
}

#ifndef ZFEW_T
#define ZFEW_T 64
#endif
bool ffn_few_supported(const zeda_layer_desc *d) { return d->T <= ZFEW_T; }

template <bool GATEUP, bool TILED, int NF, int DEPTH>
static int launch(const zeda_layer_desc *d, const void *tok, const void *w0, const void *w1, const int32_t *offsets,
                  const int32_t *sorted_slot, void *out, hipStream_t s)
{
    const int Kd = GATEUP ? d->H : d->I, F = GATEUP ? d->I : d->H, n_ft = F / (16 * NF);
    const int S = d->T * d->K, tiles = (S < d->N ? S : d->N) + S / kFewRows;  // at most this many token tiles
    ffn_few_kernel<GATEUP, TILED, NF, DEPTH><<<(unsigned)tiles * n_ft, kFewThreads, 0, s>>>(
        (const bf16_t *)tok, (const bf16_t *)w0, (const bf16_t *)w1, offsets, sorted_slot, (bf16_t *)out, d->N, d->K, Kd, F, n_ft, d->T);
    return last_launch_status();
}

template <bool GATEUP>
static int launch_any(const zeda_layer_desc *d, const void *tok, const void *w0, const void *w1, const int32_t *offsets,
                      const int32_t *sorted_slot, void *out, hipStream_t s)
{
    constexpr int NF1 = GATEUP ? 1 : 2, NF2 = GATEUP ? 2 : 4;
    if (d->weight_layout == ZEDA_WEIGHTS_TILED) {
        if (d->T <= 8) return launch<GATEUP, true, NF1, 4>(d, tok, w0, w1, offsets, sorted_slot, out, s);
        return launch<GATEUP, true, NF2, 3>(d, tok, w0, w1, offsets, sorted_slot, out, s);
    }
    if (d->T <= 8) return launch<GATEUP, false, NF1, 4>(d, tok, w0, w1, offsets, sorted_slot, out, s);
    return launch<GATEUP, false, NF2, 3>(d, tok, w0, w1, offsets, sorted_slot, out, s);
}

int launch_gateup_few(const zeda_layer_desc *d, const void *x, const void *wg, const void *wu, const int32_t *offsets,
                      const int32_t *sorted_slot, void *act, hipStream_t s)
{
    return launch_any<true>(d, x, wg, wu, offsets, sorted_slot, act, s);
}

int launch_down_few(const zeda_layer_desc *d, const void *act, const void *wd, const int32_t *offsets, void *y_slot, hipStream_t s)
{
    return launch_any<false>(d, act, wd, nullptr, offsets, nullptr, y_slot, s);
}

}  // namespace zeda
