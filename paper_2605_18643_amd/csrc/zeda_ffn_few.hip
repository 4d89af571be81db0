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
// Row-major weights take a turn through LDS instead (few_multiply_ring): loaded in fragment order, neighbouring lanes touch
// different rows, and such loads arrive at 37 GB/s per CU, half of what the row-major weights and the token rows of a call need.
#include "zeda_place.h"
#include "zeda_select.h"
#include "zeda_wave_ring.h"

namespace zeda {

constexpr int kFewThreads = 256;
constexpr int kFewWaves = kFewThreads / 64;

// this wave's share of the reduction for the first LIVE token blocks: part[a * NB + b][lane] of part.  NT: fetch the weights
// with the non-temporal hint
template <bool TILED, int NA, int NB, int LIVE, int DEPTH, bool NT>
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
            for (int a = 0; a < NA; ++a) {
                const bf16x8 *p = reinterpret_cast<const bf16x8 *>(pa[a] + (kb + s) * wstep);
                fa[d][s][a] = NT ? __builtin_nontemporal_load(p) : *p;
            }
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

// few_multiply of as many token blocks as hold rows.  Three and four blocks keep two chunks in flight: registers.
template <bool TILED, int NA, int NB, int DEPTH, bool NT>
__device__ __forceinline__ void few_multiply_rows(int rows, f32x4 (*part)[64], const bf16_t *const (&pa)[NA], const bf16_t *const (&pt)[NB],
                                                  size_t wstep, int wave, int start, int Kd)
{
    if constexpr (NB == 4) {
        if (rows > 48) return few_multiply<TILED, NA, NB, 4, 2, NT>(part, pa, pt, wstep, wave, start, Kd);
        if (rows > 32) return few_multiply<TILED, NA, NB, 3, 2, NT>(part, pa, pt, wstep, wave, start, Kd);
    }
    if (rows > 16) few_multiply<TILED, NA, NB, 2, DEPTH, NT>(part, pa, pt, wstep, wave, start, Kd);
    else few_multiply<TILED, NA, NB, 1, DEPTH, NT>(part, pa, pt, wstep, wave, start, Kd);
}

// The same from row-major weights through a ring of the wave's own in LDS (zeda_wave_ring.h): the same products in the same order.
// pa, pt: this lane's pieces of rows lane / 8 and 8 + lane / 8 of every block.  lds: the rings, whose memory holds part afterwards.
// Four blocks in flight per wave, 32 KiB of LDS a workgroup: with eight, two workgroups fit on a CU and too little is in flight between
// one's end and the next one's start (N=128, I=768, 64 tokens 191 us, four 173, three 174, two 175).
constexpr int kFewSlots = 4;
template <int NA, int NB, int LIVE, bool NT>
__device__ __forceinline__ void few_multiply_ring(uint32_t lds, f32x4 (*part)[64], const char *const (&pa)[NA][2], const char *const (&pt)[NB][2],
                                                  int wave, int start, int Kd)
{
    constexpr int SEQ = LIVE + NA, D = kFewSlots;  // blocks of a chunk of 64 k: token rows first
    const int lane = threadIdx.x & 63;
    f32x4 acc[NA][LIVE];
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < LIVE; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int n = (Kd / 64 - wave + kFewWaves - 1) / kFewWaves, first = n > 0 ? (int)((unsigned)start % (unsigned)n) : 0, total = n * SEQ;
    WaveRing<D> ring;
    ring.init(lds + wave * WaveRing<D>::BYTES);
    auto col = [&](int c) { const int q = c + first; return (uint32_t)(wave + kFewWaves * (q >= n ? q - n : q)) * 128u; };
    auto fetch = [&](int j, uint32_t at) {
        if (j < LIVE) ring.fetch(pt[j < LIVE ? j : 0][0] + at, pt[j < LIVE ? j : 0][1] + at);
        else ring.template fetch<NT ? 2 : 0>(pa[j < LIVE ? 0 : j - LIVE][0] + at, pa[j < LIVE ? 0 : j - LIVE][1] + at);
    };
#pragma unroll
    for (int i = 0; i < D; ++i)
        if (i < total) fetch(i % SEQ, col(i / SEQ));
    for (int k = 0; k < n; ++k) {
        const int i0 = k * SEQ;
        uint32_t at[D / SEQ + 2];
#pragma unroll
        for (int u = 0; u < D / SEQ + 2; ++u) at[u] = col(min(k + u, n - 1));
        // A block's fragments are read while the block before is multiplied.  (No branch lies between a read and its wait: the
        // compiler could copy the registers there, before the data is in them.)
        u32x4 cur[2], tb[LIVE][2];
        auto read = [&](int i) {
            if (i + D <= total) ring_wait_loads<2 * (D - 1)>();
            else ring_wait_loads<0>();
            ring.read(cur);
        };
        read(i0);
#pragma unroll
        for (int j = 0; j < SEQ; ++j) {
            lds_wait(cur[0], cur[1]);
            if (i0 + j + D < total) fetch((j + D) % SEQ, at[(j + D) / SEQ]);
            const u32x4 f[2] = {cur[0], cur[1]};
            if (j + 1 < SEQ) read(i0 + j + 1);
            __builtin_amdgcn_sched_barrier(0);
            if (j < LIVE) {
                tb[j < LIVE ? j : 0][0] = f[0];
                tb[j < LIVE ? j : 0][1] = f[1];
            } else {
                const int a = j < LIVE ? 0 : j - LIVE;
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int b = 0; b < LIVE; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f[s]), __builtin_bit_cast(bf16x8, tb[b][s]), acc[a][b], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __syncthreads();  // everyone is done with the rings
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < LIVE; ++b) part[a * NB + b][lane] = acc[a][b];
}

template <int NA, int NB, bool NT>
__device__ __forceinline__ void few_multiply_ring_rows(int rows, uint32_t lds, f32x4 (*part)[64], const char *const (&pa)[NA][2],
                                                       const char *const (&pt)[NB][2], int wave, int start, int Kd)
{
    if constexpr (NB == 4) {
        if (rows > 48) return few_multiply_ring<NA, NB, 4, NT>(lds, part, pa, pt, wave, start, Kd);
        if (rows > 32) return few_multiply_ring<NA, NB, 3, NT>(lds, part, pa, pt, wave, start, Kd);
    }
    if (rows > 16) few_multiply_ring<NA, NB, 2, NT>(lds, part, pa, pt, wave, start, Kd);
    else few_multiply_ring<NA, NB, 1, NT>(lds, part, pa, pt, wave, start, Kd);
}

// The routing of up to kTileSelTokens tokens from their partial logits, a token per wave; s_ids receives the ids.  The same
// additions and the same selection as in the router's second kernel, of four waves or of sixteen (tp.by_rows).
__device__ __forceinline__ void select_tokens(const TilePlace &tp, int T, int N, int K, bool lead, float (*lg)[kMaxExperts], int *s_ids)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (wave < T) {
        // (all loads in flight together: each is a trip to another XCD's results)
        constexpr int NC = kMaxExperts / 64, MAXQ = 16;
        float v[MAXQ][NC], bias[NC] = {};
#pragma unroll
        for (int q = 0; q < MAXQ; ++q)
            if (q < tp.slices) {
#pragma unroll
                for (int c = 0; c < NC; ++c) v[q][c] = tp.partial[((size_t)q * tp.Tpad + wave) * tp.E + min(lane + 64 * c, tp.E - 1)];
            }
        if (tp.bias) {
#pragma unroll
            for (int c = 0; c < NC; ++c) bias[c] = tp.bias[min(lane + 64 * c, tp.NE - 1)];
        }
#pragma unroll
        for (int q = 1; q < MAXQ; ++q)
            if (q < tp.slices) {
#pragma unroll
                for (int c = 0; c < NC; ++c) v[0][c] += v[q][c];
            }
#pragma unroll
        for (int c = 0; c < NC; ++c) lg[wave][lane + 64 * c] = v[0][c] + bias[c];
        // (a wave reads what it wrote; experts past NE are left out)
        const int id = select_wave<kMaxExperts / 64>(lg[wave], true, wave, tp.NE, N, K, tp.gate_norm, lead ? tp.ids : nullptr, tp.gates, nullptr, tp.by_rows);
        if (lane < K) s_ids[wave * K + lane] = id;
    }
    __syncthreads();
}

// Where a tile's rows come from: the tables of a placement, the ids of all slots, or the logits of all tokens (tp).
enum FewFrom { kFromTables, kFromIds, kFromLogits };

// GATEUP: tok = x[T,Kd], w0 = W_gate[N,F,Kd], w1 = W_up, out = act[S,F];  else tok = act[S,Kd], w0 = W_down[N,F,Kd],
// out = y_slot[S,F].  Kd a multiple of 64, F of 16 NF.  Up to 16 NB token rows (NB 2 or 4).  Blocks past the last token
// tile return at once.
// RING: weights and tokens go through LDS (row-major weights).
// MULTI: an expert may have more rows than a workgroup takes.
template <bool GATEUP, bool TILED, bool RING, int NF, int NB, int DEPTH, bool MULTI, int FROM>
__global__ __launch_bounds__(kFewThreads) void ffn_few_kernel(const bf16_t *__restrict__ tok, const bf16_t *__restrict__ w0,
                                                              const bf16_t *__restrict__ w1, const int32_t *__restrict__ offsets,
                                                              const int32_t *__restrict__ sorted_slot, bf16_t *__restrict__ out,
                                                              int N, int K, int Kd, int F, int n_ft, int T, TilePlace tp)
{
    static_assert(kFewThreads == kTileThreads && (GATEUP || FROM == kFromTables) && kTileSelTokens <= kFewWaves, "");
    constexpr int NA = GATEUP ? 2 * NF : NF;  // weight blocks: gate and up blocks alternate
    constexpr int PART = kFewWaves * NA * NB * 64 * 16, RINGS = RING ? kFewWaves * WaveRing<kFewSlots>::BYTES : 0;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[PART > RINGS ? PART : RINGS];
    auto s_part = reinterpret_cast<f32x4(*)[NA * NB][64]>(lds);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, kq = lane >> 4;
    const int tile = blockIdx.x / n_ft, ft = blockIdx.x - tile * n_ft;
    int4 loc;
    __shared__ TilePlaceLds<16 * NB> s_place;
    if constexpr (FROM == kFromTables) {
        loc = locate_rows<16 * NB>(offsets, N, tile);
    } else if constexpr (FROM == kFromIds) {
        loc = place_tile<16 * NB>([&](int slot) { return tp.ids[slot]; }, T * K, N, tile, ft == 0, blockIdx.x == 0, s_place, tp.out);
    } else {
        __shared__ float s_lg[kTileSelTokens][kMaxExperts];
        __shared__ int s_ids[kTileSelTokens * kMaxK];
        select_tokens(tp, T, N, K, blockIdx.x == 0, s_lg, s_ids);
        loc = place_tile<16 * NB>([&](int slot) { return s_ids[slot]; }, T * K, N, tile, ft == 0, blockIdx.x == 0, s_place, tp.out);
    }
    if (loc.z == 0) return;
    // (columns past the tile repeat its last row and are never stored; a bad index must not fault)
    auto tok_row = [&](int row) {
        row = min(row, loc.z - 1);
        const int slot = FROM != kFromTables ? s_place.list[row] : GATEUP ? sorted_slot[loc.y + row] : 0;
        return tok + (size_t)(GATEUP ? min(max(slot / K, 0), T - 1) : loc.y + row) * Kd;
    };
    // An expert starts at a chunk of its own, so that not all workgroups stream the same columns: with few rows per expert
    // the same chunk of row-major rows, often a multiple of 4 KiB apart, sits on a few memory channels.  All feature tiles
    // of an expert start alike: neighbours then read neighbouring units of tiled weights at the same time.
    const int start = loc.x * 5;
    if constexpr (RING) {
        const int r8 = lane >> 3;
        const uint32_t piece[2] = {WaveRing<kFewSlots>::piece0(), WaveRing<kFewSlots>::piece1()};
        const char *pt[NB][2], *pa[NA][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int b = 0; b < NB; ++b) pt[b][h] = reinterpret_cast<const char *>(tok_row(16 * b + 8 * h + r8)) + piece[h];
#pragma unroll
            for (int a = 0; a < NA; ++a) {
                const size_t f = (size_t)(ft * NF + (GATEUP ? a / 2 : a)) * 16 + 8 * h + r8;
                pa[a][h] = reinterpret_cast<const char *>(((GATEUP && (a & 1)) ? w1 : w0) + ((size_t)loc.x * F + f) * Kd) + piece[h];
            }
        }
        if (!MULTI || loc.w <= 16 * NB) few_multiply_ring_rows<NA, NB, true>(loc.z, lds_addr(lds), s_part[wave], pa, pt, wave, start, Kd);
        else few_multiply_ring_rows<NA, NB, false>(loc.z, lds_addr(lds), s_part[wave], pa, pt, wave, start, Kd);
    } else {
        const bf16_t *pt[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) pt[b] = tok_row(16 * b + l16) + kq * 8;
        const bf16_t *pa[NA];
#pragma unroll
        for (int a = 0; a < NA; ++a) {
            const int f = (ft * NF + (GATEUP ? a / 2 : a)) * 16;
            const bf16_t *w = ((GATEUP && (a & 1)) ? w1 : w0) + (size_t)loc.x * F * Kd;
            const int row = (f & 31) + l16;  // of the stored unit
            pa[a] = TILED ? w + (size_t)(f >> 5) * 1024 + row * 32 + (kq ^ ((row >> 2) & 3)) * 8 : w + (size_t)(f + l16) * Kd + kq * 8;
        }
        const size_t wstep = TILED ? (size_t)F * 32 : 32;  // elements from one 32-wide k block to the next
        // An expert of several token tiles has its weights fetched by each of them: they are meant to stay in the caches then.
        // (N=16, I=2048, K=1, 64 tokens, loads with one hot expert of 39 rows: 0.88 -> 0.83 of the tile kernel's time)
        if (!MULTI || loc.w <= 16 * NB) few_multiply_rows<TILED, NA, NB, DEPTH, true>(loc.z, s_part[wave], pa, pt, wstep, wave, start, Kd);
        else few_multiply_rows<TILED, NA, NB, DEPTH, false>(loc.z, s_part[wave], pa, pt, wstep, wave, start, Kd);
    }
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

// Where this kernel beats the tile kernels, and with how many 16-row token blocks a workgroup (0: not).  The real loads are
// only known on the device; what is known here is the slots per expert if they fell evenly on all N + Z experts, and the
// tile kernel's gate/up work items, one per 128 columns of I and expert.  Fitted to 37 layer shapes with 1 to 1000 tokens
// under even, Zipf and one-hot-expert loads, and with half of the slots on zero experts.  One rule for both layouts, so that both
// add in the same order; where they differ the tiled one decides: row-major weights, which the rings fetch by whole cache lines,
// would gain from this kernel almost everywhere (last item).  Below: the expert FFN's time here over the better tile kernel's,
// row-major / tiled, even loads, weights from HBM, H = 2048 where nothing else is said.
//  - up to 40 items there is next to nothing to fill the chip with (N=16, I=256, H=512: 83 rows 0.50 / 0.65, 166 rows 0.62 / 0.85);
//  - decode batches: up to 64 items the tile kernel fills a quarter of the chip (N=8, K=6, I=1024: 48 rows 0.61 / 0.92 with
//    four token blocks, 0.72 / 1.24 with two); more of them, and the rows count: N=8, I=3072, 192 items: 16 rows 0.60 / 0.83;
//    N=16, I=2304, K=16, 288 items: 16 rows 0.68 / 0.91, 32 rows 0.73 / 1.10; a filled chip, N=8, I=14336: 8 rows 0.69 / 0.88, 12 rows
//    0.70 / 0.90, at H = 4096 0.73 / 1.04 and 0.77 / 1.04; N=128, I=768: 2 rows 0.75 / 1.00, N=64, I=2048, 6 rows 0.75 / 0.98;
//  - short reductions leave the four waves a chunk or two each: N=64, I=512, H=512: 4 rows 0.77 / 0.91, 8 rows 0.78 / 0.94;
//    N=256, I=256, H=1024: half a slot per expert 0.84 / 1.03, one 0.73 / 1.03 (tiled, Zipf loads: 1.17);
//  - longer batches on a chip that the tile kernel fills: N=128, Z=32, I=768, 5 slots per expert: 0.82 / 1.01 with half of the
//    slots on zero experts (Zipf loads, tiled: 0.94), 0.82 / 1.02 with a fifth of them.  Without zero experts: N=100, I=1024, H=1536
//    0.64 / 0.91, N=128, I=768 0.74 / 0.98 at H = 1024 but 0.82 / 1.02 at H = 2048, N=200, I=512 0.76 / 0.93 (tiled 0.90-1.00 from machine to
//    machine); from H = 4096 on tiled weights are level (N=192, I=2048, 5 rows 0.97 / 0.99; N=96, I=1536 0.83 / 0.99).
//    N=128, I=384, 384 items: 5 slots 0.74 / 0.96, 10 slots 0.73 / 1.01;
//  - between one and two rounds of 256 CUs the tile kernel idles: N=48, I=768, 288 items: 18 rows 0.59 / 0.89, 25 rows 0.63 / 0.98, 30
//    rows 0.66 / 1.05; N=24, I=448, H=1152, 96 items: 30 rows 0.71 / 0.97 (20 of them real: 0.67 / 0.92) with four blocks; N=12,
//    I=704, 72 items: 40 rows 0.62 / 0.93 with four, 0.70 / 1.09 with two.  With one full round it does not: N=60, I=512, 240 items:
//    12 rows 0.69 / 1.05, 16 rows 0.70 / 1.09, 19 rows 0.72 / 1.14;
//  - beyond the rule: N=128, Z=32, I=768: 6 rows 0.83 / 1.04, 12 rows 0.85 / 1.11, 31 rows 1.00 / 1.33; N=64, I=1536: 12 rows 0.83 / 1.07.
int ffn_few_blocks(const zeda_layer_desc *d)
{
    const int64_t slots = (int64_t)d->T * d->K, experts = d->N + d->Z, cols = ceil_div(d->I, 128), items = d->N * cols;
    const int64_t hit = slots < d->N ? slots : d->N, hit_items = hit * cols;
    const bool wide = d->H >= 768 && d->I >= 384;
    // one dimension of workgroups: 2^32 work items, i.e. 2^24 workgroups (the tile kernels' grids do not grow with the layer)
    if ((hit + slots / 32) * (d->I / 16 > d->H / 32 ? d->I / 16 : d->H / 32) >= 1 << 24) return 0;
    if (items <= 40) return d->T <= 64 || slots <= 170 * experts ? 2 : 0;
    if (d->T <= 64) {
        if (hit_items <= 64) return slots <= 25 * experts ? 2 : 4;
        if (wide) return slots <= (hit_items <= 320 ? 16 : 8) * experts ? 2 : 0;
        if (d->I >= 384) return slots <= 4 * experts ? 2 : 0;
        return (hit_items <= 128 ? 2 * slots <= 3 * d->N : slots < d->N) ? 2 : 0;
    }
    if (items > 512) return (d->Z > 0 || d->I >= 1024 || d->H <= 1024) && d->H < 4096 && wide && slots <= 5 * experts ? 2 : 0;
    if (items > 320) return slots <= (wide ? 5 : 2) * experts ? 2 : 0;
    if ((items > 192 && items <= 256) || (items > 64 && !wide)) return slots <= 13 * experts ? 2 : 0;
    if (slots <= 25 * experts) return 2;
    return slots <= (items <= 80 ? 40 : d->Z > 0 ? 32 : 25) * experts ? 4 : 0;
}

// at most this many token tiles of 16 nb rows
static int64_t few_tiles(const zeda_layer_desc *d, int nb)
{
    const int64_t slots = (int64_t)d->T * d->K;
    return (slots < d->N ? slots : d->N) + slots / (16 * nb);
}

template <bool GATEUP, bool TILED, bool RING, int NB, bool MULTI>
static int launch_blocks(const zeda_layer_desc *d, const void *tok, const void *w0, const void *w1, const int32_t *offsets,
                         const int32_t *sorted_slot, void *out, const TilePlace *tp, hipStream_t s)
{
    // 16 gate and 16 up rows, or 32 rows of W_down (16 make twice the workgroups and token reads: 58 -> 61 us at 64 tokens);
    // three chunks of 64 k in flight (four leave fewer waves per SIMD: 177.5 -> 176.5 us)
    constexpr int NF = GATEUP ? 1 : 2, DEPTH = 3;
    const int Kd = GATEUP ? d->H : d->I, F = GATEUP ? d->I : d->H, n_ft = F / (16 * NF);
    const unsigned grid = (unsigned)few_tiles(d, NB) * n_ft;
#define ZEDA_FEW(FROM) ffn_few_kernel<GATEUP, TILED, RING, NF, NB, DEPTH, MULTI, FROM><<<grid, kFewThreads, 0, s>>>( \
        (const bf16_t *)tok, (const bf16_t *)w0, (const bf16_t *)w1, offsets, sorted_slot, (bf16_t *)out, d->N, d->K, Kd, F, n_ft, d->T, tp ? *tp : TilePlace{})
    if constexpr (GATEUP) {
        if constexpr (NB == 2 && !MULTI) {
            if (tp && tp->partial) {
                ZEDA_FEW(kFromLogits);
                return last_launch_status();
            }
        }
        if (tp) ZEDA_FEW(kFromIds);
        else ZEDA_FEW(kFromTables);
    } else {
        ZEDA_FEW(kFromTables);
    }
#undef ZEDA_FEW
    return last_launch_status();
}

// With a few slots per expert, an expert of several token tiles is one of many whose weights are fetched, and the second copy of
// the multiplication costs all workgroups up to half a percent (N=128, I=768, H=2048, 64 tokens, expert FFN: row-major 177.5 -> 178.0
// us, tiled 184.4 -> 185.2).
static bool few_multi(const zeda_layer_desc *d) { return d->T > 32 && (int64_t)d->T * d->K > 8 * ((int64_t)d->N + d->Z); }

// Row-major weights go through the rings where a wave has a chunk to itself (N=32, I=128, H=768, whose down projection has not: 64
// tokens 17.4 -> 18.3 us with them).  Whole layer, without / with: N=128, I=768, H=2048 one token 26.2 / 23.0 us, 32 tokens 161 / 132, 64
// tokens 214 / 173; N=64, I=1536, 64 tokens 214 / 177; N=48, I=768, 301 tokens 112 / 82; N=24, I=448, 301 tokens 36.6 / 28.9.  Tiled
// weights, whose fragments are contiguous KiB already, lose by it (N=128, I=768, 64 tokens 174 -> 189 us with eight blocks in flight).
template <bool GATEUP>
static bool few_ring(const zeda_layer_desc *d) { return (GATEUP ? d->H : d->I) >= 64 * kFewWaves; }

template <bool GATEUP, bool TILED, bool RING>
static int launch(const zeda_layer_desc *d, const void *tok, const void *w0, const void *w1, const int32_t *offsets,
                  const int32_t *sorted_slot, void *out, const TilePlace *tp, hipStream_t s)
{
    if (ffn_few_blocks(d) == 4) return launch_blocks<GATEUP, TILED, RING, 4, true>(d, tok, w0, w1, offsets, sorted_slot, out, tp, s);
    return few_multi(d) ? launch_blocks<GATEUP, TILED, RING, 2, true>(d, tok, w0, w1, offsets, sorted_slot, out, tp, s)
                        : launch_blocks<GATEUP, TILED, RING, 2, false>(d, tok, w0, w1, offsets, sorted_slot, out, tp, s);
}

template <bool GATEUP>
static int launch_layout(const zeda_layer_desc *d, const void *tok, const void *w0, const void *w1, const int32_t *offsets,
                         const int32_t *sorted_slot, void *out, const TilePlace *tp, hipStream_t s)
{
    if (d->weight_layout == ZEDA_WEIGHTS_TILED) return launch<GATEUP, true, false>(d, tok, w0, w1, offsets, sorted_slot, out, tp, s);
    return few_ring<GATEUP>(d) ? launch<GATEUP, false, true>(d, tok, w0, w1, offsets, sorted_slot, out, tp, s)
                       : launch<GATEUP, false, false>(d, tok, w0, w1, offsets, sorted_slot, out, tp, s);
}

// Up to 1024 slots (four a thread) the kernels with a workgroup per 16 or 32 columns place the slots themselves, unless there are
// so many workgroups that placing in each of them costs more than the launch it saves.  How much of it disappears under the loads
// of the CU's other workgroups depends on how long these are, i.e. on H.  Whole layer, us, with a launch / without:
//   bf16, H=2048: 12700 workgroups 264 / 257, 13800 367.7 / 365.5, 15400 383 / 386;  H=1024: 6300 73.8 / 73.1, 7700 118.1 / 123.5, 8700
//   137.7 / 142.7, 15400 212 / 225;  H=512: 6300 46.3 / 45.9, 8700 73.4 / 74.9;  H=4096: 29700 1082 / 1077
//   fp32, 640 workgroups 28.4 / 24.6 and 59.9 / 55.6;  H=256: 3300 82.5 / 80.6, 3800 100.3 / 103.0, 8700 199 / 209;  H=1024: 3300 238.3 / 236.8,
//   3800 286.6 / 291.2, 8700 584 / 596;  H=512: 18400 586 / 669;  H=2048: 5100 682 / 674, 8700 1132 / 1122
bool gateup_places(const zeda_layer_desc *d)
{
    if ((int64_t)d->T * d->K > kTileMaxSlots) return false;
    if (d->dtype == ZEDA_F32) return gateup_f32_workgroups(d) <= (d->H < 2048 ? 3500 : 9 * (int64_t)d->H / 2);
    const int nb = ffn_few_blocks(d);
    return nb > 0 && few_tiles(d, nb) * (d->I / 16) <= 7 * (int64_t)(d->H > 1024 ? d->H : 1024);
}

// A wave per token, so up to four tokens are selected there too, for a kernel of 6.6 us: 4 us in front of every workgroup's weights,
// which pays with up to four workgroups a CU.  Whole layer, us, with the kernel / without: H=2048, 384 workgroups 26.6 / 24.4, 768 32.1 /
// 30.6, 1536 49.0 / 50.6, 3200 81.9 / 89.1, 12700 266 / 328;  H=1024, 384 22.5 / 20.5, 768 28.2 / 26.3, 1536 36.4 / 38.2, 12700 158 / 219;
// H=4096, 768 64.4 / 60.7, 1584 89.1 / 90.5.
bool gateup_selects(const zeda_layer_desc *d)
{
    return d->dtype == ZEDA_BF16 && d->T <= kTileSelTokens && gateup_places(d) && ffn_few_blocks(d) == 2 && few_tiles(d, 2) * (d->I / 16) <= 1024 &&
           route_splits(d);
}

int launch_gateup_few(const zeda_layer_desc *d, const void *x, const void *wg, const void *wu, const int32_t *offsets,
                      const int32_t *sorted_slot, void *act, const TilePlace *tp, hipStream_t s)
{
    return launch_layout<true>(d, x, wg, wu, offsets, sorted_slot, act, tp, s);
}

int launch_down_few(const zeda_layer_desc *d, const void *act, const void *wd, const int32_t *offsets, void *y_slot, hipStream_t s)
{
    return launch_layout<false>(d, act, wd, nullptr, offsets, nullptr, y_slot, nullptr, s);
}

}  // namespace zeda
