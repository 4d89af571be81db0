// Router of the augmented expert pool (Section 2.1): logits over N normal + Z zero experts, the
// top-K set with a deterministic lower-index tie-break, and the routing weights (Section 4.3.4 for
// the normalisation choices).  One fused kernel: projection -> LDS -> wave-level selection.
#include "zeda_f32_tile.h"
#include "zeda_lds.h"
#include "zeda_place.h"
#include "zeda_select.h"

namespace zeda {

// this lane's NC candidates' router biases (past NE: any)
template <int NC>
__device__ __forceinline__ void load_bias(float (&b)[NC], const float *__restrict__ bias, int NE)
{
    const int l16 = threadIdx.x & 15;
#pragma unroll
    for (int c = 0; c < NC; ++c) b[c] = 0.f;
    if (bias) {
#pragma unroll
        for (int c = 0; c < NC; ++c) b[c] = bias[min(l16 + 16 * c, NE - 1)];
    }
}

// All ntok tokens of a workgroup of NWAVES waves, four per wave at a time.  lg holds NP partial logit tables
// pstride floats apart.
// s_cnt (LDS, may be NULL): [ntok / 16][kMaxExperts] counters, zeroed by the caller; every selected slot adds one to
// the counter of its expert in its block of 16 tokens (the counts do not depend on the order of the additions).
// probs (LDS, may be NULL): [ntok][LDP] table that receives every token's routing probabilities.
template <int NC, int NP, int NWAVES>
__device__ __forceinline__ void select_block(const float *lg, int LD, int pstride, const float (&bias)[NC], int ntok,
                                             int t0, int T, int NE, int N, int K, int gate_norm, int32_t *__restrict__ ids,
                                             float *__restrict__ gates, int *s_cnt = nullptr, float *probs = nullptr,
                                             int LDP = 0)
{
    const int wave = threadIdx.x >> 6;
    for (int tk0 = 4 * wave; tk0 < ntok; tk0 += 4 * NWAVES) {
        const int id = select_rows<NC, NP>(lg, LD, pstride, bias, tk0, ntok, t0, T, NE, N, K, gate_norm, ids, gates, probs, LDP);
        if (s_cnt && (unsigned)id < (unsigned)kMaxExperts) atomicAdd(&s_cnt[(tk0 >> 4) * kMaxExperts + id], 1);
    }
}

// After select_block (and a barrier): what the workgroup's blocks of 16 tokens hand to the expert-sorted placement
// and what it hands to the routing statistics.  cnt8[e][cnt_ld] bytes: slots of every block on expert e;
// p_part[workgroup][NE]: the sum of every expert's routing probability over the workgroup's tokens, added in token order (up to 64;
// 16 by 16 is no nearer to 64 bits beyond what draws differ by: 8.4e-8 and 8.6e-8, 8192 to 16384 tokens).
template <int THREADS>
__device__ __forceinline__ void publish_blocks(const int *s_cnt, const float *probs, int LDP, int ntok, int t0, int T, int NE,
                                               uint8_t *__restrict__ cnt8, int cnt_ld, float *__restrict__ p_part)
{
    const int nblk = (ntok + 15) >> 4;
    if (nblk == 1) {  // (one short loop: the two below cost 0.4 us of 16, statistics of 160 experts, 4096 tokens)
        const int nt = min(ntok, T - t0);
        for (int e = threadIdx.x; e < NE && nt > 0; e += THREADS) {
            if (cnt8) cnt8[(size_t)e * cnt_ld + (t0 >> 4)] = (uint8_t)s_cnt[e];
            if (p_part) {
                float ps = 0.f;
                for (int t = 0; t < nt; ++t) ps += probs[t * LDP + e];
                p_part[(size_t)blockIdx.x * NE + e] = ps;
            }
        }
        return;
    }
    if (cnt8) {
        for (int i = threadIdx.x; i < nblk * NE; i += THREADS) {
            const int u = i / NE, e = i - u * NE, blk = (t0 >> 4) + u;
            if (t0 + u * 16 < T) cnt8[(size_t)e * cnt_ld + blk] = (uint8_t)s_cnt[u * kMaxExperts + e];
        }
    }
    if (p_part) {
        const int nt = min(ntok, T - t0);
        for (int e = threadIdx.x; e < NE; e += THREADS) {
            float ps = 0.f;
#pragma unroll 16
            for (int t = 0; t < nt; ++t) ps += probs[t * LDP + e];
            p_part[(size_t)blockIdx.x * NE + e] = ps;
        }
    }
}

// bf16 router.  A workgroup of 16 waves (four for small pools) owns 16 TB tokens, all NE experts (experts are MFMA rows, tokens MFMA columns,
// 16x16x32) and a slice of the hidden dimension, which may be all of it.  x rows and router rows stream through an LDS ring
// in KC-wide k chunks with global->LDS loads whose 16-byte pieces are XOR-permuted by the row (on the global address) so
// that fragment reads spread over the banks.  The waves split a chunk's k steps and the expert blocks; the k steps' sums
// meet in LDS tables.  Without a split the workgroup selects for its tokens, four per wave, adding the tables in order;
// with one it leaves its logits to route_select_kernel.  All orders are fixed: the logits are reproducible.
//
// What bounds it is what a CU pulls from L2: every router row of its slice (8-row pieces of 128 bytes and more arrive at up
// to 129 GB/s per CU, 64-byte pieces at half of that), then launch and selection (route_plan weighs them).
constexpr int kRouteWaves = 16;
constexpr int kRouteWavesSmall = 4;
constexpr int kRouteSmallNB = 2;  // ... for up to 32 times this many experts (select_wave's by_rows: a candidate a lane)
// k chunk of a workgroup of 16 tb tokens and `waves` waves
__host__ __device__ constexpr int route_chunk(int tb, int waves) { return tb == 1 || (tb == 2 && waves == kRouteWavesSmall) ? 128 : 64; }

template <int NB, int TB, int W>
struct RouteCfg {
    static constexpr int THREADS = 64 * W;
    static constexpr int TOK = 16 * TB;            // tokens of the workgroup
    static constexpr int KC = route_chunk(TB, W);  // k chunk
    static constexpr int KS = KC / 32;             // MFMA k steps per chunk
    static constexpr int GROUPS = W / KS;          // expert groups: group g owns the 16-expert blocks g, g + GROUPS, ...
    static constexpr int EB = 2 * NB, BPW = (EB + GROUPS - 1) / GROUPS;
    static constexpr int ROWB = 2 * KC, PPR = ROWB / 16, RPI = 64 / PPR;  // bytes, 16-byte pieces per row; rows per load instruction
    static constexpr int ROWS = TOK + 32 * NB, STAGE = ROWS * ROWB;
    static constexpr int NI = ROWS / RPI;            // load instructions per chunk, dealt out to the waves
    static constexpr int MAX_LDS = W == kRouteWavesSmall ? 80 * 1024 : 160 * 1024;  // (two small workgroups per CU)
    static constexpr int STAGES = MAX_LDS / STAGE < 8 ? MAX_LDS / STAGE : 8;
    static constexpr int LD = NB * 32 + 1;
    static constexpr int TABLES = KS * TOK * LD * 4;  // bytes of the logit tables, which reuse the ring, as do the counters
    static constexpr int CNT_OFF = (TABLES + 15) / 16 * 16, END = CNT_OFF + TB * kMaxExperts * 4;
    static constexpr int LDS_BYTES = STAGES * STAGE > END ? STAGES * STAGE : END;
    static_assert(ROWS % RPI == 0 && STAGES >= 2 && LDS_BYTES <= MAX_LDS && GROUPS >= 1, "");
    static_assert((STAGES - 1) * ((NI + W - 1) / W) <= 63, "vmcnt is a 6-bit counter");
    static __device__ __forceinline__ int swz(int row, int piece) { return KC == 128 ? piece ^ (row & 15) : piece ^ ((row >> 1) & 7); }
};

template <int N>
__device__ __forceinline__ void route_wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// partial (may be NULL): receives the logits of the workgroup's slice of the hidden dimension instead of a selection.
// cnt8, p_part (either may be NULL): see publish_blocks.
template <int NB, int TB, int W>
__global__ __launch_bounds__(64 * W) void route_bf16_kernel(const bf16_t *__restrict__ x, const bf16_t *__restrict__ wr,
                                                                   const float *__restrict__ bias, int T, int H, int N, int NE,
                                                                   int K, int gate_norm, int32_t *__restrict__ ids,
                                                                   float *__restrict__ gates, float *__restrict__ partial, int Tpad,
                                                                   uint8_t *__restrict__ cnt8, int cnt_ld,
                                                                   float *__restrict__ p_part)
{
    typedef RouteCfg<NB, TB, W> C;
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t0 = blockIdx.x * C::TOK, l16 = lane & 15, kq = lane >> 4;
    const int ks = wave % C::KS, grp = wave / C::KS;

    float bias_c[2 * NB];
    load_bias<2 * NB>(bias_c, bias, NE);

    constexpr int NLHI = (C::NI + W - 1) / W, NLLO = C::NI / W;
    const bool hi = wave < C::NI % W || NLHI == NLLO;  // this wave issues NLHI loads per chunk, else NLLO
    const bf16_t *src[NLHI];
#pragma unroll
    for (int i = 0; i < NLHI; ++i) {
        const int row = min((wave + W * i) * C::RPI + lane / C::PPR, C::ROWS - 1), piece = lane % C::PPR;
        const bf16_t *base = row < C::TOK ? x + (size_t)min(t0 + row, T - 1) * H : wr + (size_t)min(row - C::TOK, NE - 1) * H;
        src[i] = base + (size_t)blockIdx.y * (H / gridDim.y) + C::swz(row, piece) * 8;
    }
    // All workgroups read the same router rows, and rows are a power-of-two number of bytes apart, so one k chunk of every
    // row sits on a few L2 channels: each workgroup starts at a chunk of its own (a fixed order, so results are
    // reproducible).
    const int nk = H / C::KC / gridDim.y;  // gridDim.y workgroups share a token block: each takes a slice of the hidden dimension
    const int rot = (int)((blockIdx.x * 5u) % (unsigned)nk);
    int kc = rot;  // the next chunk to fetch
    auto issue = [&](int s) {
        unsigned char *slot = lds + s * C::STAGE;
#pragma unroll
        for (int i = 0; i < NLHI; ++i)
            if (i < NLLO || hi)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src[i] + (size_t)kc * C::KC),
                                                 (__attribute__((address_space(3))) void *)(slot + (wave + W * i) * 1024), 16, 0, 0);
        kc = kc + 1 == nk ? 0 : kc + 1;
    };

    f32x4 acc[C::BPW][TB];
#pragma unroll
    for (int b = 0; b < C::BPW; ++b)
#pragma unroll
        for (int u = 0; u < TB; ++u) acc[b][u] = f32x4{0.f, 0.f, 0.f, 0.f};

#pragma unroll
    for (int c = 0; c < C::STAGES - 1; ++c) issue(c);  // (with fewer chunks than slots some are fetched again and not used)
#pragma unroll
    for (int c = 0; c < 2 * NB; ++c) asm volatile("" : "+v"(bias_c[c]));  // (fetched up here, not where the selection uses it)
    // (blocks start at multiples of 16 rows, so the piece permutation depends on l16 only)
    const uint32_t ring = lds_addr(lds), pos = C::swz(l16, 4 * ks + kq) * 16;
    int cslot = 0, fslot = C::STAGES - 1;  // slots of the chunk being multiplied and of the next one to fetch
    for (int it = 0; it < nk; ++it) {
        if (it + C::STAGES - 2 < nk) {
            if (hi) route_wait_vmcnt<(C::STAGES - 2) * NLHI>();
            else route_wait_vmcnt<(C::STAGES - 2) * NLLO>();
        } else {
            route_wait_vmcnt<0>();
        }
        __builtin_amdgcn_s_barrier();
        if (it + C::STAGES - 1 < nk) issue(fslot);
        const uint32_t cur = ring + cslot * C::STAGE;
        cslot = cslot + 1 == C::STAGES ? 0 : cslot + 1;
        fslot = fslot + 1 == C::STAGES ? 0 : fslot + 1;
        // this wave's 32-wide step of the chunk: pieces 4 ks .. 4 ks + 3 of every row (groups with fewer blocks than BPW
        // read their last block again and leave it out)
        u32x4 tb[TB], fa[C::BPW];
#pragma unroll
        for (int u = 0; u < TB; ++u) tb[u] = lds_read_b128(cur + (u * 16 + l16) * C::ROWB + pos);
#pragma unroll
        for (int b = 0; b < C::BPW; ++b)
            fa[b] = lds_read_b128(cur + (C::TOK + min(grp + C::GROUPS * b, C::EB - 1) * 16 + l16) * C::ROWB + pos);
#pragma unroll
        for (int u = 0; u < TB; ++u) lds_wait(tb[u]);
#pragma unroll
        for (int b = 0; b < C::BPW; ++b) lds_wait(fa[b]);
#pragma unroll
        for (int b = 0; b < C::BPW; ++b) {
            if (C::EB % C::GROUPS && b == C::BPW - 1 && grp + C::GROUPS * b >= C::EB) break;
#pragma unroll
            for (int u = 0; u < TB; ++u)
                acc[b][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fa[b]), __builtin_bit_cast(bf16x8, tb[u]),
                                                                    acc[b][u], 0, 0, 0);
        }
    }
    __syncthreads();  // everyone is done with the ring: its memory now holds the logits and what the selection leaves

    // acc[b][u][v]: expert 16 (grp + GROUPS b) + 4 kq + v, token 16 u + l16; one table per k step of the chunk
    float *lg = reinterpret_cast<float *>(lds);
    int *s_cnt = reinterpret_cast<int *>(lds + C::CNT_OFF);
#pragma unroll
    for (int b = 0; b < C::BPW; ++b) {
        if (grp + C::GROUPS * b >= C::EB) break;
#pragma unroll
        for (int u = 0; u < TB; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                lg[(ks * C::TOK + u * 16 + l16) * C::LD + (grp + C::GROUPS * b) * 16 + 4 * kq + v] = acc[b][u][v];
    }
    if (partial) {
        // this slice's sums (the tables added in order) go to partial[slice][token][expert], Tpad tokens: route_select_kernel adds the
        // slices in order and selects
        __syncthreads();
        f32x4 *dst = reinterpret_cast<f32x4 *>(partial + ((size_t)blockIdx.y * Tpad + t0) * (NB * 32));
        for (int i = tid; i < min(C::TOK, Tpad - t0) * NB * 8; i += C::THREADS) {
            const float *p = lg + (i / (NB * 8)) * C::LD + (i % (NB * 8)) * 4;
            f32x4 v;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v[k] = p[k];
#pragma unroll
                for (int q = 1; q < C::KS; ++q) v[k] += p[q * C::TOK * C::LD + k];
            }
            dst[i] = v;
        }
        return;
    }
    if (cnt8)
        for (int i = tid; i < TB * kMaxExperts; i += C::THREADS) s_cnt[i] = 0;
    __syncthreads();
    // The probabilities of a token overwrite its row of the first logit table once the token's logits are in registers.
    select_block<2 * NB, C::KS, W>(lg, C::LD, C::TOK * C::LD, bias_c, C::TOK, t0, T, NE, N, K, gate_norm, ids, gates,
                                             cnt8 ? s_cnt : nullptr, p_part ? lg : nullptr, C::LD);
    if (cnt8 || p_part) {
        __syncthreads();
        publish_blocks<C::THREADS>(s_cnt, lg, C::LD, C::TOK, t0, T, NE, cnt8, cnt_ld, p_part);
    }
}

// Second kernel where the hidden dimension was split: 16 tokens per workgroup.  All threads add up the slices' tables
// (16-byte loads, all slices' in flight), then a wave selects for one token (16 waves) or for four (four waves).
// cnt8, p_part (either may be NULL): see publish_blocks.  place.offsets (may be NULL): one workgroup, which then places.
constexpr int kSelectTokens = 16;
template <int NB, int NP, int W>
__global__ __launch_bounds__(64 * W) void route_select_kernel(const float *__restrict__ partial, int Tpad,
                                                              const float *__restrict__ bias, int T, int N, int NE,
                                                              int K, int gate_norm, int32_t *__restrict__ ids,
                                                              float *__restrict__ gates, uint8_t *__restrict__ cnt8,
                                                              int cnt_ld, float *__restrict__ p_part, PlaceOut place)
{
    static_assert(kSelectTokens == 16 && (W == 16 || W == 4), "one block of the per-block tables, one or four tokens a wave");
    constexpr int E = NB * 32, NC = (E + 63) / 64, LD = NC * 64, THREADS = 64 * W;
    __shared__ __attribute__((aligned(16))) float lg[kSelectTokens * LD];
    __shared__ int s_cnt[kMaxExperts], s_ids[kSelectTokens * kMaxK];
    __shared__ PlaceLds<kSelectTokens * kMaxK> s_place;
    const int t0 = blockIdx.x * kSelectTokens, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int i = threadIdx.x; i < kSelectTokens * E / 4; i += THREADS) {
        const int tk = i / (E / 4), e = (i - tk * (E / 4)) * 4;
        f32x4 b = {0.f, 0.f, 0.f, 0.f};
        if (bias) {
#pragma unroll
            for (int k = 0; k < 4; ++k) b[k] = bias[min(e + k, NE - 1)];
        }
        f32x4 v[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) v[q] = *reinterpret_cast<const f32x4 *>(partial + ((size_t)q * Tpad + t0 + tk) * E + e);
#pragma unroll
        for (int q = 1; q < NP; ++q) v[0] += v[q];
        *reinterpret_cast<f32x4 *>(lg + tk * LD + e) = v[0] + b;
    }
    for (int e = threadIdx.x; e < kMaxExperts; e += THREADS) s_cnt[e] = 0;
    __syncthreads();
    // (a token's probabilities overwrite its logits, which are in its wave's registers by then)
    int id;
    if constexpr (W == 16) {
        id = select_wave<NC>(lg + wave * LD, t0 + wave < T, (size_t)t0 + wave, NE, N, K, gate_norm, ids, gates, p_part ? lg + wave * LD : nullptr);
        if (lane < K) s_ids[wave * K + lane] = id;
    } else {
        const float no_bias[2 * NB] = {};
        id = select_rows<2 * NB, 1>(lg, LD, 0, no_bias, 4 * wave, kSelectTokens, t0, T, NE, N, K, gate_norm, ids, gates, p_part ? lg : nullptr, LD);
        if ((lane & 15) < K) s_ids[(4 * wave + (lane >> 4)) * K + (lane & 15)] = id;
    }
    if ((unsigned)id < (unsigned)kMaxExperts) atomicAdd(&s_cnt[id], 1);
    __syncthreads();
    if (cnt8 || p_part) publish_blocks<THREADS>(s_cnt, lg, LD, kSelectTokens, t0, T, NE, cnt8, cnt_ld, p_part);
    if (place.offsets) place_list<THREADS>(s_ids, T * K, N, s_place, place);
}

// fp32 router.  A workgroup owns 16 tokens and all experts; its 16 waves split the hidden dimension and, above 32
// experts, the experts: each multiplies NA blocks of 16 router rows with the token block (zeda_f32_tile.h), the slices'
// sums meet in LDS and are added in slice order, and four waves select.  NC: candidates per lane of the selection, the
// expert count in blocks of 16 rounded up to a power of two.  Loads in flight are what counts here (513 tokens of
// H = 1024, 40 experts: 33 workgroups); one wave walking expert after expert with a sum over its lanes took 70 us.
constexpr int kRouteF32Tokens = 16;
constexpr int kRouteF32Threads = 1024;

template <int NC>
__global__ __launch_bounds__(kRouteF32Threads) void route_f32_kernel(const float *__restrict__ x, const float *__restrict__ wr,
                                                                     const float *__restrict__ bias, int T, int H, int N,
                                                                     int NE, int K, int gate_norm, int32_t *__restrict__ ids,
                                                                     float *__restrict__ gates, float *__restrict__ logits_out,
                                                                     int LDg)
{
    constexpr int NA = NC < 2 ? NC : 2, GROUPS = NC / NA, SLICES = kRouteF32Threads / 64 / GROUPS, LD = NC * 16;
    static_assert(SLICES * kRouteF32Tokens * LD * 4 <= 64 * 1024, "the slices' logit tables fit in the default LDS size");
    __shared__ __attribute__((aligned(16))) float lg[SLICES * kRouteF32Tokens * LD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15;
    const int group = wave % GROUPS, slice = wave / GROUPS, t0 = blockIdx.x * kRouteF32Tokens;
    const float *pa[NA], *pb[1] = {x + (size_t)min(t0 + l16, T - 1) * H};
#pragma unroll
    for (int a = 0; a < NA; ++a) pa[a] = wr + (size_t)min((group * NA + a) * 16 + l16, NE - 1) * H;
    {
        F32Tile<NA, 1> t;
        t.run(pa, pb, slice, SLICES, (int)blockIdx.x, H);
#pragma unroll
        for (int a = 0; a < NA; ++a)  // lane l: experts 4 (l / 16) .. + 3 of the block, token l % 16
            *reinterpret_cast<f32x4 *>(lg + (slice * kRouteF32Tokens + l16) * LD + (group * NA + a) * 16 + 4 * (lane >> 4)) = t.total(a, 0);
    }
    __syncthreads();
    for (int i = tid; i < kRouteF32Tokens * LD; i += kRouteF32Threads) {
        double v = lg[i];  // (rounded once)
#pragma unroll
        for (int q = 1; q < SLICES; ++q) v += (double)lg[q * kRouteF32Tokens * LD + i];
        lg[i] = (float)v;
    }
    __syncthreads();
    if (logits_out) {  // statistics run: hand the logits (without the bias) to route_stats_kernel
        for (int i = tid; i < kRouteF32Tokens * NE; i += kRouteF32Threads)
            logits_out[(size_t)(t0 + i / NE) * LDg + (i % NE)] = lg[(i / NE) * LD + (i % NE)];
        return;
    }
    float bias_c[NC];
    load_bias<NC>(bias_c, bias, NE);
    select_block<NC, 1, kRouteF32Threads / 64>(lg, LD, 0, bias_c, kRouteF32Tokens, t0, T, NE, N, K, gate_norm, ids, gates);
}

static int launch_route_f32(const zeda_layer_desc *d, const void *x, const void *wr, const float *bias, int32_t *ids,
                            float *gates, float *logits_out, int LDg, hipStream_t s)
{
    const int NE = d->N + d->Z, grid = ceil_div(d->T, kRouteF32Tokens);
#define ZEDA_ROUTE_F32(NC) route_f32_kernel<NC><<<grid, kRouteF32Threads, 0, s>>>((const float *)x, (const float *)wr, bias, d->T, d->H, d->N, NE, d->K, d->gate_norm, ids, gates, logits_out, LDg)
    if (NE <= 16) ZEDA_ROUTE_F32(1);
    else if (NE <= 32) ZEDA_ROUTE_F32(2);
    else if (NE <= 64) ZEDA_ROUTE_F32(4);
    else if (NE <= 128) ZEDA_ROUTE_F32(8);
    else ZEDA_ROUTE_F32(16);
#undef ZEDA_ROUTE_F32
    return last_launch_status();
}

// How a bf16 router launch is split: 16 tb tokens and `waves` waves per workgroup, `slices` workgroups per token block.
struct RoutePlan {
    int tb, slices, waves;
};

// bytes of one token's logits in the scratch
static size_t route_row_bytes(const zeda_layer_desc *d) { return (size_t)ceil_div(d->N + d->Z, 32) * 32 * sizeof(float); }

// Scratch for the slices' logits: room for eight slices of 32-token blocks, halved until blocks times slices are within 256
// and the slices are whole 64-wide chunks.  Callers size workspaces once, for their largest batch, so this size is part of
// the interface: route_plan takes splits that fit into it.
size_t route_ws_bytes(const zeda_layer_desc *d)
{
    if (d->dtype != ZEDA_BF16) return 0;
    const int blocks = ceil_div(d->T, 32);
    size_t c = 1;
    while (c < 8 && blocks * 2 * c <= 256 && d->H / 64 % (2 * c) == 0) c *= 2;
    return c == 1 ? 0 : c * blocks * 32 * route_row_bytes(d);
}

// tokens whose logits the scratch holds: whole blocks of the selecting kernel
static int route_tpad(const zeda_layer_desc *d) { return ceil_div(d->T, kSelectTokens) * kSelectTokens; }

// The split whose workgroups move the least (a CU pulls router rows out of L2 at 105-129 GB/s), among those that fit into
// the scratch and run in one round: the rows a projecting workgroup reads, taken 1.4 and 1.6 times with 32 and 64 tokens
// (64-wide chunks: twice the barriers) and 1.3 times where the ring of 128-wide chunks has two slots only (above 192
// experts); with a split also the second kernel and the logits that both kernels move.  The factors are fitted to
// measurements of every split at 96 to 256 experts, H = 512 to 7168 and 1 to 40000 tokens: the chosen one is 0.6 % behind
// the best one on average.  Some of them, us, one kernel / best split:
//   H = 2048:  96 experts, 1 token 10.1 / 7.9, 512 tokens 10.8 / 9.2, 1500 10.9 / 11.4;  160 experts, 1 token 15.0 / 8.7,
//   997 tokens 13.1 / 11.7, 2048 13.1 / 12.6, 4096 13.7 / 16.6;  192 experts, 2048 tokens 14.4 / 13.4, 4096 15.1 / 17.2
//   H = 1024:  96 experts, 200 tokens 8.1 / 8.5, 160 experts 9.6 / 10.0
// Up to 64 experts there is too little to do for 16 waves (32 experts, H = 2048: 7.5 us for one token, 14.5 for 8192; four
// waves 5.6 and 9.3-10.4): four-wave workgroups, up to two per CU.  At H = 7168 a second one only gets in the way (6000
// tokens: 16-token workgroups 28.7 us, 32-token ones 25.1).
static RoutePlan route_plan(const zeda_layer_desc *d, bool scratch)
{
    const int64_t NE = d->N + d->Z, kb = 1000;
    const bool small = NE <= 32 * kRouteSmallNB;
    const size_t room = scratch ? route_ws_bytes(d) / route_row_bytes(d) : 0;  // tokens times slices
    RoutePlan best = {4, 1, small ? kRouteWavesSmall : kRouteWaves};
    int64_t least = INT64_MAX;
    for (int tb = 1; tb <= 4; tb *= 2) {
        const int64_t tok = 16 * tb, blocks = (d->T + tok - 1) / tok;
        const int chunks = d->H / route_chunk(tb, best.waves);
        for (int c = 1; c <= 16; c *= 2) {
            if (c > 1 && (chunks % c != 0 || (size_t)c * route_tpad(d) > room)) break;
            if (blocks * c > (small && c == 1 && d->H <= 4096 ? 512 : 256) && !(c == 1 && tb == 4)) break;
            const int64_t rows = (NE + tok) * d->H * 2 / c, load = blocks * c > 256 ? blocks * c : 256;  // load: of the 256 CUs
            const int64_t cost = small ? rows * (tb == 1 ? 10 : tb == 2 ? 11 : 18) / 10 * load / 256 + (c > 1 ? 100 * kb + c * NE * 128 : 0)
                                       : rows * (tb == 1 ? (NE > 192 ? 13 : 10) : tb == 2 ? 14 : 16) / 10 + (c > 1 ? 150 * kb + (c * 64 + tok * 32) * NE : 0);
            if (cost < least) { least = cost; best.tb = tb; best.slices = c; }
        }
    }
    return best;
}

// Optional outputs of a router launch (see publish_blocks, place_list); all NULL / 0 when not wanted.
struct RouteExtras {
    uint8_t *cnt8;
    int cnt_ld;
    float *p_part;
    PlaceOut place;
    TilePlace *tp;  // given: the gate/up kernel selects
};

template <int NB, int TB, int W>
static int launch_route_bf16(const zeda_layer_desc *d, const void *x, const void *wr, const float *bias, int32_t *ids,
                             float *gates, float *partial, int slices, const RouteExtras &ex, hipStream_t s)
{
    typedef RouteCfg<NB, TB, W> C;
    // the kernel uses more LDS than a launch gets by default: opt in once per kernel and device
    static bool done[kMaxDevices] = {};  // idempotent, so a race between host threads is harmless
    const int dev = current_device();
    if (dev < 0) return ZEDA_EHIP;
    if (!done[dev]) {
        if (hipFuncSetAttribute((const void *)route_bf16_kernel<NB, TB, W>, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES) != hipSuccess)
            return ZEDA_EHIP;
        done[dev] = true;
    }
    const int NE = d->N + d->Z, Tpad = route_tpad(d);
    route_bf16_kernel<NB, TB, W><<<dim3(ceil_div(d->T, C::TOK), slices), C::THREADS, C::LDS_BYTES, s>>>(
        (const bf16_t *)x, (const bf16_t *)wr, bias, d->T, d->H, d->N, NE, d->K, d->gate_norm, ids, gates, slices > 1 ? partial : nullptr, Tpad,
        ex.cnt8, ex.cnt_ld, ex.p_part);
    if (ex.tp && slices > 1) {
        ex.tp->partial = partial;
        ex.tp->slices = slices;
        ex.tp->Tpad = Tpad;
        ex.tp->E = NB * 32;
        ex.tp->by_rows = W == kRouteWavesSmall;
        return last_launch_status();
    }
    const dim3 sgrid(ceil_div(d->T, kSelectTokens));
#define ZEDA_SELECT(NP) route_select_kernel<NB, NP, W><<<sgrid, C::THREADS, 0, s>>>(partial, Tpad, bias, d->T, d->N, NE, d->K, d->gate_norm, ids, gates, ex.cnt8, ex.cnt_ld, ex.p_part, ex.place)
    if (slices == 2) ZEDA_SELECT(2);
    else if (slices == 4) ZEDA_SELECT(4);
    else if (slices == 8) ZEDA_SELECT(8);
    else if (slices == 16) ZEDA_SELECT(16);
#undef ZEDA_SELECT
    return last_launch_status();
}

template <int NB, int W>
static int launch_route_bf16_tok(const zeda_layer_desc *d, const void *x, const void *wr, const float *bias, int32_t *ids,
                                 float *gates, float *partial, const RoutePlan &p, const RouteExtras &ex, hipStream_t s)
{
    if (p.tb == 1) return launch_route_bf16<NB, 1, W>(d, x, wr, bias, ids, gates, partial, p.slices, ex, s);
    if (p.tb == 2) return launch_route_bf16<NB, 2, W>(d, x, wr, bias, ids, gates, partial, p.slices, ex, s);
    return launch_route_bf16<NB, 4, W>(d, x, wr, bias, ids, gates, partial, p.slices, ex, s);
}

template <int NB>
static int launch_route_bf16_waves(const zeda_layer_desc *d, const void *x, const void *wr, const float *bias, int32_t *ids,
                                   float *gates, float *partial, const RouteExtras &ex, hipStream_t s)
{
    const RoutePlan p = route_plan(d, partial != nullptr);
    if constexpr (NB <= kRouteSmallNB) {
        if (p.waves == kRouteWavesSmall) return launch_route_bf16_tok<NB, kRouteWavesSmall>(d, x, wr, bias, ids, gates, partial, p, ex, s);
    }
    return launch_route_bf16_tok<NB, kRouteWaves>(d, x, wr, bias, ids, gates, partial, p, ex, s);
}

static int launch_route_bf16_any(const zeda_layer_desc *d, const void *x, const void *wr, const float *bias, int32_t *ids,
                                 float *gates, float *partial, const RouteExtras &ex, hipStream_t s)
{
    switch (ceil_div(d->N + d->Z, 32)) {
        case 1: return launch_route_bf16_waves<1>(d, x, wr, bias, ids, gates, partial, ex, s);
        case 2: return launch_route_bf16_waves<2>(d, x, wr, bias, ids, gates, partial, ex, s);
        case 3: return launch_route_bf16_waves<3>(d, x, wr, bias, ids, gates, partial, ex, s);
        case 4: return launch_route_bf16_waves<4>(d, x, wr, bias, ids, gates, partial, ex, s);
        case 5: return launch_route_bf16_waves<5>(d, x, wr, bias, ids, gates, partial, ex, s);
        case 6: return launch_route_bf16_waves<6>(d, x, wr, bias, ids, gates, partial, ex, s);
        case 7: return launch_route_bf16_waves<7>(d, x, wr, bias, ids, gates, partial, ex, s);
        default: return launch_route_bf16_waves<8>(d, x, wr, bias, ids, gates, partial, ex, s);
    }
}

bool route_splits(const zeda_layer_desc *d) { return d->dtype == ZEDA_BF16 && route_plan(d, true).slices > 1; }
bool route_places(const zeda_layer_desc *d) { return d->T <= kSelectTokens && route_splits(d); }

int route_counts_ld(const zeda_layer_desc *d) { return (int)align_up((size_t)ceil_div(d->T, 16), 16); }
size_t route_counts_bytes(const zeda_layer_desc *d) { return align_up((size_t)(d->N + d->Z) * route_counts_ld(d), 256); }
bool route_counts_supported(const zeda_layer_desc *d) { return d->dtype == ZEDA_BF16; }

// ---------------------------------------------------------------------------------------------
// Batch routing statistics (Section 2.2, Eq. 4-6): f_i, P_i, the group sums and the forward values of the
// two auxiliary losses, over all T tokens as the batch.  bf16: the router kernels themselves leave, per block of 16
// tokens, the slots on every expert and the sums of the routing probabilities (the logits, the softmax and the
// selected set are in their registers anyway), and one final workgroup adds the blocks up in order
// (route_stats_final_kernel).  fp32: logits to scratch (route_f32_kernel), per-block sums (route_stats_kernel), the
// same final workgroup.  Every floating-point sum runs in a fixed order.
// ---------------------------------------------------------------------------------------------
constexpr int kStatsThreads = 256;
constexpr int kStatsTokens = 64;  // tokens per workgroup of route_stats_kernel: four batches of four per wave

template <int NC>
__global__ __launch_bounds__(kStatsThreads) void route_stats_kernel(const float *__restrict__ logits, int nsplit, int Tpad,
                                                                    int LDg, const float *__restrict__ bias, int T, int NE,
                                                                    int K, float *__restrict__ p_part,
                                                                    int32_t *__restrict__ f_part)
{
    __shared__ float s_p[16][kMaxExperts];
    __shared__ int s_f[16][kMaxExperts];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, row = lane >> 4;
    const int t0 = blockIdx.x * kStatsTokens;
    float psum[NC];
    int fcnt[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) { psum[c] = 0.f; fcnt[c] = 0; }
    for (int batch = 0; batch < kStatsTokens / 16; ++batch) {
        const int t = t0 + batch * 16 + wave * 4 + row;
        const bool ok = t < T;
        float cand[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) cand[c] = -INFINITY;
        if (ok) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (l16 + 16 * c < NE) cand[c] = logits[(size_t)t * LDg + l16 + 16 * c];
            for (int q = 1; q < nsplit; ++q) {
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    if (l16 + 16 * c < NE) cand[c] += logits[((size_t)q * Tpad + t) * LDg + l16 + 16 * c];
            }
            if (bias) {
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    if (l16 + 16 * c < NE) cand[c] += bias[l16 + 16 * c];
            }
        }
        // probabilities: softmax over all N+Z logits of the token (the row)
        float m = cand[0];
#pragma unroll
        for (int c = 1; c < NC; ++c) m = fmaxf(m, cand[c]);
        m = row_max(m);
        float ex[NC], sacc = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            ex[c] = (ok && l16 + 16 * c < NE) ? expf(cand[c] - m) : 0.f;
            sacc += ex[c];
        }
        const float all = row_sum(sacc);
        if (ok) {
#pragma unroll
            for (int c = 0; c < NC; ++c) psum[c] += ex[c] / all;
        }
        // the top-K set, as in select_rows: K rounds of (row maximum, lowest index among equals)
        int key[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) key[c] = ok && l16 + 16 * c < NE ? logit_key(cand[c]) : kNoKey;
        for (int j = 0; j < K; ++j) {
            int mm = key[0];
#pragma unroll
            for (int c = 1; c < NC; ++c) mm = max(mm, key[c]);
            mm = row_max(mm);
            int mine = INT_MAX;
#pragma unroll
            for (int c = NC - 1; c >= 0; --c)
                if (key[c] == mm) mine = l16 + 16 * c;
            int win = row_min(mine);
            if (mm == kNoKey) win = INT_MAX;  // nothing but no-numbers left: no expert
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (win == l16 + 16 * c) {
                    key[c] = kNoKey;
                    ++fcnt[c];
                }
        }
    }
    // 16 (wave, row) partial tables -> one per workgroup, added in table order
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        s_p[wave * 4 + row][l16 + 16 * c] = psum[c];
        s_f[wave * 4 + row][l16 + 16 * c] = fcnt[c];
    }
    __syncthreads();
    if (tid < NE) {
        float ps = 0.f;
        int fs = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) { ps += s_p[r][tid]; fs += s_f[r][tid]; }
        p_part[(size_t)blockIdx.x * NE + tid] = ps;
        f_part[(size_t)blockIdx.x * NE + tid] = fs;
    }
}

// Final workgroup: adds everything up.  p_part [rows][NE], a row per workgroup of the kernel before, and either f_part, int32
// counts laid out alike, or cnt8[e][cnt_ld], the counts of nblocks blocks of 16 tokens as bytes.  A thread takes four experts of
// p_part, with one 16-byte load where rows are that aligned.  The threads of an expert quad, kStatsParts at most, take every
// parts-th row, and their sums are added in a fixed order (16 experts, 16 tokens: 256 threads a quad cost 3 us, 32 cost 0.3); counts
// are added as integers, so their order does not matter.  (One thread per expert walking all rows: 142 us at 8192 tokens.)
// What it waits for is one CU's share of memory, and in short calls its own instructions, which nobody has fetched before it.  LONG
// (stats_long): twelve loads of p_part a thread in flight, and a wave for an expert's counts, eight experts in flight; else short
// loops, and a word of counts a thread.
constexpr int kStatsFinalThreads = 1024;
constexpr int kStatsParts = 32;

// Short loops / LONG, us, H = 2048: 160 experts, 16 tokens 2.7 / 8.1, 1500 4.6 / 8.5, 6000 7.2 / 9.2, 8192 9.1 / 7.6, 10000 9.7 / 8.1, 16384
// 13.7 / 7.9;  96 experts, 1500 tokens 3.9 / 5.4, 5000 5.1 / 5.6, 8192 6.3 / 4.9;  32, 8192 tokens 4.3 / 4.4, 16384 5.2 / 4.8;  256, 6000
// tokens 8.1 / 9.2, 8192 11.6 / 8.6;  250, whose rows have no 16-byte pieces, 8192 tokens 19.6 / 24.8, 16384 25.1 / 24.8.
static bool stats_long(int cnt_ld, int NE) { return cnt_ld >= 32 * 16 && NE % 4 == 0; }

template <bool LONG>
__global__ __launch_bounds__(kStatsFinalThreads) void route_stats_final_kernel(const float *__restrict__ p_part, int prows,
                                                                               const int32_t *__restrict__ f_part,
                                                                               const uint8_t *__restrict__ cnt8, int cnt_ld,
                                                                               int nblocks, int T, int N, int NE, int K,
                                                                               float alpha, float w, float *__restrict__ f,
                                                                               float *__restrict__ P, float *__restrict__ summary)
{
    __shared__ f32x4 s_part[kStatsFinalThreads];
    __shared__ int s_cnt[kMaxExperts];
    __shared__ float s_f[kMaxExperts], s_P[kMaxExperts];
    const int tid = threadIdx.x, quads = (NE + 3) / 4, parts = min(min(kStatsFinalThreads / quads, kStatsParts), prows);
    const int quad = tid % quads, part = tid / quads;
    for (int e = tid; e < kMaxExperts; e += kStatsFinalThreads) s_cnt[e] = 0;
    __syncthreads();
    // of a word of counts (blocks 16 wi .. + 15): what is there
    auto clip = [&](uint4 &v, int wi) {
        auto mask = [&](int q) {
            const int left = nblocks - (wi * 16 + q * 4);
            return left >= 4 ? ~0u : left <= 0 ? 0u : (1u << (8 * left)) - 1u;
        };
        v.x &= mask(0); v.y &= mask(1); v.z &= mask(2); v.w &= mask(3);
    };
    auto add_word = [](const uint4 &v, int c) {
        c = (int)__builtin_amdgcn_sad_u8(v.x, 0u, (unsigned)c);
        c = (int)__builtin_amdgcn_sad_u8(v.y, 0u, (unsigned)c);
        c = (int)__builtin_amdgcn_sad_u8(v.z, 0u, (unsigned)c);
        return (int)__builtin_amdgcn_sad_u8(v.w, 0u, (unsigned)c);
    };
    const int words = cnt_ld / 16;
    if constexpr (LONG) {
        constexpr int WAVES = kStatsFinalThreads / 64, U = 8;
        const int lane = tid & 63;
        for (int e0 = tid >> 6; e0 < NE; e0 += WAVES * U) {
            int c[U] = {};
            for (int wi = lane; wi < words; wi += 64) {
                uint4 v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const uint4 *>(cnt8 + (size_t)min(e0 + WAVES * u, NE - 1) * cnt_ld + wi * 16);
                if (wi * 16 + 16 > nblocks) {
#pragma unroll
                    for (int u = 0; u < U; ++u) clip(v[u], wi);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) c[u] = add_word(v[u], c[u]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int all = __builtin_amdgcn_readlane(wave_scan(c[u]), 63);
                if (lane == 0 && e0 + WAVES * u < NE) s_cnt[e0 + WAVES * u] = all;
            }
        }
    }
    if (part < parts) {
        f32x4 ps = {0.f, 0.f, 0.f, 0.f};
        int fs[4] = {0, 0, 0, 0};
        const int col = quad * 4;
        if constexpr (LONG) {
            constexpr int U = 12;  // (a loop unrolled by the compiler would take what is left over one load after the other)
            for (int b0 = part; b0 < prows; b0 += parts * U) {
                f32x4 v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const f32x4 *>(p_part + (size_t)min(b0 + u * parts, prows - 1) * NE + col);
#pragma unroll
                for (int u = 0; u < U; ++u) ps += b0 + u * parts < prows ? v[u] : f32x4{0.f, 0.f, 0.f, 0.f};
            }
        } else if (NE % 4 == 0) {
#pragma unroll 8
            for (int b = part; b < prows; b += parts) {
                ps += *reinterpret_cast<const f32x4 *>(p_part + (size_t)b * NE + col);
                if (f_part) {
                    const int4 c = *reinterpret_cast<const int4 *>(f_part + (size_t)b * NE + col);
                    fs[0] += c.x; fs[1] += c.y; fs[2] += c.z; fs[3] += c.w;
                }
            }
        } else {
#pragma unroll 8
            for (int b = part; b < prows; b += parts)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const size_t at = (size_t)b * NE + min(col + q, NE - 1);  // (past NE: not used)
                    ps[q] += p_part[at];
                    if (f_part) fs[q] += f_part[at];
                }
        }
        s_part[tid] = ps;
        if (!LONG && f_part)
            for (int q = 0; q < 4; ++q)
                if (quad * 4 + q < NE) atomicAdd(&s_cnt[quad * 4 + q], fs[q]);
    }
    if (!LONG && !f_part) {
        for (int i = tid; i < NE * words; i += kStatsFinalThreads) {
            const int e = i / words, wi = i - e * words;
            uint4 v = *reinterpret_cast<const uint4 *>(cnt8 + (size_t)e * cnt_ld + wi * 16);
            clip(v, wi);
            atomicAdd(&s_cnt[e], add_word(v, 0));
        }
    }
    __syncthreads();
    if (tid < NE) {
        float ps = 0.f;
#pragma unroll LONG ? 8 : 4
        for (int q = 0; q < parts; ++q) ps += s_part[q * quads + tid / 4][tid % 4];
        s_P[tid] = ps / (float)T;
        s_f[tid] = (float)((double)s_cnt[tid] / (double)T);
        f[tid] = s_f[tid];
        P[tid] = s_P[tid];
    }
    __syncthreads();
    // the group sums: one wave, lane l the experts l, l + 64, ..., then a fixed order over the lanes
    if (tid < 64) {
        float v[5] = {0.f, 0.f, 0.f, 0.f, 0.f};  // f_E, P_E, f_Z, P_Z, sum of f P
        for (int i = tid; i < NE; i += 64) {
            v[4] += s_f[i] * s_P[i];
            v[i < N ? 0 : 2] += s_f[i];
            v[i < N ? 1 : 3] += s_P[i];
        }
#pragma unroll
        for (int q = 0; q < 5; ++q) v[q] = wave_sum(v[q]);
        if (tid == 0) {
            const float fE = v[0], PE = v[1], fZ = v[2], PZ = v[3];
            const int Z = NE - N;
            summary[0] = fE; summary[1] = PE; summary[2] = fZ; summary[3] = PZ;
            summary[4] = fZ / (float)K;
            summary[5] = alpha * (float)NE / (float)K * v[4];                                  // Eq. 4
            summary[6] = alpha * ((float)N + (float)Z * w) / (float)K *
                         (fE * PE / (float)N + (Z > 0 ? fZ * PZ / ((float)Z * w) : 0.f));       // Eq. 5-6
        }
    }
}

// scratch: the logit tables, then the per-block sums (sizes are part of the interface, see route_ws_bytes)
static size_t stats_logits_bytes(const zeda_layer_desc *d)
{
    const size_t Tpad = (size_t)ceil_div(d->T, 32) * 32;
    return align_up(Tpad * ceil_div(d->N + d->Z, 32) * 32 * sizeof(float), 256);
}
size_t routing_stats_ws_bytes(const zeda_layer_desc *d)
{
    const size_t NE = (size_t)(d->N + d->Z);
    if (d->dtype == ZEDA_BF16)  // split-k scratch of the router, per-block counts, per-block probability sums
        return align_up(route_ws_bytes(d), 256) + route_counts_bytes(d) + align_up((size_t)ceil_div(d->T, 16) * NE * 4, 256);
    const size_t nblk = (size_t)ceil_div(d->T, kStatsTokens);
    return stats_logits_bytes(d) + align_up(nblk * NE * 4, 256) * 2;
}

int launch_routing_stats(const zeda_layer_desc *d, const void *x, const void *wr, const float *bias, float alpha, float w,
                         float *f, float *P, float *summary, void *ws, hipStream_t s)
{
    const int NE = d->N + d->Z;
    if (d->dtype == ZEDA_BF16) {
        float *partial = route_ws_bytes(d) ? (float *)ws : nullptr;
        uint8_t *cnt8 = (uint8_t *)ws + align_up(route_ws_bytes(d), 256);
        float *p_part = (float *)(cnt8 + route_counts_bytes(d));
        const RouteExtras ex = {cnt8, route_counts_ld(d), p_part, {}, nullptr};
        const RoutePlan plan = route_plan(d, partial != nullptr);
        const int prows = ceil_div(d->T, plan.slices > 1 ? kSelectTokens : 16 * plan.tb);  // workgroups that select
        const int rc = launch_route_bf16_any(d, x, wr, bias, nullptr, nullptr, partial, ex, s);
        if (rc != ZEDA_OK) return rc;
        const auto kernel = stats_long(ex.cnt_ld, NE) ? route_stats_final_kernel<true> : route_stats_final_kernel<false>;
        kernel<<<1, kStatsFinalThreads, 0, s>>>(p_part, prows, nullptr, cnt8, ex.cnt_ld, ceil_div(d->T, 16), d->T, d->N, NE, d->K, alpha, w, f, P, summary);
        return last_launch_status();
    }
    const int NB = ceil_div(NE, 32), LDg = NB * 32;
    const int Tpad = ceil_div(d->T, kRouteF32Tokens) * kRouteF32Tokens, nblk = ceil_div(d->T, kStatsTokens);
    float *logits = (float *)ws;
    float *p_part = (float *)((char *)ws + stats_logits_bytes(d));
    int32_t *f_part = (int32_t *)((char *)p_part + align_up((size_t)nblk * NE * 4, 256));
    if (launch_route_f32(d, x, wr, bias, nullptr, nullptr, logits, LDg, s) != ZEDA_OK) return ZEDA_EHIP;
#define ZEDA_STATS(NC) route_stats_kernel<NC><<<nblk, kStatsThreads, 0, s>>>(logits, 1, Tpad, LDg, bias, d->T, NE, d->K, p_part, f_part)
    switch (ceil_div(NE, 16)) {
        case 1: ZEDA_STATS(1); break;   case 2: ZEDA_STATS(2); break;   case 3: ZEDA_STATS(3); break;
        case 4: ZEDA_STATS(4); break;   case 5: ZEDA_STATS(5); break;   case 6: ZEDA_STATS(6); break;
        case 7: ZEDA_STATS(7); break;   case 8: ZEDA_STATS(8); break;   case 9: ZEDA_STATS(9); break;
        case 10: ZEDA_STATS(10); break; case 11: ZEDA_STATS(11); break; case 12: ZEDA_STATS(12); break;
        case 13: ZEDA_STATS(13); break; case 14: ZEDA_STATS(14); break; case 15: ZEDA_STATS(15); break;
        default: ZEDA_STATS(16); break;
    }
#undef ZEDA_STATS
    if (hipGetLastError() != hipSuccess) return ZEDA_EHIP;
    route_stats_final_kernel<false><<<1, kStatsFinalThreads, 0, s>>>(p_part, nblk, f_part, nullptr, 0, nblk, d->T, d->N, NE, d->K, alpha, w, f, P,
                                                         summary);
    return last_launch_status();
}

int launch_route(const zeda_layer_desc *d, const void *x, const void *wr, const float *bias, int32_t *ids, float *gates,
                 float *partial, uint8_t *cnt8, const PlaceOut *place, TilePlace *tp, hipStream_t s)
{
    if (d->dtype == ZEDA_BF16) {
        const RouteExtras ex = {cnt8, cnt8 ? route_counts_ld(d) : 0, nullptr, place ? *place : PlaceOut{}, tp};
        return launch_route_bf16_any(d, x, wr, bias, ids, gates, partial, ex, s);
    }
    return launch_route_f32(d, x, wr, bias, ids, gates, nullptr, 0, s);
}

}  // namespace zeda
