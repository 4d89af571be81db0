// Top-K selection and routing weights of one token from its logits (Section 2.1, Section 4.3.4), by rows of 16 lanes or by
// whole waves.
#pragma once
#include <limits.h>

#include "zeda_internal.h"

namespace zeda {

// Selection runs four tokens per wave, one per row of 16 lanes (the unit of the VALU's data-parallel-primitive
// cross-lane path), so all reductions stay inside a row and need no LDS traffic and no scalar round trips.
// row_ror rotates a value inside its row; max/min folded over rotations by 8, 4, 2, 1 leave every lane of the
// row with the row's result, and since max and min do not depend on the order all lanes agree exactly.
template <int N>
__device__ __forceinline__ int dpp_row_ror(int v)
{
    return __builtin_amdgcn_mov_dpp(v, 0x120 + N, 0xf, 0xf, true);
}
__device__ __forceinline__ int row_max(int v)
{
    v = max(v, dpp_row_ror<8>(v));
    v = max(v, dpp_row_ror<4>(v));
    v = max(v, dpp_row_ror<2>(v));
    v = max(v, dpp_row_ror<1>(v));
    return v;
}
__device__ __forceinline__ float row_max(float v)
{
    v = fmaxf(v, __int_as_float(dpp_row_ror<8>(__float_as_int(v))));
    v = fmaxf(v, __int_as_float(dpp_row_ror<4>(__float_as_int(v))));
    v = fmaxf(v, __int_as_float(dpp_row_ror<2>(__float_as_int(v))));
    v = fmaxf(v, __int_as_float(dpp_row_ror<1>(__float_as_int(v))));
    return v;
}
__device__ __forceinline__ int row_min(int v)
{
    v = min(v, dpp_row_ror<8>(v));
    v = min(v, dpp_row_ror<4>(v));
    v = min(v, dpp_row_ror<2>(v));
    v = min(v, dpp_row_ror<1>(v));
    return v;
}
// Integers in the order of the floats (both zeros alike; no-numbers come last, as kNoKey): one max instruction takes the
// lane permutation along, where a float max first quiets its operands.
constexpr int kNoKey = INT_MIN;
__device__ __forceinline__ int logit_key(float v)
{
    const int b = __float_as_int(v + 0.0f);  // -0 -> +0
    return v == v ? b ^ ((b >> 31) & 0x7fffffff) : kNoKey;
}
__device__ __forceinline__ float key_logit(int k) { return __int_as_float(k ^ ((k >> 31) & 0x7fffffff)); }
// Sum over the row in one fixed order (an inclusive scan with row_shr 1, 2, 4, 8 leaves the total in the row's
// last lane), handed to every lane of the row, so that all lanes divide by the same number.
__device__ __forceinline__ float row_sum(float v)
{
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x111, 0xf, 0xf, false));  // lanes without a source add zero
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x112, 0xf, 0xf, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x114, 0xf, 0xf, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x118, 0xf, 0xf, false));
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 15));
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 31));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 47));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
    const int r = (threadIdx.x & 63) >> 4;
    return r == 0 ? r0 : r == 1 ? r1 : r == 2 ? r2 : r3;
}

// Sum over all 64 lanes in a fixed order, returned to every lane.
__device__ __forceinline__ float wave_sum(float v)
{
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x111, 0xf, 0xf, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x112, 0xf, 0xf, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x114, 0xf, 0xf, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x118, 0xf, 0xf, false));
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 15));
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 31));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 47));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
    return (r0 + r1) + (r2 + r3);
}

// Selection and gates for the four tokens tk0..tk0+3 of the workgroup's block (whose fp32 logits are rows of
// lg in LDS), executed by one wave: token tk0 + r belongs to lane row r, and lane l of the row holds the
// candidates l, l + 16, ... (NC of them).  One round: the row maximum, then the lowest expert index among the
// candidates equal to it (ties go to the lower index), which its owner then removes.  Lane j of the row keeps
// slot j, so lanes 0..K-1 end up with the slots in descending-logit order (K <= 16).
// Returns the expert of the slot this lane keeps (lane j < K of a row: slot j of the row's token), or -1.
// bias: this lane's candidates' biases.
// probs (may be NULL): an LDS table [token][LDP] that receives, for every token of the wave, the routing
// probability of every expert (softmax over all NE logits).
template <int NC, int NP>
__device__ __forceinline__ int select_rows(const float *lg, int LD, int pstride, const float (&bias)[NC], int tk0,
                                           int ntok, int t0, int T, int NE, int N, int K, int gate_norm,
                                           int32_t *__restrict__ ids, float *__restrict__ gates, float *probs = nullptr,
                                           int LDP = 0)
{
    const int lane = threadIdx.x & 63, l16 = lane & 15, tk = tk0 + (lane >> 4);
    const bool ok = tk < ntok && t0 + tk < T;
    int cand[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int e = l16 + 16 * c;
        // the NP partial sums over slices of the hidden dimension, added in a fixed order, then the bias (columns past
        // NE of the tables are readable and left out)
        float v = lg[tk * LD + e];
#pragma unroll
        for (int q = 1; q < NP; ++q) v += lg[q * pstride + tk * LD + e];
        int key = logit_key(v + bias[c]);
        asm volatile("" : "+v"(key));  // (no branch around every candidate)
        cand[c] = ok && e < NE ? key : kNoKey;
    }
    auto local_max = [&]() {
        int m = cand[0];
#pragma unroll
        for (int c = 1; c < NC; ++c) m = max(m, cand[c]);
        return m;
    };
    int m = row_max(local_max());
    const float all_max = key_logit(m);
    float all_sum = 0.f;
    if (gate_norm == ZEDA_GATE_SOFTMAX || probs) {
        float ex[NC], sacc = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            ex[c] = (ok && l16 + 16 * c < NE) ? expf(key_logit(cand[c]) - all_max) : 0.f;
            sacc += ex[c];
        }
        all_sum = row_sum(sacc);
        if (probs && ok) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (l16 + 16 * c < NE) probs[tk * LDP + l16 + 16 * c] = ex[c] / all_sum;
        }
    }
    int my_id = 0;
    float my_logit = -INFINITY;
    for (int j = 0; j < K; ++j) {
        if (j > 0) m = row_max(local_max());
        int mine = INT_MAX;
#pragma unroll
        for (int c = NC - 1; c >= 0; --c)
            if (cand[c] == m) mine = l16 + 16 * c;  // descending c: the lowest index survives
        int win = row_min(mine);
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (win == l16 + 16 * c) cand[c] = kNoKey;
        if (m == kNoKey) win = INT_MAX;  // nothing but no-numbers left: no expert, gate 0
        if (l16 == j) { my_id = win; my_logit = m == kNoKey ? -INFINITY : key_logit(m); }
    }
    const bool slot = l16 < K;
    const float ex = slot ? expf(my_logit - all_max) : 0.f;
    float dn;
    if (gate_norm == ZEDA_GATE_SOFTMAX) dn = all_sum;
    else if (gate_norm == ZEDA_GATE_TOPK_NORM) dn = row_sum(ex);
    else dn = row_sum((slot && my_id < N) ? ex : 0.f);
    if (slot && ok && ids) {
        const size_t o = (size_t)(t0 + tk) * K + l16;
        ids[o] = my_id;
        gates[o] = dn > 0.f ? ex / dn : 0.f;
    }
    return (slot && ok) ? my_id : -1;
}

// The same for one token by a whole wave: lane l holds the candidates l, l + 64, ...; a round's winner is found from
// ballots, lowest candidate group and lane first, i.e. the lowest index.  Shorter rounds than the above (few
// candidates per lane): for workgroups with a wave for every token.  lg: the token's logits, biases included.
// by_rows (NE <= 64): the softmax denominator is added in the order of select_rows; everything else does not depend on an order.
template <int NC>
__device__ __forceinline__ int select_wave(const float *lg, bool ok, size_t t, int NE, int N, int K, int gate_norm,
                                           int32_t *__restrict__ ids, float *__restrict__ gates, float *probs = nullptr,
                                           bool by_rows = false)
{
    const int lane = threadIdx.x & 63;
    int cand[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int e = lane + 64 * c;
        int key = logit_key(lg[e]);
        asm volatile("" : "+v"(key));
        cand[c] = ok && e < NE ? key : kNoKey;
    }
    auto wave_max = [&]() {
        int m = cand[0];
#pragma unroll
        for (int c = 1; c < NC; ++c) m = max(m, cand[c]);
        m = row_max(m);
        return max(max(__builtin_amdgcn_readlane(m, 0), __builtin_amdgcn_readlane(m, 16)),
                   max(__builtin_amdgcn_readlane(m, 32), __builtin_amdgcn_readlane(m, 48)));
    };
    int m = wave_max();
    const float all_max = key_logit(m);
    float all_sum = 0.f;
    if (gate_norm == ZEDA_GATE_SOFTMAX || probs) {
        float ex[NC], sacc = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            ex[c] = (ok && lane + 64 * c < NE) ? expf(key_logit(cand[c]) - all_max) : 0.f;
            sacc += ex[c];
        }
        if (by_rows) {
            sacc = 0.f;
#pragma unroll
            for (int c = 0; c < 4; ++c) sacc += __shfl(ex[0], (lane & 15) + 16 * c);
            all_sum = row_sum(sacc);
        } else {
            all_sum = wave_sum(sacc);
        }
        if (probs && ok) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (lane + 64 * c < NE) probs[lane + 64 * c] = ex[c] / all_sum;
        }
    }
    int my_id = 0;
    float my_logit = -INFINITY;
    for (int j = 0; j < K; ++j) {
        if (j > 0) m = wave_max();
        int win = INT_MAX;
#pragma unroll
        for (int c = NC - 1; c >= 0; --c) {
            const unsigned long long eq = __ballot(cand[c] == m);
            if (eq) win = 64 * c + __ffsll((long long)eq) - 1;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (win == lane + 64 * c) cand[c] = kNoKey;
        if (m == kNoKey) win = INT_MAX;  // nothing but no-numbers left: no expert, gate 0
        if (lane == j) { my_id = win; my_logit = m == kNoKey ? -INFINITY : key_logit(m); }
    }
    const bool slot = lane < K;
    const float ex = slot ? expf(my_logit - all_max) : 0.f;
    float dn;
    if (gate_norm == ZEDA_GATE_SOFTMAX) dn = all_sum;
    else if (gate_norm == ZEDA_GATE_TOPK_NORM) dn = row_sum(ex);
    else dn = row_sum((slot && my_id < N) ? ex : 0.f);
    if (slot && ok && ids) {
        ids[t * K + lane] = my_id;
        gates[t * K + lane] = dn > 0.f ? ex / dn : 0.f;
    }
    return (slot && ok) ? my_id : -1;
}

}  // namespace zeda
