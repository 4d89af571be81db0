// Expert-sorted placement of a short slot list by one workgroup (Section 2.1: slots on zero experts are dropped), and the
// way back from a tile of the sorted rows to its expert.
#pragma once
#include "zeda_internal.h"

namespace zeda {

// lanes of the wave whose slot is on the same normal expert as this lane's (0 for a lane that is on none)
__device__ __forceinline__ unsigned long long same_expert_lanes(int id, bool real)
{
    unsigned long long m = __ballot(real);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const unsigned long long bb = __ballot((id >> b) & 1);
        m &= ((id >> b) & 1) ? bb : ~bb;
    }
    return real ? m : 0ull;
}

// Where a placement goes (see zeda_dispatch for the meaning of the tables).
struct PlaceOut {
    int32_t *offsets, *sorted_slot, *slot_to_row, *num_real, *num_real_copy;
};

// LDS of place_list for at most SLOTS slots
template <int SLOTS>
struct PlaceLds {
    int cnt[SLOTS / 64][kMaxExperts];  // slots of wave w's group on every expert, then the running rows
    int first[kMaxExperts];
    int wsum[kMaxExperts / 64];
};

// The S <= SLOTS slots of s_ids (LDS), one group of 64 per wave, by a workgroup of THREADS threads that has met since s_ids
// was written.  Stable: ascending slot index inside an expert.
template <int THREADS, int SLOTS>
__device__ __forceinline__ void place_list(const int *s_ids, int S, int N, PlaceLds<SLOTS> &s, const PlaceOut &o)
{
    static_assert(THREADS >= SLOTS && SLOTS % 64 == 0 && THREADS >= kMaxExperts, "one wave per group, one thread per expert");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, groups = (S + 63) / 64;
    for (int i = tid; i < groups * kMaxExperts; i += THREADS) (&s.cnt[0][0])[i] = 0;
    __syncthreads();
    const int slot = tid;
    const bool in = slot < S;
    const int id = in ? s_ids[slot] : -1;
    const bool real = (unsigned)id < (unsigned)N;
    const unsigned long long m = same_expert_lanes(id, real);
    const int rank = __popcll(m & ((1ull << lane) - 1ull));
    if (real && rank == 0) s.cnt[wave][id] = __popcll(m);
    __syncthreads();
    int total = 0;
    if (tid < kMaxExperts) {
        for (int w = 0; w < groups; ++w) total += s.cnt[w][tid];
        int incl = total;
#pragma unroll
        for (int sh = 1; sh < 64; sh <<= 1) {
            const int v = __shfl_up(incl, sh);
            if (lane >= sh) incl += v;
        }
        if (lane == 63) s.wsum[wave] = incl;
        s.first[tid] = incl - total;
    }
    __syncthreads();
    if (tid < kMaxExperts) {
        int row = s.first[tid];
        for (int w = 0; w < wave; ++w) row += s.wsum[w];
        if (tid < N) o.offsets[tid] = row;
        if (tid == N - 1) {
            o.offsets[N] = row + total;
            o.num_real[0] = row + total;
            if (o.num_real_copy) o.num_real_copy[0] = row + total;
        }
        for (int w = 0; w < groups; ++w) {
            const int c = s.cnt[w][tid];
            s.cnt[w][tid] = row;
            row += c;
        }
    }
    __syncthreads();
    if (real) {
        const int r = s.cnt[wave][id] + rank;
        o.sorted_slot[r] = slot;
        o.slot_to_row[slot] = r;
    } else if (in) {
        o.slot_to_row[slot] = -1;
    }
}

// Token tile `tile` of the expert-sorted rows, ROWS rows to a tile: {expert, first row, rows, rows of the expert}, rows = 0
// past the last tile.  By a whole wave (lane l holds experts 4l..4l+3); the same for all lanes.
template <int ROWS>
__device__ __forceinline__ int4 locate_rows(const int32_t *__restrict__ offsets, int N, int tile)
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
    int excl = incl - local, e = 0, row0 = 0, rows = 0, all = 0;
    const unsigned long long mine = __ballot(tile >= excl && tile < incl);
    if (mine == 0) return make_int4(0, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (tile >= excl && tile < excl + nt[q]) {
            e = 4 * lane + q;
            row0 = off[q] + (tile - excl) * ROWS;
            all = off[q + 1] - off[q];
            rows = min(ROWS, off[q + 1] - row0);
        }
        excl += nt[q];
    }
    const int src = __ffsll((long long)mine) - 1;
    return make_int4(__builtin_amdgcn_readlane(e, src), __builtin_amdgcn_readlane(row0, src), __builtin_amdgcn_readlane(rows, src),
                     __builtin_amdgcn_readlane(all, src));
}

}  // namespace zeda
