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

// Inclusive sum over the lanes of a wave.
__device__ __forceinline__ int wave_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr 1, 2, 4, 8: inside rows of 16 lanes
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // a row's total to the next row
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // the first half's total to the second
    return v;
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
    const int incl = wave_scan(local);
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

// Short slot lists are placed by the gate/up kernels themselves: every workgroup counts the experts' slots, finds the expert of
// its token tile and collects the tile's slots; what the later kernels read is written by the workgroups of the first feature
// tile.  Instead of a launch of 4 to 5 us that is half a microsecond or more of every workgroup (gateup_places: for how many it
// pays).  Whole layer, with the launch / without: T=64, H=256, I=128, N=8, K=2, fp32 22.9 / 18.3 us; N=24, I=448, 300 tokens
// (900 slots) 39.7 / 36.6; N=128, I=768, 64 tokens (512 slots, 6900 workgroups) 175.3 / 173.8.
constexpr int kTileThreads = 256;
constexpr int kTileMaxSlots = 4 * kTileThreads;

// What such a kernel starts from and writes: the ids of all slots, or the logits of up to kTileSelTokens tokens, left by the router's
// first kernel in `slices` tables [Tpad][E], from which it selects (by_rows: the router's second kernel would do so with four waves).
constexpr int kTileSelTokens = 4;
struct TilePlace {
    int32_t *ids;
    PlaceOut out;
    float *gates;
    const float *partial, *bias;
    int slices, Tpad, E, NE, gate_norm;
    bool by_rows;
};

template <int ROWS>
struct TilePlaceLds {
    alignas(16) int hist[kMaxExperts];  // slots on every expert (read four at a time)
    int cnt[kTileMaxSlots / 64];        // slots of every 64-slot group on the tile's expert
    int list[ROWS];                     // the tile's slots, ascending
};

// As locate_rows, from the S <= kTileMaxSlots slots whose ids id_of(slot) returns; by a workgroup of kTileThreads threads.  first:
// this workgroup writes the tile's rows of o's tables; lead: also what belongs to no tile.
template <int ROWS, typename IdOf>
__device__ __forceinline__ int4 place_tile(const IdOf &id_of, int S, int N, int tile, bool first, bool lead, TilePlaceLds<ROWS> &s, const PlaceOut &o)
{
    static_assert(kTileThreads == kMaxExperts, "one thread per expert");
    static_assert(alignof(TilePlaceLds<ROWS>) == alignof(int4), "hist is read in 16-byte pieces");
    constexpr int G = kTileMaxSlots / kTileThreads, W = kTileThreads / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int id[G];
#pragma unroll
    for (int i = 0; i < G; ++i) id[i] = tid + kTileThreads * i < S ? id_of(tid + kTileThreads * i) : -1;
    s.hist[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < G; ++i)
        if ((unsigned)id[i] < (unsigned)N) atomicAdd(&s.hist[id[i]], 1);
    __syncthreads();
    // lane l: experts 4l .. 4l + 3; rows in the low half (at most 1024), token tiles in the high one
    const int4 c4 = *reinterpret_cast<const int4 *>(&s.hist[4 * lane]);
    const int c[4] = {c4.x, c4.y, c4.z, c4.w};
    int nt[4], local = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        nt[q] = (c[q] + ROWS - 1) / ROWS;
        local += (nt[q] << 16) + c[q];
    }
    const int incl = wave_scan(local), all = __builtin_amdgcn_readlane(incl, 63);
    int row = (incl - local) & 0xffff, first_tile = (incl - local) >> 16;
    if (lead) {
        if (wave == 0) {
            int at = row;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (4 * lane + q < N) o.offsets[4 * lane + q] = at;
                at += c[q];
            }
            if (lane == 0) {
                o.offsets[N] = o.num_real[0] = all & 0xffff;
                if (o.num_real_copy) o.num_real_copy[0] = all & 0xffff;
            }
        }
#pragma unroll
        for (int i = 0; i < G; ++i)
            if (tid + kTileThreads * i < S && (unsigned)id[i] >= (unsigned)N) o.slot_to_row[tid + kTileThreads * i] = -1;
    }
    if (tile >= all >> 16) return make_int4(0, 0, 0, 0);
    int e = 0, row0 = 0, rows = 0, mine = 0, skip = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (tile >= first_tile && tile < first_tile + nt[q]) {
            e = 4 * lane + q;
            skip = (tile - first_tile) * ROWS;  // the expert's rows in the tiles before
            row0 = row + skip;
            rows = min(ROWS, c[q] - skip);
            mine = c[q];
        }
        first_tile += nt[q];
        row += c[q];
    }
    const int src = __ffsll((long long)__ballot(rows > 0)) - 1;
    e = __builtin_amdgcn_readlane(e, src);
    row0 = __builtin_amdgcn_readlane(row0, src);
    rows = __builtin_amdgcn_readlane(rows, src);
    mine = __builtin_amdgcn_readlane(mine, src);
    skip = __builtin_amdgcn_readlane(skip, src);
    unsigned long long m[G];
#pragma unroll
    for (int i = 0; i < G; ++i) {
        m[i] = __ballot(id[i] == e);
        if (lane == 0) s.cnt[W * i + wave] = __popcll(m[i]);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < G; ++i) {
        if (!m[i]) continue;
        int at = __popcll(m[i] & ((1ull << lane) - 1ull)) - skip;
        for (int g = 0; g < W * i + wave; ++g) at += s.cnt[g];
        if (id[i] == e && at >= 0 && at < rows) s.list[at] = tid + kTileThreads * i;
    }
    __syncthreads();
    if (first && tid < rows) {
        const int slot = s.list[tid];
        o.sorted_slot[row0 + tid] = slot;
        o.slot_to_row[slot] = row0 + tid;
    }
    return make_int4(e, row0, rows, mine);
}

}  // namespace zeda
