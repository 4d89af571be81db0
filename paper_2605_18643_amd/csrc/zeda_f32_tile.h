// Building block of the fp32 kernels: a wave multiplies NA blocks of 16 weight rows with NB blocks of 16 token rows on the
// fp32 matrix instruction (16x16x4, IEEE fp32 products and sums), operands straight from global memory.
//
// A lane loads 16 bytes - four consecutive k of one row: lane l holds row l % 16, k = 4 (l / 16) .. + 3 of a 16-wide step -
// and the four matrix instructions of the step take one component each, so that the k of one instruction are 4 apart;
// both operands are permuted alike, so the sum runs over all of them.  Two steps cover the 128 bytes of a cache line.
//
// The fp32 layers are small (their weights are streamed once, an expert has tens of rows), so what bounds the kernels is
// loads in flight and the number of waves, not the matrix units: the hidden dimension of one output tile is split over the
// waves of a workgroup, each keeps the loads of the next 32 k in flight, and nothing goes through LDS but the waves' sums.
//
// Precision: the 32 products of a chunk are added as four sums of eight in the matrix unit and a tree over the four; chunk
// sums and the FFN's slices are added in 64 bits and rounded once, so that the error is the chunks' own, however many there
// are.  (Sums of sixteen per chunk and a plain sum over the slices end farther from the 64-bit result than the sums over 64
// lanes that these kernels replaced.  A compensated fp32 sum that is exact whichever summand is the larger one takes six
// additions where this takes a conversion and an addition: 6 % more of the FFN, 2 % of the router.)
#pragma once
#include "zeda_internal.h"

namespace zeda {

typedef double f64x2 __attribute__((ext_vector_type(2)));

template <int NA, int NB>
struct F32Tile {
    f64x2 acc[NA][NB][2];

    struct Frags {
        f32x4 a[2][NA], b[2][NB];
    };

    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[a][b][0] = acc[a][b][1] = f64x2{0., 0.};
    }
    // pa, pb: this lane's rows (at k = 0); the 32 k from k0 on.  Past Kd (a multiple of 4) the rows' first values stand in
    // until mask() clears them: a select here would wait for the loads where they are issued
    __device__ __forceinline__ static void load(Frags &f, const float *const (&pa)[NA], const float *const (&pb)[NB], int k0, int Kd)
    {
        const int kl = k0 + 4 * ((threadIdx.x & 63) >> 4);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int k = kl + 16 * s, kc = k < Kd ? k : 0;
#pragma unroll
            for (int a = 0; a < NA; ++a) f.a[s][a] = *reinterpret_cast<const f32x4 *>(pa[a] + kc);
#pragma unroll
            for (int b = 0; b < NB; ++b) f.b[s][b] = *reinterpret_cast<const f32x4 *>(pb[b] + kc);
        }
    }
    // zero both operands past Kd in the chunk at k0
    __device__ __forceinline__ static void mask(Frags &f, int k0, int Kd)
    {
        if (k0 + 32 <= Kd) return;
        const int kl = k0 + 4 * ((threadIdx.x & 63) >> 4);
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const bool in = kl + 16 * s < Kd;
#pragma unroll
            for (int a = 0; a < NA; ++a) f.a[s][a] = in ? f.a[s][a] : zero;
#pragma unroll
            for (int b = 0; b < NB; ++b) f.b[s][b] = in ? f.b[s][b] : zero;
        }
    }
    __device__ __forceinline__ static void fold(f64x2 (&sm)[2], const f32x4 (&c)[4])
    {
        const f32x4 v = (c[0] + c[1]) + (c[2] + c[3]);
#pragma unroll
        for (int q = 0; q < 4; ++q) sm[q >> 1][q & 1] += (double)v[q];
    }
    // (the scheduling barriers keep the compiler from starting all blocks at once, which costs more registers than there
    // are; a block's sums are folded while the next block's products run)
    __device__ __forceinline__ void multiply(const Frags &f)
    {
        f32x4 c[2][4];
#pragma unroll
        for (int i = 0; i < NA * NB; ++i) {
            const int a = i / NB, b = i % NB;
#pragma unroll
            for (int h = 0; h < 4; ++h) c[i & 1][h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int h = 0; h < 4; ++h)
                    c[i & 1][h] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.a[h >> 1][a][2 * (h & 1) + q], f.b[h >> 1][b][2 * (h & 1) + q],
                                                                       c[i & 1][h], 0, 0, 0);
            if (i > 0) fold(acc[(i - 1) / NB][(i - 1) % NB], c[(i & 1) ^ 1]);
            __builtin_amdgcn_sched_barrier(0);
        }
        fold(acc[NA - 1][NB - 1], c[(NA * NB - 1) & 1]);
    }
    // a block's sums, rounded
    __device__ __forceinline__ f32x4 total(int a, int b) const
    {
        f32x4 v;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = (float)acc[a][b][q >> 1][q & 1];
        return v;
    }
    // slice `slice` of `slices`: the 32-wide chunks slice, slice + slices, ..., starting at one that depends on rot (rows
    // are often a multiple of 4 KiB apart, which puts a chunk of every row on one L2 channel: workgroups that start at
    // different chunks spread over the channels)
    __device__ __forceinline__ void run(const float *const (&pa)[NA], const float *const (&pb)[NB], int slice, int slices, int rot,
                                        int Kd)
    {
        clear();
        const int n = ((Kd + 31) / 32 - slice + slices - 1) / slices, step = 32 * slices, end = 32 * slice + n * step;
        if (n <= 0) return;
        int k0 = 32 * slice + (int)((unsigned)rot % (unsigned)n) * step;
        Frags cur, nxt;
        load(cur, pa, pb, k0, Kd);
        for (int i = 1; i < n; ++i) {
            const int k1 = k0 + step < end ? k0 + step : 32 * slice;
            load(nxt, pa, pb, k1, Kd);
            mask(cur, k0, Kd);
            multiply(cur);
            cur = nxt;
            k0 = k1;
        }
        mask(cur, k0, Kd);
        multiply(cur);
    }
};

}  // namespace zeda
