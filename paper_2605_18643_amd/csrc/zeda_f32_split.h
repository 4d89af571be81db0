// Building block of the fp32 expert FFN: a wave multiplies NA blocks of 16 weight rows with NB blocks of 16 token rows on the
// bf16 matrix instruction, every fp32 number as the sum of three bf16 numbers, operands through a ring of its own in LDS.
//
// Why not the fp32 instruction: it runs at the rate of the vector unit and keeps vector instructions out while it does (16x16x4
// in a register-only loop, two waves per SIMD: 32 cycles each, 59 with the 20 vector instructions between every eight that add
// the sums up).  x = hi + mid + lo is exact with each part rounded to nearest; of the nine products of parts six matter, the
// other three are below 2^-26 of the product.  Six 16x16x32 take 96 cycles of the matrix unit where eight 16x16x4 take 256, and
// the vector unit is free for the splitting (44 instructions per 16 x 32 block of an operand).
//
// A lane's fragments are two pieces of four consecutive k of one row: lane l holds row l % 16, pieces l / 16 and 4 + l / 16 of
// the 32 k; both operands are permuted alike, so the sum runs over all of them.
//
// Precision: the products of a chunk of 32 k are added in the matrix unit, smallest parts first; chunk sums and the slices of the
// waves are added in 64 bits and rounded once.  Error against 64 bits, 2-norm, whole layer: T=513, H=1024, I=512 1.46e-7 (four sums of
// eight products on the fp32 instruction and a tree over them: 1.60e-7).
//
// Magnitudes that round to a bf16 infinity have no such sum: rows with one are reported, and the caller computes what depends
// on them in another way.
#pragma once
#include "zeda_wave_ring.h"

namespace zeda {

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr float kSplitMax = 3.38e38f;  // (the largest bf16 is 3.3895e38)

// D: blocks that the wave keeps in flight
template <int NA, int NB, int D>
struct F32Split {
    static constexpr int SEQ = NB + NA;  // blocks of a chunk of 32 k: token rows first
    f64x2 acc[NA][NB][2];

    struct Parts {
        bf16x8 hi, mid, lo;
    };

    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[a][b][0] = acc[a][b][1] = f64x2{0., 0.};
    }
    // zero what lies past the row's `left` bytes in the fragments of the chunk
    __device__ __forceinline__ static void mask(u32x4 (&f)[2], uint32_t left)
    {
        if (left >= 128) return;
        const uint32_t at = ((threadIdx.x & 63) >> 4) * 16;
#pragma unroll
        for (int s = 0; s < 2; ++s) f[s] = at + 64 * s < left ? f[s] : u32x4{0u, 0u, 0u, 0u};
    }
    __device__ __forceinline__ static void fold(f64x2 (&sm)[2], const f32x4 &v)
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) sm[q >> 1][q & 1] += (double)v[q];
        asm volatile("" : "+v"(sm[0]), "+v"(sm[1]));  // (here, not for all blocks at the chunk's end: registers)
    }
    // eight elements a lane.  huge: whether one of them is past kSplitMax
    __device__ __forceinline__ static Parts split(const u32x4 (&f)[2], bool &huge)
    {
        u32x4 part[3];
        float largest = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v0 = __uint_as_float(f[i >> 1][2 * (i & 1)]), v1 = __uint_as_float(f[i >> 1][2 * (i & 1) + 1]);
            largest = fmaxf(fmaxf(fabsf(v0), fabsf(v1)), largest);
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const uint32_t two = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){v0, v1}, bf16x2));
                part[p][i] = two;
                v0 -= __uint_as_float(two << 16);
                v1 -= __uint_as_float(two & 0xffff0000u);
            }
        }
        huge = largest > kSplitMax;
        return {__builtin_bit_cast(bf16x8, part[0]), __builtin_bit_cast(bf16x8, part[1]), __builtin_bit_cast(bf16x8, part[2])};
    }

    // lds: this wave's ring.  The rows of weight block a start at base[a % 2] + wo[a][.] bytes, those of token block b at pb[b][.]
    // ([0]: row lane / 8 of the block, [1]: row 8 + lane / 8).  Kd: a multiple of 4.  huge_tok, huge_w: LDS addresses of 16 NB and 16 NA
    // bytes, zeroed by the caller, that receive ones for rows with an element past kSplitMax.
    // Slice `slice` of `slices`: the 32-wide chunks slice, slice + slices, ..., starting at one that depends on rot (rows
    // are often a multiple of 4 KiB apart, which puts a chunk of every row on one L2 channel: workgroups that start at
    // different chunks spread over the channels)
    __device__ __forceinline__ void run(uint32_t lds, const float *base0, const float *base1, const uint32_t (&wo)[NA][2],
                                        const float *const (&pb)[NB][2], uint32_t huge_tok, uint32_t huge_w, int slice, int slices, int rot,
                                        int Kd)
    {
        clear();
        const int n = ((Kd + 31) / 32 - slice + slices - 1) / slices;
        if (n <= 0) return;
        const int first = (int)((unsigned)rot % (unsigned)n), total = n * SEQ, l16 = threadIdx.x & 15;
        const uint32_t rowb = (uint32_t)Kd * 4;
        WaveRing<D> ring;
        ring.init(lds);
        auto col = [&](int c) { const int q = c + first; return (uint32_t)(slice + (q >= n ? q - n : q) * slices) * 128u; };
        // (pieces past the end of a row repeat its last one, until mask() clears them)
        auto fetch = [&](int j, uint32_t at) {
            const uint32_t o0 = min(at + WaveRing<D>::piece0(), rowb - 16), o1 = min(at + WaveRing<D>::piece1(), rowb - 16);
            if (j < NB) {
                const float *const *p = pb[j < NB ? j : 0];
                ring.fetch(reinterpret_cast<const char *>(p[0]) + o0, reinterpret_cast<const char *>(p[1]) + o1);
            } else {
                const int a = j < NB ? 0 : j - NB;
                const char *w = reinterpret_cast<const char *>(a & 1 ? base1 : base0);
                ring.fetch(w + (wo[a][0] + o0), w + (wo[a][1] + o1));
            }
        };
#pragma unroll
        for (int i = 0; i < D; ++i)
            if (i < total) fetch(i % SEQ, col(i / SEQ));
        Parts tb[NB];
        for (int k = 0; k < n; ++k) {
            const int i0 = k * SEQ;
            uint32_t at[D / SEQ + 2];
#pragma unroll
            for (int u = 0; u < D / SEQ + 2; ++u) at[u] = col(min(k + u, n - 1));
            // A block's fragments are read while the block before is multiplied.  (No branch lies between a read and its wait: the
            // compiler could copy the registers there, before the data is in them.)
            u32x4 cur[2];
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
                mask(cur, rowb - at[0]);
                const int a = j < NB ? 0 : j - NB, t = j < NB ? j : 0;
                bool huge;
                const Parts w = split(cur, huge);
                if (__any(huge) && huge) lds_write_b8((j < NB ? huge_tok + 16 * t : huge_w + 16 * a) + l16, 1);
                if (j + 1 < SEQ) read(i0 + j + 1);
                __builtin_amdgcn_sched_barrier(0);
                if (j < NB) {
                    tb[t] = w;
                } else {
                    f32x4 c[NB];
                    auto product = [&](bf16x8 Parts::*x, bf16x8 Parts::*y, bool zero) {
#pragma unroll
                        for (int b = 0; b < NB; ++b) {
                            if (zero) c[b] = f32x4{0.f, 0.f, 0.f, 0.f};
                            c[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.*x, tb[b].*y, c[b], 0, 0, 0);
                        }
                    };
                    product(&Parts::lo, &Parts::hi, true);
                    product(&Parts::hi, &Parts::lo, false);
                    product(&Parts::mid, &Parts::mid, false);
                    product(&Parts::mid, &Parts::hi, false);
                    product(&Parts::hi, &Parts::mid, false);
                    product(&Parts::hi, &Parts::hi, false);
#pragma unroll
                    for (int b = 0; b < NB; ++b) fold(acc[a][b], c[b]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
};

}  // namespace zeda
