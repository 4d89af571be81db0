// Building block of the fp32 expert FFN: a wave multiplies NA blocks of 16 weight rows with NB blocks of 16 token rows on the
// bf16 matrix instruction, every fp32 number as the sum of three bf16 numbers, operands through a ring of its own in LDS.
//
// Why not the fp32 instruction: it runs at the rate of the vector unit and keeps vector instructions out while it does (16x16x4
// in a register-only loop, two waves per SIMD: 32 cycles each, 59 with the 20 vector instructions between every eight that add
// the sums up).  x = hi + mid + lo is exact inside the window below, with each part rounded to nearest; of the nine products of parts
// six are formed, the other three are below 2^-26 of the product (Henry, Tang, Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations", ARITH 2019).  Six 16x16x32 take 96 cycles of the matrix unit where
// eight 16x16x4 take 256, and the vector unit is free for the splitting (44 instructions per 16 x 32 block of an operand, and 8 for
// the window: 513 tokens, H=1024, I=512 94.3 -> 96.4 us a layer).
//
// A lane's fragments are two pieces of four consecutive k of one row: lane l holds row l % 16, pieces l / 16 and 4 + l / 16 of
// the 32 k; both operands are permuted alike, so the sum runs over all of them.
//
// Precision: a chunk's 6 x 32 products of parts are added in one fp32 accumulator of the matrix unit, smallest parts first, where the
// fp32 instruction adds eight whole products; chunk sums and the slices of the waves are added in 64 bits and rounded once.  Error
// against 64 bits, 2-norm, whole layer: T=513, H=1024, I=512 1.46e-7 (four sums of eight products on the fp32 instruction and a tree
// over them: 1.60e-7).
//
// The window: nonzero magnitudes from 2^-110 to 2^60.  Inside it the parts are bf16 numbers, subnormal ones among them, which
// the matrix unit takes and gives as the fp32 instruction does (probed: products, accumulators and results down to 2^-149); and
// neither a product nor a chunk's sum of 32 can overflow (2^125).  Below it low parts fall off the end of bf16; above it an
// overflowing product is infinity minus infinity in its parts, or infinite where both factors' hi rounded up.  Rows with an
// element outside are reported, and the caller multiplies them on the fp32 instruction (zeda_f32_tile.h).  No-numbers pass: they
// come out as such either way.
#pragma once
#include "zeda_wave_ring.h"

namespace zeda {

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr float kSplitMin = 0x1p-110f, kSplitMax = 0x1p60f;

// D: blocks that the wave keeps in flight
template <int NA, int NB, int D>
struct F32Split {
    static constexpr int SEQ = NB + NA;  // blocks of a chunk of 32 k: token rows first
    static_assert(16 * NB <= 32 && 16 * NA <= 64, "a bit per row");
    f64x2 acc[NA][NB][2];
    uint32_t odd_tok;  // bit 16 b + r: row r of token block b has an element outside the window, its sums are not to be used
    uint64_t odd_w;    // the same of the weight blocks

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
    // eight elements a lane.  odd: receives a bit for each of the block's 16 rows, is there an element outside the window
    __device__ __forceinline__ static Parts split(const u32x4 (&f)[2], uint32_t &odd)
    {
        float largest = 0.f, least = kSplitMin;
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
            const float v0 = __uint_as_float(f[i >> 2][i & 3]), v1 = __uint_as_float(f[i >> 2][(i & 3) + 1]);
            largest = fmaxf(fmaxf(fabsf(v0), fabsf(v1)), largest);
            least = fminf(fminf(fabsf(v0), fabsf(v1)), least);
        }
        odd = 0;
        if (__any(largest > kSplitMax || least < kSplitMin)) {  // (zeros come here too)
            uint32_t low = ~0u;  // smallest 2 |element| - 1 in bits, which zeros leave alone
#pragma unroll
            for (int i = 0; i < 8; ++i) low = min(low, 2 * f[i >> 2][i & 3] - 1);
            const unsigned long long m = __ballot(largest > kSplitMax || low < 2 * __float_as_uint(kSplitMin) - 1);
            const uint32_t h = (uint32_t)(m | (m >> 32));
            odd = (h | (h >> 16)) & 0xffffu;
        }
        u32x4 part[3];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v0 = __uint_as_float(f[i >> 1][2 * (i & 1)]), v1 = __uint_as_float(f[i >> 1][2 * (i & 1) + 1]);
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const uint32_t two = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){v0, v1}, bf16x2));
                part[p][i] = two;
                v0 -= __uint_as_float(two << 16);
                v1 -= __uint_as_float(two & 0xffff0000u);
            }
        }
        return {__builtin_bit_cast(bf16x8, part[0]), __builtin_bit_cast(bf16x8, part[1]), __builtin_bit_cast(bf16x8, part[2])};
    }

    // lds: this wave's ring.  The rows of weight block a start at base[a % 2] + wo[a][.] bytes, those of token block b at pb[b][.]
    // ([0]: row lane / 8 of the block, [1]: row 8 + lane / 8).  Kd: a multiple of 4.
    // Slice `slice` of `slices`: the 32-wide chunks slice, slice + slices, ..., starting at one that depends on rot (rows
    // are often a multiple of 4 KiB apart, which puts a chunk of every row on one L2 channel: workgroups that start at
    // different chunks spread over the channels)
    __device__ __forceinline__ void run(uint32_t lds, const float *base0, const float *base1, const uint32_t (&wo)[NA][2],
                                        const float *const (&pb)[NB][2], int slice, int slices, int rot, int Kd)
    {
        clear();
        odd_tok = 0;
        odd_w = 0;
        const int n = ((Kd + 31) / 32 - slice + slices - 1) / slices;
        if (n <= 0) return;
        const int first = (int)((unsigned)rot % (unsigned)n), total = n * SEQ;
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
        constexpr uint32_t ALL_TOK = ~0u >> (32 - 16 * NB);
        constexpr uint64_t ALL_W = ~0ull >> (64 - 16 * NA);
        for (int k = 0; k < n; k = odd_tok == ALL_TOK || odd_w == ALL_W ? n : k + 1) {  // (then nothing of this will be used)
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
                uint32_t odd;
                const Parts w = split(cur, odd);
                if (j < NB) odd_tok |= odd << (16 * t);
                else odd_w |= (uint64_t)odd << (16 * a);
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
        ring_wait_loads<0>();
    }
};

}  // namespace zeda
