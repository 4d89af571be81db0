// A wave's private LDS ring of row blocks, for kernels whose waves split the reduction dimension.
//
// A block is 16 rows x 128 bytes (64 k in bf16, 32 in fp32), fetched with two global->LDS loads of 1 KiB: lane l takes 16
// bytes of row l / 8 (and of row 8 + l / 8), so eight neighbouring lanes read one cache line.  That order is what counts: out
// of L2, all CUs at once, it delivers 86-102 GB/s per CU, while the order that the 16-row matrix instructions want in their
// registers - neighbouring lanes in different rows - delivers 32-38 GB/s, into LDS or into registers alike.  The ring is the
// turn from one to the other: a fragment is the 16 bytes of row l % 16 at k piece 4 s + l / 16, s the step of two.
//
// Nobody else reads the ring, so there is no barrier: a wave waits for its own loads (vmcnt, in order), reads a block's two
// fragments, and refills the slot as soon as they have landed.
#pragma once
#include "zeda_lds.h"

namespace zeda {

constexpr int kRingBlock = 2048;  // 16 rows x 128 bytes

// position of 16-byte piece p of row r of a block (an involution in p): the 16 rows of a fragment read hit distinct banks
__device__ __forceinline__ int ring_swz(int row, int piece) { return piece ^ ((row >> 1) & 7); }

template <int N>
__device__ __forceinline__ void ring_wait_loads()  // at most N loads of this wave are still in flight
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// D: slots, i.e. blocks in flight.
template <int D>
struct WaveRing {
    static_assert(D >= 2 && 2 * D <= 63, "vmcnt is a 6-bit counter");
    static constexpr int BYTES = D * kRingBlock;
    uint32_t base, fill, take, frag;  // LDS address; byte offsets of the slots to fill and to read next; of this lane's fragment

    __device__ __forceinline__ void init(uint32_t lds)
    {
        const int lane = threadIdx.x & 63;
        base = lds;
        fill = take = 0;
        frag = (uint32_t)((lane & 15) * 128 + ring_swz(lane & 15, lane >> 4) * 16);
    }
    // byte of a row's 128 that this lane fetches, in the first and in the second half of a block
    __device__ __forceinline__ static uint32_t piece0() { return (uint32_t)ring_swz((threadIdx.x & 63) >> 3, threadIdx.x & 7) * 16; }
    __device__ __forceinline__ static uint32_t piece1() { return piece0() ^ 64; }
    // lo, hi: where this lane's pieces of rows 0..7 and 8..15 are.  CPOL: cache policy bits of the loads (2: non-temporal)
    template <int CPOL = 0>
    __device__ __forceinline__ void fetch(const void *lo, const void *hi)
    {
        typedef const __attribute__((address_space(1))) void *global_ptr;
        typedef __attribute__((address_space(3))) void *lds_ptr;
        const uint32_t at = base + fill;
        __builtin_amdgcn_global_load_lds((global_ptr)lo, (lds_ptr)(uintptr_t)at, 16, 0, CPOL);
        __builtin_amdgcn_global_load_lds((global_ptr)hi, (lds_ptr)(uintptr_t)(at + 1024), 16, 0, CPOL);
        fill = fill == (D - 1) * kRingBlock ? 0 : fill + kRingBlock;
    }
    // start reading the two fragments of the next block.  (Not to be left in flight across a branch or around a loop: the compiler
    // may copy registers there, before the data is in them.)
    __device__ __forceinline__ void read(u32x4 (&f)[2])
    {
        const uint32_t at = base + take + frag;
        f[0] = lds_read_b128(at);
        f[1] = lds_read_b128(at ^ 64);
        take = take == (D - 1) * kRingBlock ? 0 : take + kRingBlock;
    }
};


}  // namespace zeda
