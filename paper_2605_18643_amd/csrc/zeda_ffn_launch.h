// Tile shapes of the expert GEMM kernels (zeda_ffn_tile.h) and the rules that pick one.  Included by zeda_ffn.hip for the
// gate/up GEMM and by zeda_ffn_down.hip for the down GEMM: two translation units, as their many instantiations take long
// to compile.
#pragma once
#include "zeda_ffn_tile.h"

namespace zeda {

//              G FB WF NSW NST KC   (NSW, NST: depth of the weight and of the token ring)
typedef TileCfg<4, 2, 4, 2, 2, 64> CfgPrefill;  // 256 tokens x 256 weight rows, 8 waves, one workgroup per CU
typedef TileCfg<4, 2, 2, 2, 2, 64> CfgNarrow;   // 256 tokens x 128 weight rows, 4 waves: any H % 128 == 0, I % 64 == 0
typedef TileCfg<1, 2, 2, 4, 4, 32> CfgDecode;   // 64 tokens x 128 weight rows, 4 waves, two workgroups per CU
// tiled weights come in 32-wide k blocks: 32-wide chunks, four deep
typedef TileCfg<4, 2, 4, 4, 4, 32> CfgPrefillT;
typedef TileCfg<4, 2, 4, 4, 2, 32, 64> CfgPrefillTP;  // the same, token rows 64 k at a time
typedef TileCfg<4, 2, 2, 4, 4, 32> CfgNarrowT;
// 320 tokens x 256 weight rows (token ring three deep): an expert with a few rows more than a multiple of 256 gets
// one token tile less than CfgPrefillTP would give it, i.e. one pass less over its weights.  It is the second
// geometry of the adaptive kernel, which picks one of the two from the expert loads.  (With the 64-wide token ring, which
// leaves it half the room to turn results in, it gains 1-2 % at 8192 tokens and loses 1.5 % at 6000.)
typedef TileCfg<5, 2, 4, 4, 3, 32> CfgPrefillT5;

// Persistent grid: as many workgroups as the device holds at once, rounded down to a multiple of 8 so that
// every XCD gets the same number (the kernel reads the count from gridDim).
template <class C, bool GATEUP, bool TILED>
static int resident_grid()
{
    static int grids[kMaxDevices] = {};  // per instantiation and device; idempotent, so a race between host threads is harmless
    const int dev = current_device();
    if (dev < 0) return 0;
    int &grid = grids[dev];
    if (grid == 0) {
        auto kern = ffn_bf16_kernel<C, GATEUP, TILED>;
        int cus = 0, per_cu = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kern, C::THREADS, C::LDS_BYTES) != hipSuccess)
            return 0;
        const int g = cus * (per_cu > 0 ? per_cu : 1) / 8 * 8;
        grid = g > 0 ? g : 8;
    }
    return grid;
}

template <class CA, class CB, bool GATEUP, bool TILED>
static int launch_adaptive_kernel(const zeda_layer_desc *d, const void *tok, const void *w0, const void *w1,
                                  const int32_t *offsets, const int32_t *sorted_slot, void *out, hipStream_t s)
{
    constexpr int kLds = CA::LDS_BYTES > CB::LDS_BYTES ? CA::LDS_BYTES : CB::LDS_BYTES;
    auto kern = ffn_bf16_adaptive_kernel<CA, CB, GATEUP, TILED>;
    static int grids[kMaxDevices] = {};  // (as in resident_grid)
    const int dev = current_device();
    if (dev < 0) return ZEDA_EHIP;
    int &grid = grids[dev];
    if (grid == 0) {
        int cus = 0, per_cu = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kLds) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kern, CA::THREADS, kLds) != hipSuccess)
            return ZEDA_EHIP;
        const int g = cus * (per_cu > 0 ? per_cu : 1) / 8 * 8;
        grid = g > 0 ? g : 8;
    }
    const int Kdim = GATEUP ? d->H : d->I, Fdim = GATEUP ? d->I : d->H;
    const int n_ftiles = GATEUP ? Fdim / (CA::BF / 2) : Fdim / CA::BF;
    kern<<<grid, CA::THREADS, kLds, s>>>((const bf16_t *)tok, (const bf16_t *)w0, (const bf16_t *)w1, offsets, sorted_slot,
                                         (bf16_t *)out, d->N, d->K, Kdim, Fdim, n_ftiles, d->T);
    return last_launch_status();
}

// Whether the expert loads may sit just above a multiple of the 256-row tile, where the wide tile saves a pass over
// the weights (the adaptive kernel then decides on the device; where they cannot, the plain kernel saves the 1-2 %
// the second geometry costs the first).  The mean row count is T*K/N when every slot is real - loads then cluster
// around it - and anything below that with zero experts.
static bool rows_may_straddle_tile(const zeda_layer_desc *d)
{
    const double all_real = (double)d->T * d->K / d->N;
    // (at a thousand rows per expert and more the passes saved no longer pay for it: measured on config 4)
    if (d->Z > 0) return all_real > 256.0 && all_real < 1024.0;
    for (int k = 1; k <= 2; ++k)
        if (all_real > 240.0 * k && all_real <= 330.0 * k) return true;
    return false;
}

// Whether experts have enough rows for the 64-wide token ring, by the slots per expert of the whole pool.  It saves half of
// the token rows' trips through the vector memory path (T=4096, N=128: gate/up 172 -> 163 us, down 101 -> 98; N=64, I=1536:
// 286 -> 275 us a layer), but a row is asked for two chunks ahead instead of three, which tells where a chunk is multiplied
// in no time (31 rows per expert, 50 slots: gate/up 133 -> 144 us, down 72 -> 81; level at 78 rows, 125 slots).
static bool rows_fill_groups(const zeda_layer_desc *d) { return (int64_t)d->T * d->K >= 110 * ((int64_t)d->N + d->Z); }
// That ring addresses token rows (of x, of act) with 32-bit byte offsets; above 4 GiB of them the 32-wide one is taken.
static bool rows_addressable(const zeda_layer_desc *d)
{
    return (uint64_t)d->T * d->H * 2 <= UINT32_MAX && (uint64_t)d->T * d->K * d->I * 2 <= UINT32_MAX;
}

template <class C, bool GATEUP, bool TILED>
static int launch_tile_kernel(const zeda_layer_desc *d, const void *tok, const void *w0, const void *w1,
                              const int32_t *offsets, const int32_t *sorted_slot, void *out, hipStream_t s)
{
    const int grid = resident_grid<C, GATEUP, TILED>();
    if (grid == 0) return ZEDA_EHIP;
    const int Kdim = GATEUP ? d->H : d->I, Fdim = GATEUP ? d->I : d->H;
    const int n_ftiles = GATEUP ? Fdim / (C::BF / 2) : Fdim / C::BF;
    ffn_bf16_kernel<C, GATEUP, TILED><<<grid, C::THREADS, C::LDS_BYTES, s>>>((const bf16_t *)tok, (const bf16_t *)w0,
                                                                     (const bf16_t *)w1, offsets, sorted_slot,
                                                                     (bf16_t *)out, d->N, d->K, Kdim, Fdim, n_ftiles, d->T);
    return last_launch_status();
}

// Feature tiles must divide the output width: gate/up tiles are BF/2 columns of I, down tiles BF columns of H.
template <class C>
static bool cfg_fits(const zeda_layer_desc *d)
{
    return d->I % (C::BF / 2) == 0 && d->H % C::BF == 0;
}

template <bool GATEUP>
static int launch_bf16(const zeda_layer_desc *d, const void *tok, const void *w0, const void *w1, const int32_t *offsets,
                       const int32_t *sorted_slot, void *out, hipStream_t s)
{
    // Decode batches with too many rows or too short a reduction for the few-row kernel: one token tile per expert, and small
    // enough for two workgroups a CU (N=8, I=14336, 12 rows: 577 us row-major against 618 with CfgPrefill, 416 against 449 tiled).
    if (d->T <= CfgDecode::BT) {
        return d->weight_layout == ZEDA_WEIGHTS_TILED ? launch_tile_kernel<CfgDecode, GATEUP, true>(d, tok, w0, w1, offsets, sorted_slot, out, s)
                                                      : launch_tile_kernel<CfgDecode, GATEUP, false>(d, tok, w0, w1, offsets, sorted_slot, out, s);
    }
    if (d->weight_layout == ZEDA_WEIGHTS_TILED) {
        if (cfg_fits<CfgPrefillT>(d)) {
            if (rows_may_straddle_tile(d))
                return rows_addressable(d) ? launch_adaptive_kernel<CfgPrefillTP, CfgPrefillT5, GATEUP, true>(d, tok, w0, w1, offsets, sorted_slot, out, s)
                                           : launch_adaptive_kernel<CfgPrefillT, CfgPrefillT5, GATEUP, true>(d, tok, w0, w1, offsets, sorted_slot, out, s);
            if (rows_fill_groups(d) && rows_addressable(d)) return launch_tile_kernel<CfgPrefillTP, GATEUP, true>(d, tok, w0, w1, offsets, sorted_slot, out, s);
            return launch_tile_kernel<CfgPrefillT, GATEUP, true>(d, tok, w0, w1, offsets, sorted_slot, out, s);
        }
        return launch_tile_kernel<CfgNarrowT, GATEUP, true>(d, tok, w0, w1, offsets, sorted_slot, out, s);
    }
    if (cfg_fits<CfgPrefill>(d))
        return launch_tile_kernel<CfgPrefill, GATEUP, false>(d, tok, w0, w1, offsets, sorted_slot, out, s);
    return launch_tile_kernel<CfgNarrow, GATEUP, false>(d, tok, w0, w1, offsets, sorted_slot, out, s);
}

}  // namespace zeda
