// Grouped SwiGLU expert FFN over the real slots only (Appendix D, Eq. 10: the 6*H*H_e FLOPs of the
// gate, up and down projections are spent on the (1 - r_ZE) share of slots that landed on a normal
// expert).  Two grouped GEMMs on the bf16 MFMA units with fp32 accumulation:
//   gate/up:  act[r, i]  = silu(<x[tok(r)], W_gate[e][i]>) * <x[tok(r)], W_up[e][i]>
//   down:     y_slot[r,h] = <act[r], W_down[e][h]>
// for the rows r of expert e in expert-sorted order.  Both operands have the reduction dimension
// contiguous, so every MFMA fragment is one 16-byte LDS read.  The tile kernel is in zeda_ffn_tile.h;
// zeda_ffn_launch.h picks the tile shapes.  fp32 layers: zeda_ffn_f32.hip; few rows per expert: zeda_ffn_few.hip.
#include "zeda_ffn_launch.h"

namespace zeda {

// Tiled weight layout.  A matrix W[F][Kd] (F, Kd multiples of 32) is stored as (F/32) x (Kd/32) units of 2 KiB,
// unit (rb, kb) at index kb * (F/32) + rb, so that the row blocks of one k block follow each other: the
// consecutive row blocks of a feature tile are then one contiguous run of 8-16 KiB per k chunk.  A
// unit holds rows 32rb..32rb+31, columns 32kb..32kb+31 as 32 rows of 64 bytes, the four 16-byte pieces of
// row r permuted as in the LDS ring (piece p at position p ^ ((r >> 2) & 3)): it is the LDS image of that
// block, so the GEMM copies it with contiguous 1 KiB loads - which is what lets HBM stream at full rate
// (row-major weights are fetched as 64- or 128-byte pieces 2*Kd bytes apart).
// One thread per 16-byte piece of the output; `mats` matrices of F x Kd follow each other.
__global__ __launch_bounds__(256) void pack_weights_kernel(const bf16_t *__restrict__ w, bf16_t *__restrict__ out, int F,
                                                           int Kd, size_t pieces)
{
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= pieces) return;
    const int pos = idx & 3, r = (idx >> 2) & 31;
    const size_t unit = idx >> 7;
    const int kbs = Kd / 32, units_per_mat = (F / 32) * kbs;
    const size_t mat = unit / units_per_mat;
    const int u = (int)(unit - mat * units_per_mat), rbs = F / 32, kb = u / rbs, rb = u - kb * rbs;
    const int p = pos ^ ((r >> 2) & 3);
    const bf16x8 v = *reinterpret_cast<const bf16x8 *>(w + (mat * F + rb * 32 + r) * Kd + kb * 32 + p * 8);
    *reinterpret_cast<bf16x8 *>(out + idx * 8) = v;
}

int launch_pack_weights(const zeda_layer_desc *d, const void *w, void *out, bool down, hipStream_t s)
{
    const int F = down ? d->H : d->I, Kd = down ? d->I : d->H;
    const size_t pieces = (size_t)d->N * F * Kd / 8;
    pack_weights_kernel<<<(unsigned)((pieces + 255) / 256), 256, 0, s>>>((const bf16_t *)w, (bf16_t *)out, F, Kd, pieces);
    return last_launch_status();
}

int launch_gateup(const zeda_layer_desc *d, const void *x, const void *wg, const void *wu, const int32_t *offsets,
                  const int32_t *sorted_slot, void *act, const TilePlace *tp, hipStream_t s)
{
    if (d->dtype == ZEDA_BF16 && ffn_few_blocks(d)) return launch_gateup_few(d, x, wg, wu, offsets, sorted_slot, act, tp, s);
    if (d->dtype == ZEDA_BF16) return launch_bf16<true>(d, x, wg, wu, offsets, sorted_slot, act, s);
    return launch_gateup_f32(d, x, wg, wu, offsets, sorted_slot, act, tp, s);
}

}  // namespace zeda
