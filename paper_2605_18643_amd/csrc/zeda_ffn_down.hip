// Down projection of the expert FFN (Appendix D, Eq. 10): the second of the two grouped GEMMs, see zeda_ffn.hip.
#include "zeda_ffn_launch.h"

namespace zeda {

int launch_down(const zeda_layer_desc *d, const void *act, const void *wd, const int32_t *offsets, void *y_slot,
                hipStream_t s)
{
    if (d->dtype == ZEDA_BF16 && ffn_few_blocks(d)) return launch_down_few(d, act, wd, offsets, y_slot, s);
    if (d->dtype == ZEDA_BF16) return launch_bf16<false>(d, act, wd, nullptr, offsets, nullptr, y_slot, s);
    return launch_down_f32(d, act, wd, offsets, y_slot, s);
}

}  // namespace zeda
