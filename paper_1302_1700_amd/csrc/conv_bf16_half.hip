// bfloat16 layers whose input channels are an odd multiple of 16
// (conv_impl.h, half-step walk).
#include "conv_impl.h"

namespace fs {

hipError_t launch_conv_bf16_half(const ConvArgs &a, int mb, int nb, int wn, int wk, int gx, int gy, hipStream_t s)
{
    return conv::dispatch_tile<true, false, true, true>(a, mb, nb, wn, wk, gx, gy, s);
}

int conv_blocks_per_cu_bf16_half(int mb, int nb, int wn, int wk, bool run, int lds)
{
    return conv::tile_blocks_per_cu<true, false, true, true>(mb, nb, wn, wk, run, lds);
}

}  // namespace fs
