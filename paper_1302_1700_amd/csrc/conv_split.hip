// Float32 layers with bounded inputs on the f16 matrix cores: every operand
// as two f16 values (conv_impl.h, half-step walk).
#include "conv_impl.h"

namespace fs {

hipError_t launch_conv_split(const ConvArgs &a, int mb, int nb, int wn, int wk, int gx, int gy, hipStream_t s)
{
    return conv::dispatch_tile<false, false, true, true>(a, mb, nb, wn, wk, gx, gy, s);
}

int conv_blocks_per_cu_split(int mb, int nb, int wn, int wk, bool run, int lds)
{
    return conv::tile_blocks_per_cu<false, false, true, true>(mb, nb, wn, wk, run, lds);
}

}  // namespace fs
