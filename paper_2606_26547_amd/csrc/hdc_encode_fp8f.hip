// Encoder instantiations for the E4M3 compute type on fp32 features.
#include "hdc_encode_impl.h"

namespace hdc {
hipError_t launch_encode_fp8f(const EncodeArgs &a, int mode, Tile tile, hipStream_t st)
{
    return launch_fp32<C_FP8>(a, mode, tile, st);
}
}  // namespace hdc
