// Encoder instantiations for the fp32 compute type (fp32 features).
#include "hdc_encode_impl.h"

namespace hdc {
hipError_t launch_encode_f32(const EncodeArgs &a, int mode, Tile tile, hipStream_t st)
{
    return launch_fp32<C_F32>(a, mode, tile, st);
}
}  // namespace hdc
