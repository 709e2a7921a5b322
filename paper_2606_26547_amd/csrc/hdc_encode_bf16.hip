// Encoder instantiations for the bf16 compute type (fp32 features).
#include "hdc_encode_impl.h"

namespace hdc {
hipError_t launch_encode_bf16(const EncodeArgs &a, int mode, Tile tile, hipStream_t st)
{
    return launch_fp32<C_BF16>(a, mode, tile, st);
}
}  // namespace hdc
