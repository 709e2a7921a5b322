// Encoder instantiations: uint8 features on the int8 path.
#include "hdc_encode_impl.h"

namespace hdc {
hipError_t launch_encode_u8(const EncodeArgs &a, int mode, Tile tile, hipStream_t st)
{
    return launch_bytes<C_I8, W_ALT>(a, mode, tile, st);
}
}  // namespace hdc
