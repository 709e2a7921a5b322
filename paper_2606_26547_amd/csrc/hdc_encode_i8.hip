// Encoder instantiations: int8 features on the int8 path.
#include "hdc_encode_impl.h"

namespace hdc {
hipError_t launch_encode_i8(const EncodeArgs &a, int mode, Tile tile, hipStream_t st)
{
    return launch_bytes<C_I8, W_ROWS>(a, mode, tile, st);
}
}  // namespace hdc
