// Encoder instantiations for the E4M3 compute type on byte features.
#include "hdc_encode_impl.h"

namespace hdc {
hipError_t launch_encode_fp8(const EncodeArgs &a, int mode, Tile tile, hipStream_t st)
{
    if (a.poff)   // E4M3 rows of the shifted projection
        return launch_bytes<C_FP8, W_ROWS>(a, mode, tile, st);
    return launch_bytes<C_FP8, W_ALT>(a, mode, tile, st);
}
}  // namespace hdc
