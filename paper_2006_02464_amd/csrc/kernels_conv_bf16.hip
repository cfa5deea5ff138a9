// The direct-to-LDS convolution's plain forms in bf16 storage.
#include "conv_dlds_tiles.h"

namespace cw {

hipError_t launch_conv_tiles_bf16(ConvTile tile, int bk, int mode, const ConvArgs &a, hipStream_t s) { return launch_tiles<bf16>(tile, bk, mode, a, s); }

}  // namespace cw
