// The direct-to-LDS convolution's plain forms in fp16 storage.
#include "conv_dlds_tiles.h"

namespace cw {

hipError_t launch_conv_tiles_f16(ConvTile tile, int bk, int mode, const ConvArgs &a, hipStream_t s) { return launch_tiles<f16>(tile, bk, mode, a, s); }

}  // namespace cw
