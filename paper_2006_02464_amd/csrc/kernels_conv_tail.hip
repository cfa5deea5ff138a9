// The direct-to-LDS convolution, 1x1 stride-1 form, for input channels that are no multiple of the K slice (Cin % 32 == 0): the
// last slice's missing chunks are fetched out of range, as zeros.  The register-staged kernel, which took these
// shapes with K slices of 32, needs 1.4-2.2 us more for 160-480 channels than its neighbours of whole slices here
// (DenseNet batch 6: 238 -> 228 us).  The plan never splits K here; a forced or installed split does.
#include "conv_dlds_launch.h"

namespace cw {

template <typename T, bool SPLITK>
static hipError_t launch_tail(ConvTile tile, const ConvArgs &a, hipStream_t s) {
    dim3 grid;
    int block;
    const int bk = conv_bk(a, false, tile);
    tile = bk == 64 ? conv_tile_k64(conv_tile_tail(tile)) : conv_tile_tail(tile);
    conv_grid(tile, a, &grid, &block);
    switch (tile) {
        case T128x128: return launch_one<T, 128, 128, 2, 2, 64, MODE_TAIL, SPLITK>(grid, block, a, s);
        case T128x128w8: return launch_one<T, 128, 128, 2, 4, 64, MODE_TAIL, SPLITK>(grid, block, a, s);
        case T128x64: return launch_one<T, 128, 64, 2, 2, 64, MODE_TAIL, SPLITK>(grid, block, a, s);
        case T64x64: return launch_one<T, 64, 64, 2, 2, 64, MODE_TAIL, SPLITK>(grid, block, a, s);
        case T64x32: return launch_one<T, 64, 32, 2, 1, 64, MODE_TAIL, SPLITK>(grid, block, a, s);
        case T32x64: return launch_one<T, 32, 64, 1, 2, 64, MODE_TAIL, SPLITK>(grid, block, a, s);
        case T32x32: return launch_one<T, 32, 32, 1, 1, 64, MODE_TAIL, SPLITK>(grid, block, a, s);
        case T128x64k128: return launch_one<T, 128, 64, 2, 2, 128, MODE_TAIL, SPLITK>(grid, block, a, s);
        case T64x64k128: return launch_one<T, 64, 64, 2, 2, 128, MODE_TAIL, SPLITK>(grid, block, a, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_conv_dlds_tail(DType dt, ConvTile tile, bool splitk, const ConvArgs &a, hipStream_t s) {
    if (dt == DT_F16) return splitk ? launch_tail<f16, true>(tile, a, s) : launch_tail<f16, false>(tile, a, s);
    return splitk ? launch_tail<bf16, true>(tile, a, s) : launch_tail<bf16, false>(tile, a, s);
}

}  // namespace cw
