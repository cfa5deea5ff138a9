// The plain forms' tiles on the direct-to-LDS kernel, for the two files that instantiate them (one per storage type).
#pragma once
#include "conv_dlds_launch.h"

namespace cw {

template <typename T, int MODE, bool SPLITK>
static hipError_t launch_tile(ConvTile tile, int bk, const ConvArgs &a, hipStream_t s) {
    if (MODE == MODE_STEM) tile = conv_tile_one_group(tile);
    if (bk == 64) tile = conv_tile_k64(tile);
    else if (bk == 256) return launch_conv_dlds_k256(std::is_same<T, f16>::value ? DT_F16 : DT_BF16, tile, MODE, SPLITK, a, s);
    if (conv_tile_small(tile)) return launch_conv_dlds_small(std::is_same<T, f16>::value ? DT_F16 : DT_BF16, tile, MODE, SPLITK, a, s);
    dim3 grid;
    int block;
    conv_grid(tile, a, &grid, &block);
    switch (tile) {
        case T128x128: return launch_one<T, 128, 128, 2, 2, 64, MODE, SPLITK>(grid, block, a, s);
        case T128x64: return launch_one<T, 128, 64, 2, 2, 64, MODE, SPLITK>(grid, block, a, s);
        case T64x64: return launch_one<T, 64, 64, 2, 2, 64, MODE, SPLITK>(grid, block, a, s);
        case T64x32: return launch_one<T, 64, 32, 2, 1, 64, MODE, SPLITK>(grid, block, a, s);
        case T32x64: return launch_one<T, 32, 64, 1, 2, 64, MODE, SPLITK>(grid, block, a, s);
        case T32x32: return launch_one<T, 32, 32, 1, 1, 64, MODE, SPLITK>(grid, block, a, s);
        case T128x64w2: return launch_one<T, 128, 64, 2, 1, 64, MODE, SPLITK>(grid, block, a, s);
        case T64x128w2: return launch_one<T, 64, 128, 1, 2, 64, MODE, SPLITK>(grid, block, a, s);
        case T256x64: return launch_one<T, 256, 64, 4, 1, 64, MODE, SPLITK>(grid, block, a, s);
        case T128x128w8: return launch_one<T, 128, 128, 2, 4, 64, MODE, SPLITK>(grid, block, a, s);
        case T128x64k128:
            if constexpr (MODE != MODE_STEM) return launch_one<T, 128, 64, 2, 2, 128, MODE, SPLITK>(grid, block, a, s);
            return hipErrorInvalidValue;
        case T64x64k128:
            if constexpr (MODE != MODE_STEM) return launch_one<T, 64, 64, 2, 2, 128, MODE, SPLITK>(grid, block, a, s);
            return hipErrorInvalidValue;
        case T64x32k128:
            if constexpr (MODE != MODE_STEM) return launch_one<T, 64, 32, 2, 1, 128, MODE, SPLITK>(grid, block, a, s);
            return hipErrorInvalidValue;
        case T32x64k128:
            if constexpr (MODE != MODE_STEM) return launch_one<T, 32, 64, 1, 2, 128, MODE, SPLITK>(grid, block, a, s);
            return hipErrorInvalidValue;
        case T32x32k128:
            if constexpr (MODE != MODE_STEM) return launch_one<T, 32, 32, 1, 1, 128, MODE, SPLITK>(grid, block, a, s);
            return hipErrorInvalidValue;
        case T128x64k128g2:
            if constexpr (MODE != MODE_STEM) return launch_one<T, 128, 64, 2, 2, 128, MODE, SPLITK, 2>(grid, block, a, s);
            return hipErrorInvalidValue;
        case T64x64k128g2:
            if constexpr (MODE != MODE_STEM) return launch_one<T, 64, 64, 2, 2, 128, MODE, SPLITK, 2>(grid, block, a, s);
            return hipErrorInvalidValue;
        case T64x64k128g4:
            if constexpr (MODE != MODE_STEM) return launch_one<T, 64, 64, 2, 2, 128, MODE, SPLITK, 4>(grid, block, a, s);
            return hipErrorInvalidValue;
        case T64x32k128g4:
            if constexpr (MODE != MODE_STEM) return launch_one<T, 64, 32, 2, 1, 128, MODE, SPLITK, 4>(grid, block, a, s);
            return hipErrorInvalidValue;
        case T32x64k128g4:
            if constexpr (MODE != MODE_STEM) return launch_one<T, 32, 64, 1, 2, 128, MODE, SPLITK, 4>(grid, block, a, s);
            return hipErrorInvalidValue;
        case T32x32k128g4:
            if constexpr (MODE != MODE_STEM) return launch_one<T, 32, 32, 1, 1, 128, MODE, SPLITK, 4>(grid, block, a, s);
            return hipErrorInvalidValue;
        case T32x32k128g8:
            if constexpr (MODE != MODE_STEM) return launch_one<T, 32, 32, 1, 1, 128, MODE, SPLITK, 8>(grid, block, a, s);
            return hipErrorInvalidValue;
        case T128x64g2:
            if constexpr (MODE != MODE_STEM) return launch_one<T, 128, 64, 2, 2, 64, MODE, SPLITK, 2>(grid, block, a, s);
            return hipErrorInvalidValue;
        case T64x64g2:
            if constexpr (MODE != MODE_STEM) return launch_one<T, 64, 64, 2, 2, 64, MODE, SPLITK, 2>(grid, block, a, s);
            return hipErrorInvalidValue;
        case T32x32g4:
            if constexpr (MODE != MODE_STEM) return launch_one<T, 32, 32, 1, 1, 64, MODE, SPLITK, 4>(grid, block, a, s);
            return hipErrorInvalidValue;
        case T256x128w8: return launch_one<T, 256, 128, 4, 2, 64, MODE, SPLITK>(grid, block, a, s);
        case T128x256w8: return launch_one<T, 128, 256, 2, 4, 64, MODE, SPLITK>(grid, block, a, s);
        case T256x256w8: return launch_one<T, 256, 256, 4, 2, 64, MODE, SPLITK>(grid, block, a, s);
        case T256x128: return launch_one<T, 256, 128, 2, 2, 64, MODE, SPLITK>(grid, block, a, s);
        default: return hipErrorInvalidValue;
    }
}

template <typename T, bool SPLITK>
static hipError_t launch_mode(ConvTile tile, int bk, int mode, const ConvArgs &a, hipStream_t s) {
    switch (mode) {
        case MODE_GEMM: return launch_tile<T, MODE_GEMM, SPLITK>(tile, bk, a, s);
        case MODE_CONV: return launch_tile<T, MODE_CONV, SPLITK>(tile, bk, a, s);
        case MODE_STEM: return launch_tile<T, MODE_STEM, SPLITK>(tile, 64, a, s);
        default: return hipErrorInvalidValue;
    }
}

template <typename T>
static hipError_t launch_tiles(ConvTile tile, int bk, int mode, const ConvArgs &a, hipStream_t s) {
    return a.split_k > 1 ? launch_mode<T, true>(tile, bk, mode, a, s) : launch_mode<T, false>(tile, bk, mode, a, s);
}

}  // namespace cw
