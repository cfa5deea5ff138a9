// The direct-to-LDS convolution with K slices of 256 (Cin % 256 == 0): for long K and few tiles.
// With one or two workgroups on a CU a K slice costs its barrier and the wait for its loads, about 0.28 us for a
// slice of 128 whatever its width up to there; slices of 256 pay that half as often, until the 64 bytes a clock
// a CU loads are the bound (a 32x32 tile moves 32 KB a slice: 0.21 us).  Four or eight groups of waves share a slice's
// 16 steps of matrix instructions.  Measured, slices of 128 -> 256: 3x3, 256 channels, 14x14, batch 1 7.0 -> 6.3 us; 3x3, 512
// channels, 7x7, batch 8 10.9 -> 9.2 us and batch 16 14.4 -> 12.0 us.
// The plan takes 32x32, 64x32 and 32x64 in four groups, K whole or split, 32x32 in eight now and then and, for the fewest pixels, 32x32
// in parts (kernels_conv_small.hip).  64x64 and the wider tiles in eight groups are left to a forced or installed tile.
#include "conv_dlds_launch.h"

namespace cw {

template <typename T, int MODE, bool SPLITK>
static hipError_t launch_k256(ConvTile tile, const ConvArgs &a, hipStream_t s) {
    if (conv_tile_small(tile)) return launch_conv_dlds_small(std::is_same<T, f16>::value ? DT_F16 : DT_BF16, tile, MODE, SPLITK, a, s);
    dim3 grid;
    int block;
    conv_grid(tile, a, &grid, &block);
    switch (tile) {
        case T32x32k256g4: return launch_one<T, 32, 32, 1, 1, 256, MODE, SPLITK, 4>(grid, block, a, s);
        case T32x32k256g8: return launch_one<T, 32, 32, 1, 1, 256, MODE, SPLITK, 8>(grid, block, a, s);
        case T64x32k256g4: return launch_one<T, 64, 32, 2, 1, 256, MODE, SPLITK, 4>(grid, block, a, s);
        case T64x32k256g8: return launch_one<T, 64, 32, 2, 1, 256, MODE, SPLITK, 8>(grid, block, a, s);
        case T32x64k256g4: return launch_one<T, 32, 64, 1, 2, 256, MODE, SPLITK, 4>(grid, block, a, s);
        case T32x64k256g8: return launch_one<T, 32, 64, 1, 2, 256, MODE, SPLITK, 8>(grid, block, a, s);
        case T64x64k256g4: return launch_one<T, 64, 64, 2, 2, 256, MODE, SPLITK, 4>(grid, block, a, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_conv_dlds_k256(DType dt, ConvTile tile, int mode, bool splitk, const ConvArgs &a, hipStream_t s) {
    if (mode != MODE_GEMM && mode != MODE_CONV) return hipErrorInvalidValue;
#define CW_K256(T_, M_) return splitk ? launch_k256<T_, M_, true>(tile, a, s) : launch_k256<T_, M_, false>(tile, a, s)
    if (dt == DT_F16) {
        if (mode == MODE_GEMM) { CW_K256(f16, MODE_GEMM); }
        CW_K256(f16, MODE_CONV);
    }
    if (mode == MODE_GEMM) { CW_K256(bf16, MODE_GEMM); }
    CW_K256(bf16, MODE_CONV);
#undef CW_K256
}

}  // namespace cw
