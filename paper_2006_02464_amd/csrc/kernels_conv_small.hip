// The direct-to-LDS convolution on 32x32 tiles in parts, each on a workgroup of its own (four groups of one wave, 16x16x32 matrix
// instructions): quarters of 16x16, or halves of 32 pixels x 16 channels or 16 x 32.  For few pixels and long K.
// The networks' own layers are split in K on quarters with slices of 256 alone; other shapes on all five.
// A workgroup's K walk is bound by what its CU loads, 64 bytes a clock: a slice of 256 for a whole tile is 32 KB, for
// a quarter half of that, and where whole tiles leave most of the CUs idle (batch 1: 56 workgroups in stage 3, 32 in stage 4)
// the four quarters run beside each other.  The groups' accumulators, a quarter as many, are also added up sooner.
// First workgroup's start to last store, 32x32k256g4 -> in quarters, batch 1: 3x3 of 256 channels at 14x14 4.85 -> 3.39 us, of 512
// channels at 7x7 7.53 (5.85 with K in 4 parts) -> 5.05, 1x1 2048 -> 512 at 7x7 4.56 -> 3.30, 1024 -> 256 at 14x14 3.19 -> 2.37.
// With 64x64 tiles whose four waves each own the whole tile for a quarter of K (half the LDS reads per matrix
// instruction) the 3x3 of stage 3 at batch 16 took 9.4 us, on 64x64 in four groups of four waves 9.2: not kept.
#include "conv_dlds_launch.h"

namespace cw {

template <typename T, int MODE, bool SPLITK>
static hipError_t launch_small(ConvTile tile, const ConvArgs &a, hipStream_t s) {
    dim3 grid;
    int block;
    conv_grid(tile, a, &grid, &block);
    switch (tile) {
        case T32x32k128g4q: return launch_one<T, 16, 16, 1, 1, 128, MODE, SPLITK, 4, 16>(grid, block, a, s);
        case T32x32k128g4n: return launch_one<T, 32, 16, 1, 1, 128, MODE, SPLITK, 4, 16>(grid, block, a, s);
        case T32x32k128g4m: return launch_one<T, 16, 32, 1, 1, 128, MODE, SPLITK, 4, 16>(grid, block, a, s);
        case T32x32k256g4q: return launch_one<T, 16, 16, 1, 1, 256, MODE, SPLITK, 4, 16>(grid, block, a, s);
        case T32x32k256g4n: return launch_one<T, 32, 16, 1, 1, 256, MODE, SPLITK, 4, 16>(grid, block, a, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_conv_dlds_small(DType dt, ConvTile tile, int mode, bool splitk, const ConvArgs &a, hipStream_t s) {
    if (mode != MODE_GEMM && mode != MODE_CONV) return hipErrorInvalidValue;
#define CW_SMALL(T_, M_) return splitk ? launch_small<T_, M_, true>(tile, a, s) : launch_small<T_, M_, false>(tile, a, s)
    if (dt == DT_F16) {
        if (mode == MODE_GEMM) { CW_SMALL(f16, MODE_GEMM); }
        CW_SMALL(f16, MODE_CONV);
    }
    if (mode == MODE_GEMM) { CW_SMALL(bf16, MODE_GEMM); }
    CW_SMALL(bf16, MODE_CONV);
#undef CW_SMALL
}

}  // namespace cw
