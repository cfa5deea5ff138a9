// Launches of the direct-to-LDS implicit-GEMM convolution: checks, dispatch and the fused / pair forms.  The per-tile
// body is in conv_dlds_body.h, the plain forms' tiles in conv_dlds_tiles.h.
#include <cstring>

#include "conv_dlds_launch.h"

namespace cw {

// Two independent convolutions that read the same tensor (the first 1x1 of a bottleneck and the
// projection shortcut beside it) in one launch: the first nb0 workgroups take the first, the rest
// the second.  Same instantiation for both (general addressing mode, no split-K); one dispatch,
// one set-up latency and one tail instead of two.
struct alignas(64) ConvLines { unsigned long long v[16]; };   // of each its first two argument lines, which hold all it reads
static_assert(offsetof(ConvArgs, khp) == sizeof(ConvLines), "argument lines");
template <typename T, int BM, int BN, int WARPS_M, int WARPS_N, int BK, int NS, int KG, int MT, bool LOADERS>
__global__ __launch_bounds__((conv_threads<WARPS_M, WARPS_N, KG, LOADERS>())) void conv_dlds_pair_kernel(const ConvLines l0, const ConvLines l1) {
    ConvArgs a0, a1;
    __builtin_memcpy(&a0, &l0, sizeof l0);
    __builtin_memcpy(&a1, &l1, sizeof l1);
    const int nb0 = conv_nb_tiles(a0.nb) * conv_parts<BM, BN, MT>();
    if ((int)blockIdx.x < nb0)
        conv_body<T, BM, BN, WARPS_M, WARPS_N, BK, NS, MODE_CONV, false, false, KG, MT, LOADERS>(a0, blockIdx.x, a0.nb, 0u);
    else
        conv_body<T, BM, BN, WARPS_M, WARPS_N, BK, NS, MODE_CONV, false, false, KG, MT, LOADERS>(a1, blockIdx.x - nb0, a1.nb, 0u);
}

template <typename T, int BM, int BN, int MODE, int KG>
static hipError_t launch_fused_one(const ConvArgs &a_in, hipStream_t s) {
    ConvArgs a = a_in;
    a.nb = (a.M + BM - 1) / BM;
    constexpr int NS = RingDepth<BM, BN, 64>::value;
    constexpr size_t ring = (size_t)NS * (BM + BN) * 64 * 2;
    auto kern = conv_dlds_kernel<T, BM, BN, 2, 2, 64, NS, MODE, false, true, KG>;
    constexpr size_t bias_off = std::max<size_t>(ring, fused_lds_bytes(BM, BN, KG));
    static_assert(bias_off + (BN + kFusedMaxCout2 + BN) * 4 <= 160 * 1024, "fused form does not fit the LDS");
    const size_t need = bias_off + (size_t)(BN + a.Cout2 + (a.w3 ? BN : 0)) * 4;
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)(bias_off + (BN + kFusedMaxCout2 + BN) * 4));
    if (attr != hipSuccess) return attr;
    if (a.Cout2 % fused_chunk(BN, KG) != 0) return hipErrorInvalidValue;
    if (a.w3 && BN / (2 * KG) < 32) return hipErrorInvalidValue;   // the third layer needs whole 32-channel tiles per wave
    ConvRest<MODE, false, true> rest;
    rest.pack(a);
    kern<<<dim3((a.M + BM - 1) / BM, 1, 1), 256 * KG, need, s>>>(a.x, a.w, a.res, a.y, a.M, a.K, a.Cout | (conv_ldy(a) << 16), a.Cin | (conv_ldx(a) << 16), conv_pack_relu(a), 0u, rest CW_STAMP_PASS);
    return hipGetLastError();
}

void conv_fused_grid(int bm, int kg, const ConvArgs &a, dim3 *grid, int *block) {
    *grid = dim3((a.M + bm - 1) / bm, 1, 1);
    *block = 256 * kg;
}

bool conv_fused_ok(int bm, int kg, int cout, int cout2) {
    if ((cout != 64 && cout != 128) || (bm != 64 && bm != 128) || (bm == 128 && cout == 128) || (kg != 1 && kg != 2)) return false;
    return cout2 >= cout && cout2 % fused_chunk(cout, kg) == 0 && cout2 <= kFusedMaxCout2;
}

hipError_t launch_conv_fused(DType dt, int bm, int kg, const ConvArgs &a, hipStream_t s) {
    // first layer: any convolution this kernel takes, Cout 64 or 128, whole K in one workgroup;
    // second layer: 1x1 over its output with a residual
    if (a.Cin % 64 != 0 || a.K != a.kh * a.kw * a.Cin || a.K % 64 != 0 || a.split_k != 1 || a.ktiles_per_split != a.K / 64 || a.partial)
        return hipErrorInvalidValue;
    if (!conv_fused_ok(bm, kg, a.Cout, a.Cout2)) return hipErrorInvalidValue;
    if (!a.w2 || !a.bias2) return hipErrorInvalidValue;
    if (a.wd ? (a.Cout != 64 || !a.x2 || !a.biasd) : !a.res) return hipErrorInvalidValue;
    if (!a.res && !a.wd) return hipErrorInvalidValue;
    // third layer: over the second layer's output, as many channels as the first layer has; with the projection
    // form only as one wave group (the 64-channel form is planned that way)
    if (a.w3 && ((a.wd && kg != 1) || !a.bias3 || !a.y3 || (long long)a.M * a.Cout * 2 >= (1ll << 31) || (long long)a.Cout * a.Cout2 * 2 >= (1ll << 31)))
        return hipErrorInvalidValue;
    if (a.nz > 1) return hipErrorInvalidValue;   // the batched form's strides share their place with the third layer's pointers
    if (a.kh * a.kw > 32 || (long long)a.M * a.Cout2 * 2 >= (1ll << 31) || (long long)a.Cout * a.K * 2 >= (1ll << 31)) return hipErrorInvalidValue;
    if (conv_ldx(a) != a.Cin || conv_ldy(a) != a.Cout) return hipErrorInvalidValue;   // the fused form takes dense tensors only
    if ((long long)a.B * a.H * a.W * a.Cin * 2 + (long long)(conv_pad_h(a) * a.W + conv_pad_w(a)) * a.Cin * 2 >= (1ll << 31)) return hipErrorInvalidValue;
    const bool gemm = a.kh == 1 && a.kw == 1 && a.stride == 1 && a.pad == 0;
#define CW_FUSED_T(T_, BM_, BN_, KG_) return gemm ? launch_fused_one<T_, BM_, BN_, MODE_GEMM, KG_>(a, s) : launch_fused_one<T_, BM_, BN_, MODE_CONV, KG_>(a, s)
#define CW_FUSED(BM_, BN_)                                                       \
    do {                                                                         \
        if (dt == DT_F16) {                                                      \
            if (kg == 2) { CW_FUSED_T(f16, BM_, BN_, 2); }                       \
            CW_FUSED_T(f16, BM_, BN_, 1);                                        \
        }                                                                        \
        if (kg == 2) { CW_FUSED_T(bf16, BM_, BN_, 2); }                          \
        CW_FUSED_T(bf16, BM_, BN_, 1);                                           \
    } while (0)
    if (a.Cout == 64 && bm == 128) CW_FUSED(128, 64);
    if (a.Cout == 64) CW_FUSED(64, 64);
    CW_FUSED(64, 128);
#undef CW_FUSED
#undef CW_FUSED_T
}

template <typename T, int BM, int BN, int WARPS_M, int WARPS_N, int BK, int KG, int MT, bool LOADERS>
static hipError_t launch_pair_form(const ConvArgs &a0, const ConvArgs &a1, unsigned nb0, unsigned nb1, hipStream_t s) {
    constexpr int NS = RingDepth<BM, BN, BK>::value;
    constexpr size_t stage_bytes = (size_t)(BM + BN) * BK * 2;
    auto kern = conv_dlds_pair_kernel<T, BM, BN, WARPS_M, WARPS_N, BK, NS, KG, MT, LOADERS>;
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)(NS * stage_bytes));
    if (attr != hipSuccess) return attr;
    const size_t used = std::max((size_t)std::min(NS, std::max(a0.ktiles_per_split, a1.ktiles_per_split)) * stage_bytes, (size_t)(KG >= 4 || LOADERS ? KG : KG - 1) * BM * BN * 4);
    ConvLines l0, l1;
    memcpy(&l0, &a0, sizeof l0);
    memcpy(&l1, &a1, sizeof l1);
    kern<<<dim3((nb0 + nb1) * conv_parts<BM, BN, MT>(), 1, 1), conv_threads<WARPS_M, WARPS_N, KG, LOADERS>(), used, s>>>(l0, l1);
    return hipGetLastError();
}

template <typename T, int BM, int BN, int WARPS_M, int WARPS_N, int BK, int KG, int MT = 32>
static hipError_t launch_pair_one(const ConvArgs &a0_in, const ConvArgs &a1_in, hipStream_t s) {
    ConvArgs a0 = a0_in, a1 = a1_in;
    constexpr int TM = MT == 16 ? 32 : BM, TN = MT == 16 ? 32 : BN, WAVES = WARPS_M * WARPS_N * KG;
    const unsigned nb0 = ((a0.M + TM - 1) / TM) * ((a0.Cout + TN - 1) / TN), nb1 = ((a1.M + TM - 1) / TM) * ((a1.Cout + TN - 1) / TN);
    if (!conv_panel_ok(a0, TN, nb0) || !conv_panel_ok(a1, TN, nb1)) return hipErrorInvalidValue;
    a0.nb = conv_pack_nb((int)nb0, a0.panel_log2);
    a1.nb = conv_pack_nb((int)nb1, a1.panel_log2);
    if constexpr (conv_has_loaders(MODE_CONV, false, false, BM, BN, WAVES, KG)) {
        if (conv_loads_apart(MODE_CONV, true, BM, BN, BK, WAVES, std::max(a0.K, a1.K), (long long)nb0 + nb1))
            return launch_pair_form<T, BM, BN, WARPS_M, WARPS_N, BK, KG, MT, true>(a0, a1, nb0, nb1, s);
    }
    return launch_pair_form<T, BM, BN, WARPS_M, WARPS_N, BK, KG, MT, false>(a0, a1, nb0, nb1, s);
}

bool conv_pair_tile_ok(ConvTile tile) {
    switch (tile) {
        case T128x64: case T128x64k128: case T64x64: case T64x64k128: case T64x32k128: case T32x64k128: case T32x32k128:
        case T32x32k128g4: case T64x64k128g2: case T128x128: case T128x128w8: case T32x32: case T32x32g4:
        case T32x32k128g4q: case T32x32k128g4n: case T32x32k128g4m: return true;
        default: return false;
    }
}

static bool conv_pair_member_ok(const ConvArgs &a, int bk) {
    if (a.Cin % bk != 0 || a.K != a.kh * a.kw * a.Cin || a.kwp != a.kw || a.kh * a.kw > 32 || a.split_k != 1 || a.partial) return false;
    if (a.ktiles_per_split != a.K / bk || a.M <= 0 || a.Cout % 32 != 0) return false;
    if (conv_ldx(a) < a.Cin || conv_ldy(a) < a.Cout) return false;
    if ((long long)a.B * a.H * a.W * conv_ldx(a) * 2 + (long long)(conv_pad_h(a) * a.W + conv_pad_w(a)) * conv_ldx(a) * 2 >= (1ll << 31)) return false;
    return (long long)a.M * conv_ldy(a) * 2 < (1ll << 31) && (long long)a.Cout * a.K * 2 < (1ll << 31);
}

void conv_pair_grid(ConvTile tile, const ConvArgs &a0, const ConvArgs &a1, dim3 *grid, int *block) {
    const TileDim d = conv_tile_dim(tile);
    *grid = dim3(((a0.M + d.bm - 1) / d.bm) * ((a0.Cout + d.bn - 1) / d.bn) + ((a1.M + d.bm - 1) / d.bm) * ((a1.Cout + d.bn - 1) / d.bn), 1, d.parts());
    *block = d.threads;
}

hipError_t launch_conv_pair(DType dt, ConvTile tile, const ConvArgs &a0, const ConvArgs &a1, hipStream_t s) {
    if (!conv_pair_tile_ok(tile)) return hipErrorInvalidValue;
    const int bk = conv_tile_dim(tile).bk;
    if (!conv_pair_member_ok(a0, bk) || !conv_pair_member_ok(a1, bk)) return hipErrorInvalidValue;
#define CW_PAIR(BM_, BN_, WM_, WN_, BK_, ...)                                                           \
    return dt == DT_F16 ? launch_pair_one<f16, BM_, BN_, WM_, WN_, BK_, __VA_ARGS__>(a0, a1, s) : launch_pair_one<bf16, BM_, BN_, WM_, WN_, BK_, __VA_ARGS__>(a0, a1, s)
    switch (tile) {
        case T128x64: CW_PAIR(128, 64, 2, 2, 64, 1);
        case T128x64k128: CW_PAIR(128, 64, 2, 2, 128, 1);
        case T64x64: CW_PAIR(64, 64, 2, 2, 64, 1);
        case T64x64k128: CW_PAIR(64, 64, 2, 2, 128, 1);
        case T64x32k128: CW_PAIR(64, 32, 2, 1, 128, 1);
        case T32x64k128: CW_PAIR(32, 64, 1, 2, 128, 1);
        case T32x32k128: CW_PAIR(32, 32, 1, 1, 128, 1);
        case T32x32k128g4: CW_PAIR(32, 32, 1, 1, 128, 4);
        case T64x64k128g2: CW_PAIR(64, 64, 2, 2, 128, 2);
        case T128x128: CW_PAIR(128, 128, 2, 2, 64, 1);
        case T128x128w8: CW_PAIR(128, 128, 2, 4, 64, 1);
        case T32x32: CW_PAIR(32, 32, 1, 1, 64, 1);
        case T32x32g4: CW_PAIR(32, 32, 1, 1, 64, 4);
        case T32x32k128g4q: CW_PAIR(16, 16, 1, 1, 128, 4, 16);
        case T32x32k128g4n: CW_PAIR(32, 16, 1, 1, 128, 4, 16);
        case T32x32k128g4m: CW_PAIR(16, 32, 1, 1, 128, 4, 16);
        default: return hipErrorInvalidValue;
    }
#undef CW_PAIR
}

// Called by launch_conv (which has validated the shapes) for every convolution with
// Cin % 64 == 0 and for a first convolution in stem form; bk = conv_bk() of the shape under
// this tile.
hipError_t launch_conv_dlds(DType dt, ConvTile tile, int bk, int mode, const ConvArgs &a, hipStream_t s) {
    if (mode == MODE_STEM) {
        if (bk != 64 || a.Cin != 4 || a.K != 256 || a.kwp != 8 || a.khp != 8 || a.pad != 0 || a.stride % 2 != 0 || a.W % 2 != 0)
            return hipErrorInvalidValue;
        // every 8-tap window must start inside the (padded) image
        if ((a.Ho - 1) * a.stride >= a.H || (a.Wo - 1) * a.stride >= a.W) return hipErrorInvalidValue;
    } else if ((bk != 64 && bk != 128 && bk != 256) || (a.Cin % bk != 0) != (mode == MODE_TAIL) || a.K != a.kh * a.kw * a.Cin) {
        return hipErrorInvalidValue;
    }
    if (mode == MODE_TAIL) return launch_conv_dlds_tail(dt, tile, a.split_k > 1, a, s);
    return dt == DT_F16 ? launch_conv_tiles_f16(tile, bk, mode, a, s) : launch_conv_tiles_bf16(tile, bk, mode, a, s);
}

}  // namespace cw

#ifdef CW_STAMPS
ulonglong2 *cw::cw_stamps = nullptr;
unsigned cw::cw_stamp_next = 0;
extern "C" {
// The next convolution launch is number 0 again (call it before the first one); the stamps of launch l's first workgroups.
int32_t cw_stamps_reset(void) {
    const size_t bytes = (size_t)cw::kStampLaunches * cw::kStampGroups * sizeof(ulonglong2);
    if (!cw::cw_stamps && (hipMalloc(reinterpret_cast<void **>(&cw::cw_stamps), bytes) != hipSuccess ||
                           hipMemset(cw::cw_stamps, 0, bytes) != hipSuccess || hipDeviceSynchronize() != hipSuccess)) return -1;
    cw::cw_stamp_next = 0;
    return 0;
}
int32_t cw_stamps_read(uint32_t launch, uint32_t groups, unsigned long long *host) {
    return hipMemcpy(host, cw::cw_stamps + (size_t)(launch % cw::kStampLaunches) * cw::kStampGroups,
                     (groups < cw::kStampGroups ? groups : cw::kStampGroups) * sizeof(ulonglong2), hipMemcpyDeviceToHost) == hipSuccess ? 0 : -1;
}
}
#endif
