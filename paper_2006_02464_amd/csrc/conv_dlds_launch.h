// Entry point and launch of one convolution on the direct-to-LDS kernel, for the files that instantiate it.
#pragma once
#include "conv_loader_body.h"

namespace cw {

#ifdef CW_STAMPS
// A build for tune.py: workgroup b of convolution launch number l since the last reset leaves {start, end} in ticks of 10 ns at
// cw_stamps[(l % kStampLaunches) * kStampGroups + b], end = the stores of all its waves have been taken (in wave groups every wave
// ends by itself).  Nothing before the first reset, which allocates the room.
constexpr unsigned kStampLaunches = 256, kStampGroups = 16384;
extern ulonglong2 *cw_stamps;
extern unsigned cw_stamp_next;
#define CW_STAMP_ARG , ulonglong2 *stamps
#define CW_STAMP_BEGIN const unsigned long long stamp_from = __builtin_amdgcn_s_memrealtime();
#define CW_STAMP_END                                                                                            \
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                                                            \
    __syncthreads();                                                                                            \
    const unsigned stamp = blockIdx.x + conv_nb_tiles(nb) * conv_parts<BM, BN, MT>() * blockIdx.y;              \
    if (threadIdx.x == 0 && stamps && stamp < kStampGroups)                                                     \
        stamps[stamp] = make_ulonglong2(stamp_from, __builtin_amdgcn_s_memrealtime());
#define CW_STAMP_PASS , cw_stamps ? cw_stamps + (size_t)(cw_stamp_next++ % kStampLaunches) * kStampGroups : nullptr
#else
#define CW_STAMP_ARG
#define CW_STAMP_BEGIN
#define CW_STAMP_END
#define CW_STAMP_PASS
#endif

// Workgroups of a tile: of the forms on 16x16 MFMA tiles a workgroup computes a BM x BN part of a 32x32 tile.
template <int BM, int BN, int MT>
constexpr int conv_parts() { return MT == 16 ? (32 / BM) * (32 / BN) : 1; }

// What a form of the kernel reads of ConvArgs beyond the leading scalars.  The runtime copies a launch's arguments to the device
// by the byte: 320 of them cost the issuing thread 0.4 us more than 128, as much as a ninth of the launch, and an EXEC by graph replay
// 4.4 us at batch 1 (ResNet-50, 211.9 -> 207.5).
template <int MODE, bool SPLITK, bool FUSED>
struct alignas(64) ConvRest {   // general addressing: one line of geometry, then what is needed late
    int32_t B, H, W, Ho, Wo, kh, kw, stride, pad;
    FastDiv wo_div, ho_div;
    int32_t Cout2;
    const float *bias;
    const void *w2;
    int32_t split_k, ktiles_per_split;
    float *partial;
    int32_t *counters;
    void pack(const ConvArgs &a) {
        B = a.B; H = a.H; W = a.W; Ho = a.Ho; Wo = a.Wo; kh = a.kh; kw = a.kw; stride = a.stride; pad = a.pad; wo_div = a.wo_div; ho_div = a.ho_div;
        Cout2 = a.Cout2; bias = a.bias; w2 = a.w2; split_k = a.split_k; ktiles_per_split = a.ktiles_per_split; partial = a.partial; counters = a.counters;
    }
    __device__ __forceinline__ void unpack(ConvArgs &a) const {
        a.B = B; a.H = H; a.W = W; a.Ho = Ho; a.Wo = Wo; a.kh = kh; a.kw = kw; a.stride = stride; a.pad = pad; a.wo_div = wo_div; a.ho_div = ho_div;
        a.bias = bias;
        if constexpr (SPLITK) { a.split_k = split_k; a.ktiles_per_split = ktiles_per_split; a.partial = partial; a.counters = counters; }
    }
};
template <int MODE>
struct alignas(64) ConvRestGemm {   // 1x1 stride 1: B*H*W = M, one tap
    const float *bias;
    const void *w2;
    int32_t Cout2;
    int32_t split_k;
    union {
        struct { long long zs_x, zs_w, zs_y; };   // batched form
        struct { float *partial; int32_t *counters; long long ktiles_per_split; };
    };
    void pack(const ConvArgs &a) {
        bias = a.bias; w2 = a.w2; Cout2 = a.Cout2; split_k = a.split_k;
        if (a.split_k > 1) { partial = a.partial; counters = a.counters; ktiles_per_split = a.ktiles_per_split; }
        else { zs_x = a.zs_x; zs_w = a.zs_w; zs_y = a.zs_y; }
    }
    template <bool SPLITK>
    __device__ __forceinline__ void unpack_gemm(ConvArgs &a) const {
        a.B = 1; a.H = 1; a.W = a.M; a.Ho = 1; a.Wo = a.M; a.kh = 1; a.kw = 1; a.stride = 1; a.pad = 0;
        a.bias = bias;
        if constexpr (SPLITK) { a.split_k = split_k; a.ktiles_per_split = (int)ktiles_per_split; a.partial = partial; a.counters = counters; }
    }
};
template <bool SPLITK>
struct alignas(64) ConvRest<MODE_GEMM, SPLITK, false> : ConvRestGemm<MODE_GEMM> {
    __device__ __forceinline__ void unpack(ConvArgs &a) const { this->template unpack_gemm<SPLITK>(a); }
};
template <bool SPLITK>
struct alignas(64) ConvRest<MODE_TAIL, SPLITK, false> : ConvRestGemm<MODE_TAIL> {
    __device__ __forceinline__ void unpack(ConvArgs &a) const { this->template unpack_gemm<SPLITK>(a); }
};
template <int MODE>
struct ConvRest<MODE, false, true> : ConvArgs {   // the fused form reads all of it
    void pack(const ConvArgs &a) { static_cast<ConvArgs &>(*this) = a; }
    __device__ __forceinline__ void unpack(ConvArgs &a) const { a = *this; }
};

template <int WARPS_M, int WARPS_N, int KG, bool LOADERS>
constexpr int conv_threads() { return 64 * (WARPS_M * WARPS_N * KG + (LOADERS ? kLoaderWaves : 0)); }

// The tile on the body that is the form's.
template <typename T, int BM, int BN, int WARPS_M, int WARPS_N, int BK, int NS, int MODE, bool SPLITK, bool FUSED, int KG, int MT, bool LOADERS>
static __device__ __forceinline__ void conv_body(const ConvArgs &a, const int bid, const int nb, const unsigned magic) {
    if constexpr (LOADERS) conv_loader_body<T, BM, BN, WARPS_M, WARPS_N, BK, NS, MODE, KG>(a, bid, nb, magic);
    else conv_dlds_body<T, BM, BN, WARPS_M, WARPS_N, BK, NS, MODE, SPLITK, FUSED, KG, false, MT>(a, bid, nb);
}

template <typename T, int BM, int BN, int WARPS_M, int WARPS_N, int BK, int NS, int MODE, bool SPLITK, bool FUSED = false, int KG = 1, int MT = 32, bool LOADERS = false>
__global__ __launch_bounds__((conv_threads<WARPS_M, WARPS_N, KG, LOADERS>())) void conv_dlds_kernel(const void *x, const void *w, const void *res, void *y,
                                                                                 int M, int K, int cout_ldy, int cin_ldx, unsigned nb_relu, unsigned magic,
                                                                                 const ConvRest<MODE, SPLITK, FUSED> rest CW_STAMP_ARG) {
    CW_STAMP_BEGIN
    // The ten leading arguments (14 dwords, all the user SGPRs there are beside the argument
    // pointer): this file is compiled with kernel-argument preloading, so
    // they are in SGPRs when a wave starts and the first address arithmetic does not wait for a
    // load of the argument block.  Everything else is read from `rest` when it is needed.
    // Cout and Cin carry the pixel pitches of y and x in their upper halves, so that the 1x1 form
    // still needs nothing beyond the preloaded scalars for its addressing, and the tile count the activation in its top two bits (in
    // the argument block, a load of it stays in flight across the K walk, and every LDS read there then waits for all of them).
    const int nb = (int)(nb_relu & 0x3fffffffu);
    ConvArgs a;
    a.x = x; a.w = w; a.res = res; a.y = y;
    a.M = M; a.K = K;
    rest.unpack(a);
    a.x = x; a.w = w; a.res = res; a.y = y;
    a.M = M; a.K = K; a.Cout = cout_ldy & 0xffff; a.Cin = cin_ldx & 0xffff; a.nb = nb; a.relu = (int)(nb_relu >> 30);
    a.ld = (int)(((unsigned)cin_ldx >> 16) | ((unsigned)cout_ldy & 0xffff0000u));
    if constexpr (MODE == MODE_GEMM && !SPLITK && !FUSED && MT == 32) {
        // batched form: one GEMM per blockIdx.z, operands advanced by the strides in the last argument line
        if (blockIdx.z != 0) {
            a.x = static_cast<const char *>(x) + (long long)blockIdx.z * rest.zs_x;
            a.w = static_cast<const char *>(w) + (long long)blockIdx.z * rest.zs_w;
            a.y = static_cast<char *>(y) + (long long)blockIdx.z * rest.zs_y;
        }
    }
    if constexpr (FUSED || SPLITK || MODE == MODE_STEM) {
        conv_body<T, BM, BN, WARPS_M, WARPS_N, BK, NS, MODE, SPLITK, FUSED, KG, MT, LOADERS>(a, blockIdx.x, nb, magic);
        CW_STAMP_END
    } else if (__builtin_expect((int)blockIdx.x < conv_nb_tiles(nb) * conv_parts<BM, BN, MT>(), 1)) {
        conv_body<T, BM, BN, WARPS_M, WARPS_N, BK, NS, MODE, SPLITK, FUSED, KG, MT, LOADERS>(a, blockIdx.x, nb, magic);
        CW_STAMP_END
    } else {   // a workgroup that reads ahead (its code behind the convolution's, which most launches find cold)
        const int wgs = conv_nb_tiles(nb) * conv_parts<BM, BN, MT>();
        constexpr int readers = conv_prefetch_threads(conv_threads<WARPS_M, WARPS_N, KG, LOADERS>());
        if ((int)threadIdx.x >= readers) return;
        const int nt = ((int)gridDim.x - wgs) * readers, lines = rest.Cout2;
        const char *p = static_cast<const char *>(rest.w2);
        for (int i = ((int)blockIdx.x - wgs) * readers + (int)threadIdx.x; i < lines; i += nt * kPrefetchPerThread) {
            unsigned v[kPrefetchPerThread];
#pragma unroll
            for (int u = 0; u < kPrefetchPerThread; ++u)
                v[u] = *reinterpret_cast<const unsigned *>(p + (size_t)min(i + u * nt, lines - 1) * 128);
#pragma unroll
            for (int u = 0; u < kPrefetchPerThread; ++u) asm volatile("" : : "v"(v[u]));
        }
    }
}

static inline uint32_t conv_pack_relu(const ConvArgs &a) { return (uint32_t)a.nb | (uint32_t)a.relu << 30; }   // panel_log2 <= 3: bits 28 and 29

// A tile numbering in 2^p panels needs the channel tiles to divide evenly, and the tile count must
// leave the bits above kPanelShift free.
static bool conv_panel_ok(const ConvArgs &a, int bn, unsigned tiles) {
    if (tiles >= (1u << kPanelShift) || a.panel_log2 < 0 || a.panel_log2 > 3) return false;
    const int tiles_n = (a.Cout + bn - 1) / bn;
    return a.panel_log2 == 0 || tiles_n % (1 << a.panel_log2) == 0;
}

template <typename T, int BM, int BN, int WARPS_M, int WARPS_N, int BK, int MODE, bool SPLITK, int KG, int MT, bool LOADERS>
static hipError_t launch_form(dim3 grid, const ConvArgs &a, hipStream_t s) {
    ConvRest<MODE, SPLITK, false> rest;
    rest.pack(a);
    constexpr int NS = RingDepth<BM, BN, BK>::value;
    constexpr size_t stage_bytes = (size_t)(BM + BN) * BK * 2;
    static_assert(NS * stage_bytes <= 160 * 1024, "ring does not fit the LDS");
    auto kern = conv_dlds_kernel<T, BM, BN, WARPS_M, WARPS_N, BK, NS, MODE, SPLITK, false, KG, MT, LOADERS>;
    // More than 64 KiB of LDS per workgroup has to be requested once per kernel; done on first
    // use (under LOAD's graph recording or the first plain EXEC), never per launch afterwards.
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)(NS * stage_bytes));
    if (attr != hipSuccess) return attr;
    const uint32_t magic = conv_tile_magic(grid.x, (unsigned)(a.Cout + BN - 1) / BN);
    // a K walk shorter than the ring only ever touches its first stages (the wave groups' exchange
    // at the end needs its own room)
    if (!SPLITK && MODE != MODE_STEM && a.Cout2 > 0 && a.w2 && a.nz <= 1) grid.x += conv_prefetch_wgs(a.Cout2);
    const size_t used = std::max((size_t)std::min(NS, a.ktiles_per_split) * stage_bytes, (size_t)(KG >= 4 || LOADERS ? KG : KG - 1) * BM * BN * 4);
    kern<<<grid, conv_threads<WARPS_M, WARPS_N, KG, LOADERS>(), used, s>>>(a.x, a.w, a.res, a.y, a.M, a.K, a.Cout | (conv_ldy(a) << 16), a.Cin | (conv_ldx(a) << 16), conv_pack_relu(a), magic, rest CW_STAMP_PASS);
    return hipGetLastError();
}

template <typename T, int BM, int BN, int WARPS_M, int WARPS_N, int BK, int MODE, bool SPLITK, int KG = 1, int MT = 32>
static hipError_t launch_one(dim3 grid, int block, const ConvArgs &a_in, hipStream_t s) {
    ConvArgs a = a_in;
    if (!conv_panel_ok(a, BN, grid.x)) return hipErrorInvalidValue;
    a.nb = conv_pack_nb((int)grid.x, a.panel_log2);
    if (MODE == MODE_TAIL ? a.nz > 1 : a.K % BK != 0 && MODE != MODE_STEM) return hipErrorInvalidValue;
    if (!SPLITK && a.ktiles_per_split != (MODE == MODE_STEM ? (a.kh + 1) / 2 : (a.K + BK - 1) / BK)) return hipErrorInvalidValue;  // the kernel walks the whole K
    if (a.nz > 1 && (MT != 32 || MODE != MODE_GEMM || SPLITK || a.bias || a.res || grid.z != (unsigned)a.nz)) return hipErrorInvalidValue;
    constexpr unsigned PARTS = conv_parts<BM, BN, MT>();
    if (a.nz <= 1 && grid.z != PARTS) return hipErrorInvalidValue;
    constexpr int WAVES = WARPS_M * WARPS_N * KG;
    if (block != 64 * WAVES) return hipErrorInvalidValue;
    if (PARTS > 1) grid = dim3(grid.x * PARTS, grid.y, 1);   // the workgroups that read ahead come behind all the parts
    if constexpr (conv_has_loaders(MODE, SPLITK, false, BM, BN, WAVES, KG)) {
        if (conv_loads_apart(MODE, false, BM, BN, BK, WAVES, a.K, (long long)grid.x * grid.z))
            return launch_form<T, BM, BN, WARPS_M, WARPS_N, BK, MODE, SPLITK, KG, MT, true>(grid, a, s);
    }
    return launch_form<T, BM, BN, WARPS_M, WARPS_N, BK, MODE, SPLITK, KG, MT, false>(grid, a, s);
}

}  // namespace cw
