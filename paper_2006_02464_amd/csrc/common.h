// Internal types shared by the plan compiler, the kernels and the C ABI.
// gfx950 (CDNA4) only.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace cw {

typedef _Float16 f16;
typedef __bf16 bf16;

enum DType : int32_t { DT_F16 = 0, DT_BF16 = 1 };

// Kernel families (cw_launch_info.kind).
enum Kind : int32_t {
    K_CAST_INPUT = 0,  // fp32 NCHW -> storage-type NHWC4
    K_CONV = 1,        // implicit-GEMM convolution on MFMA, fused epilogue, optional split-K
    K_MAXPOOL = 3,
    K_GAVGPOOL = 4,
    K_FC = 5,
    K_SOFTMAX = 6,
    K_DWCONV = 7,      // depthwise convolution (one filter per channel), fused epilogue
    K_COPY_CHANNELS = 8,  // a tensor into a channel range of a wider one (CONCAT sources that cannot write there themselves)
    K_WINO_INPUT = 9,   // Winograd F(2x2, 3x3): input tiles -> 16 transformed matrices
    K_WINO_OUTPUT = 10, // ... 16 product matrices -> 2x2 output tiles, fused epilogue
    K_RESIDENT = 11,    // a run of convolution layers as one launch of resident workgroups (kernels_resident.hip)
};

// Activation codes (cw_op.relu, ConvArgs.relu / relu2).
enum Act : int32_t { ACT_NONE = 0, ACT_RELU = 1, ACT_HSWISH = 2 };

// Division by a run-time constant as multiply + shifts (Granlund-Montgomery round-up method).
struct FastDiv {
    uint32_t magic, sh1, sh2;
};
inline FastDiv make_fast_div(uint32_t d) {
    uint32_t l = 0;
    while ((1ull << l) < d) ++l;  // ceil(log2 d)
    FastDiv f;
    f.magic = (uint32_t)(((1ull << 32) * ((1ull << l) - d)) / d + 1);
    f.sh1 = l < 1 ? l : 1;
    f.sh2 = l > 0 ? l - 1 : 0;
    return f;
}

// Implicit GEMM view of a convolution (also used for the stem with Cin padded to 4 and
// the filter row padded to 8 taps): M = B*Ho*Wo output pixels, N = Cout, K = kh*kwp*Cin.
// The fields are ordered by who reads them, in runs of 64 bytes (the struct is aligned to that, and
// with it the kernel-argument segment): a workgroup's first instructions wait for every argument line
// they touch, and each further line costs a fixed fraction of a microsecond per launch.  Line 0
// is all a 1x1 stride-1 convolution without split-K reads; line 1 adds what the general
// addressing needs; split-K, the first convolution and the fused forms read on.
struct alignas(64) ConvArgs {
    // ---- line 0
    const void *x;      // NHWC [B][H][W][Cin]
    const void *w;      // packed [Cout][K], k = (r*kwp + s)*Cin + c
    const float *bias;  // [Cout]
    const void *res;    // NHWC like y, or nullptr
    void *y;            // NHWC [B][Ho][Wo][Cout]
    int32_t M, K;
    int32_t Cout, Cin;
    int32_t relu;
    int32_t nb;         // output tiles of this convolution = workgroups along x (set by the launch code)
    // ---- line 1
    int32_t B, H, W, Ho, Wo;
    int32_t kh, kw, stride;
    int32_t pad;        // padding in height | padding in width << 16 (conv_set_pad / conv_pad_h / conv_pad_w)
    FastDiv wo_div, ho_div;  // for m -> (image, row, column)
    int32_t ld;         // elements per pixel in memory: of x | of y << 16 (= Cin | Cout << 16 unless a tensor is
                        // a channel range of a wider one: CONCAT without copies); res is always dense
    // ---- line 2
    int32_t khp;        // filter rows in the packed weights (first convolution: may be padded to 8)
    int32_t split_k, ktiles_per_split;
    int32_t relu2;
    float *partial;     // split-K: [split][M][Cout] fp32, else nullptr
    int32_t *counters;  // split-K: one arrival counter per output tile, zero between launches
    // Fused second layer (launch_conv_fused only): a 1x1 stride-1 convolution over this one's
    // output, y = act2(res + bias2 + W2 * act(bias + W * x)).  `res`, `y` then belong to the second
    // layer ([M][Cout2]); the first layer's output is never stored.
    // In the plain form w2 and Cout2 name memory the launch reads ahead for a later one (conv_prefetch_*): Cout2 pieces
    // of 128 bytes from w2 on, 0 for none.
    const void *w2;      // packed [Cout2][Cout]
    const float *bias2;  // [Cout2]
    int32_t Cout2;
    int32_t kwp;         // filter columns in the packed weights (first convolution: padded to 8)
    // Optional projection shortcut computed in the same launch instead of read as `res`:
    // res[m][:] = biasd + Wd * x2[m][:], x2 = [M][Cout] pixels aligned with the output (a 1x1
    // stride-1 projection of a tensor with Cout channels).  wd == nullptr: `res` is read.
    const void *x2;      // NHWC [M][Cout]
    const void *wd;      // packed [Cout2][Cout]
    const float *biasd;  // [Cout2]
    // Batched form (1x1 stride-1 addressing, no split-K): nz > 1 runs nz independent GEMMs of this
    // shape in one launch; workgroups with blockIdx.z = z take x, w and y advanced by z times these
    // byte strides (bias and res are not used then).  Read only by z > 0.
    int32_t nz;
    int32_t panel_log2;  // host side only: tile numbering of this launch (conv_pack_nb); the kernel gets it inside its tile count
    union {
        struct { long long zs_x, zs_w, zs_y; };
        // Fused form only (never batched): a third layer, the 1x1 stride-1 convolution that reads the
        // second layer's output (the next bottleneck's reduce), y3 = act3(bias3 + W3 * y), Cout3 = Cout.
        // y is still stored (it is the next block's shortcut); y3 is stored besides.  w3 == nullptr: none.
        // Together with the in-launch projection (wd) only in the one-group form.
        struct { const void *w3; const float *bias3; void *y3; };
    };
    int32_t relu3;
};
static_assert(offsetof(ConvArgs, B) == 64 && offsetof(ConvArgs, khp) == 128 && sizeof(ConvArgs) == 256, "argument lines");
// Tile numbering.  A launch's workgroups go to the 8 XCDs in turn and each XCD keeps a contiguous run
// of tile numbers, so the numbering decides what an XCD's L2 has to fetch.  Numbering 0 walks the
// tiles row by row (all channel tiles of a block of pixels, then the next pixels): every XCD reads
// an eighth of the pixels and all the weights.  Numbering p > 0 cuts the channel tiles into 2^p
// panels and walks panel after panel: an XCD reads 1/2^p of the weights and 2^p/8 of the pixels,
// which is less traffic where the weights outweigh the activations (small M, long K).  The kernel
// receives  tiles | p << 28  as its tile count (a preloaded scalar: no argument load is waited for).
constexpr int kPanelShift = 28;
__host__ __device__ inline int conv_pack_nb(int tiles, int panel_log2) { return tiles | (panel_log2 << kPanelShift); }
__host__ __device__ inline int conv_nb_tiles(int nb) { return nb & ((1 << kPanelShift) - 1); }
__host__ __device__ inline int conv_nb_panel(int nb) { return (int)((unsigned)nb >> kPanelShift); }
__host__ __device__ inline int conv_pad_h(const ConvArgs &a) { return a.pad & 0xffff; }
__host__ __device__ inline int conv_pad_w(const ConvArgs &a) { return (int)((unsigned)a.pad >> 16); }
__host__ __device__ inline int conv_ldx(const ConvArgs &a) { return a.ld & 0xffff; }
__host__ __device__ inline int conv_ldy(const ConvArgs &a) { return (int)((unsigned)a.ld >> 16); }
inline void conv_set_pad(ConvArgs &a, int pad_h, int pad_w) { a.pad = pad_h | (pad_w << 16); }
inline void conv_set_ld(ConvArgs &a, int ldx, int ldy) { a.ld = ldx | (ldy << 16); }
// Reading ahead.  The weights of the next launches may have to come from HBM (several resident models outgrow the
// 256 MB last-level cache): workgroups behind a launch's tiles read one word of every 128 bytes of them, which brings them
// into that cache.  Measured, 3x3 of 256 channels at 14x14, batch 16, whose weights come from HBM: 12.0 -> 10.1 us a
// launch; with weights already in the cache 10.0 either way, and a whole ResNet-50 EXEC at batch 1 is 0.6 us longer for it.
constexpr int kPrefetchMinBytes = 256 * 1024;   // of a smaller tensor every workgroup that uses it waits for a miss or two at most
constexpr int kPrefetchMaxTiles = 512;   // two a CU, most of which run at once; behind more, the reads would come late
constexpr int kPrefetchLines = 256;      // per workgroup: a CU has only so many misses in flight (one workgroup per 4096 made ResNet-152 4 % slower)
constexpr int kPrefetchPerThread = 4;    // reads a thread has in flight
constexpr int conv_prefetch_wgs(int lines) { return lines < 64 * kPrefetchLines ? (lines + kPrefetchLines - 1) / kPrefetchLines : 64; }
// Threads of a workgroup that read; the others would take the lines of further workgroups, several times as many a CU.
constexpr int conv_prefetch_threads(int threads) { return threads < kPrefetchLines ? threads : kPrefetchLines; }
constexpr int kMaxChannels = 32768;  // channel counts and pitches travel in 16 bits

// Maps of at least this many pixels are averaged by the 16-wave kernel (one wave per 64 channels below).
constexpr int kGapWideFrom = 256;
// Depthwise convolution: y[m][c] = act(res[m][c] + bias[c] + sum_{r,s} x[pixel(m) + (r,s)][c] * w[r][s][c]).
struct DwArgs {
    const void *x;      // NHWC, ldx elements per pixel
    const void *w;      // packed [kh][kw][C]
    const float *bias;  // [C]
    const void *res;    // dense NHWC like y, or nullptr
    void *y;            // NHWC, ldy elements per pixel
    int32_t B, H, W, C, Ho, Wo, kh, kw, stride, pad, act, ldx, ldy;
    FastDiv c8_div, wo_div, ho_div;   // of the 3x3 form (set by the launch code)
};
// One output pixel a thread, taps one after the other; 3x3: all taps together; 3x3 stride 1: two pixels a thread.
enum DwForm { DW_ANY, DW_TAPS, DW_PAIRS };
constexpr unsigned kDwPairsFrom = 512;    // above so many workgroups of one pixel a thread
constexpr unsigned kDwPairThreads = 128;  // workgroup of the pairs
DwForm dw_form(const DwArgs &a);
dim3 dw_grid(const DwArgs &a);

// Winograd F(2x2, 3x3) for a 3x3 stride-1 pad-1 convolution.  Output pixels are cut into 2x2 tiles,
// th x tw per image (th = ceil(Ho/2), tw = ceil(Wo/2)), tiles = B*th*tw.  The input transform writes
// V[16][tiles][C]; after 16 GEMMs with the transformed weights U[16][Cout][C] (one batched launch
// of the convolution kernel), the output transform reads Mx[16][tiles][Cout] and writes y.
struct WinoArgs {
    const void *x;      // input transform: NHWC activations (ldx elements per pixel); output transform: Mx
    void *y;            // input transform: V; output transform: NHWC result (dense)
    const float *bias;  // output transform: [Cout]
    const void *res;    // output transform: dense NHWC like y, or nullptr
    int32_t B, H, W, C, th, tw, ldx, act;   // H, W: image size (= output size); C: channels of the tensor being transformed
};

// ---- resident multi-layer launch ---------------------------------------------------------------
// A run of consecutive convolution layers executed by ONE launch of 256 workgroups that stay on
// their CUs: the batch is cut into 8 partitions of B/8 images, partition p is computed by the 32
// workgroups that run on XCD p, and a layer's tiles start as soon as the tiles of the layers it reads
// (same partition, hence same XCD and same L2) have signalled completion through per-tile flags.
// Tile shapes the resident kernel holds (all on 4 waves, so that one workgroup can run any of them):
enum ResVariant : int32_t {
    RV_128x128 = 0, RV_128x64, RV_64x64, RV_128x64k128, RV_64x64k128, RV_32x32k128g4, RV_32x32g4, N_RES_VARIANTS
};
struct ResVariantDim { int bm, bn, bk; };
inline ResVariantDim res_variant_dim(int v) {
    switch (v) {
        case RV_128x128: return {128, 128, 64};
        case RV_128x64: return {128, 64, 64};
        case RV_64x64: return {64, 64, 64};
        case RV_128x64k128: return {128, 64, 128};
        case RV_64x64k128: return {64, 64, 128};
        case RV_32x32k128g4: return {32, 32, 128};
        default: return {32, 32, 64};
    }
}
// One layer of the program (device memory).  a.x, a.res and a.y hold byte offsets into the workspace
// of the tensors' first image, a.w and a.bias device addresses; partition p adds p * ps_*.
struct alignas(64) ResLayer {
    ConvArgs a;
    long long ps_x, ps_y, ps_res;
    int32_t variant;     // ResVariant; the addressing mode follows from the shape (1x1 stride 1: plain matrix)
    int32_t tiles;       // per partition
    int32_t dep[2];      // program indices of the layers that produce this layer's input and residual, or -1
    int32_t flag_base;   // this layer's first completion flag within a partition's flags
    int32_t pad_[3];
};
constexpr int kResPartitions = 8;          // = XCDs of the device
constexpr int kResGroupsPerPartition = 32; // workgroups per partition = CUs per XCD
// Workspace header behind the split-K counters: [epoch word at 0, abort word at byte 128 (holds the epoch of an
// abandoned launch), unused up to 256 B][completion flags]
constexpr size_t kResidentBytes = (size_t)1 << 20;
constexpr size_t kResidentFlagsOff = 256;
struct ResidentArgs {
    const ResLayer *layers;   // device
    int32_t n_layers;
    char *workspace;          // base the layers' activation offsets are relative to
    unsigned *flags;          // [kResPartitions][flags_per_part]
    int32_t flags_per_part;
    unsigned *epoch;          // flags equal to *epoch + 1 mean "done in this launch"
    unsigned *error;          // host-visible word: set when a wait times out or a workgroup is on the wrong XCD
    unsigned spin_limit;
};

struct CopyArgs {
    const void *src;    // [pixels][ld_src], the first C channels of every pixel are copied
    void *dst;          // [pixels][ld_dst] (already offset to the destination channel)
    int32_t pixels, C, ld_src, ld_dst;
};


struct CastArgs {
    const float *x;  // NCHW fp32 [B][C][H][W]
    void *y;         // NHWC4 [B][Hp][Wp][4]: the image inside a zero border of `pad` pixels
    int32_t B, C, H, W;
    int32_t pad, Hp, Wp;  // Hp = H + 2*pad, Wp = W + 2*pad rounded up to even
    int32_t *zero;        // n_zero words the launch also clears (the arrival counters of the launches behind it)
    int32_t n_zero;
};

// The head of a network as one launch (kernels_head.hip): first convolution (kh x kh, stride 2, packed filter rows of 8 taps x 4
// channels) over the fp32 images, with a 3x3 stride-2 pad-1 max pool and a 1x1 convolution cout -> n1 behind it or without.
struct HeadArgs {
    const float *x;       // NCHW fp32 [B][C][H][W]
    const void *w;        // packed [cout][8][8][4]
    const float *bias;
    void *y;              // NHWC: the pooled tensor, or the convolution's output
    const void *w1;       // packed [n1][cout]
    const float *bias1;
    void *y1;             // NHWC [B][Po][Qo]
    int32_t *zero;        // n_zero words the launch also clears
    int32_t n_zero, B, C, H, W, pad, Ho, Wo, Po, Qo, act, act1, ldy, ldy1;
    int32_t kh, cout, n1, pool;
    int32_t tiles_h, tiles_w;   // tiles of an image (set by the launch code)
};
constexpr int kHeadTallFrom = 256;   // pooled tiles of 7 x 8 from so many on (one a CU), 3 x 8 below, which is the shorter chain

struct PoolArgs {
    const void *x;  // NHWC
    void *y;        // NHWC (maxpool) / fp32 [B][C] (global average)
    int32_t B, H, W, C, Ho, Wo, k, stride, pad;
};

struct FcArgs {
    const float *f;  // [B][In] fp32
    const void *w;   // [Out][In]
    const float *bias;
    float *z;        // [B][Out]
    int32_t B, In, Out;
    // FC and softmax in one launch (p != nullptr; B <= 16, Out <= 1024): K is split over split_k
    // workgroups per 16 outputs, which meet through `partial` and arrival counters like the
    // convolution's split-K; the workgroup that finishes the last 16 outputs computes p = softmax(z).
    float *p;           // [B][Out] probabilities, or nullptr: logits only (the unfused kernel)
    float *partial;     // [split_k][16][Out] fp32 (split_k > 1); without p: [kFcWaves][B][Out rounded up to 16], z is left to the softmax
    int32_t *counters;  // ceil(Out/16) + 1 arrival counters, zero between launches
    int32_t split_k;    // 1, 2 or 4; In % (128 * split_k) == 0
    // The global average pool in the FC's launch (px != nullptr): no f, the averages stay in LDS.
    const void *px;     // [B][hw][In] in the storage type
    int32_t hw;
};
// Every workgroup of the FC then pools the whole map: each of its eight waves its own part of the channels, in items of 64 channels of a
// sample.  The pool's launch and round trip are worth 8 loads a lane, 1, 2 or 4 items (the return value, 0: launches of their
// own) times 8 pixels each: EXEC of ResNet-18 64x64 batch 1 87.4 -> 85.2 us, batch 4 88.6 -> 86.3, 224x224 batch 1 94.7 -> 92.5, ResNet-50
// 97x97 batch 1 184.1 -> 183.1; with 16 to 32 loads it is the other way round (ResNet-50 224x224 batch 1, 28 loads, 197.7 -> 200.3;
// MobileNet 150x99 batch 3, 18, 88.6 -> 95.6), and eight items do not fit the registers beside their weights.
constexpr int pool_fc_items(int64_t B, int64_t in, int64_t hw) {
    if (B < 1 || in < 1 || hw < 1 || in % 512 != 0 || in / 512 * B > 4) return 0;
    const int items = (int)(in / 512 * B), g = items == 3 ? 4 : items;
    return g * ((hw + 7) / 8) <= 8 ? g : 0;
}
constexpr int kFcSoftmaxMaxBatch = 16, kFcSoftmaxMaxOut = 1024;

// The FC's parts of K, each a sum of its own: by the waves of a workgroup, or (fc_in_parts) by workgroups, for the softmax to add up.  Up to 1024
// features, where the weights' way to the chip is the smaller part: whole EXECs by graph replay, of which two processes of one side differ by up to 0.6 %, DenseNet batch 6
// 206.7 -> 204.7 us, Inception batch 5 92.7 -> 91.2, ResNet-18 batch 8 133.9 -> 132.6; with 2048 from eight samples on, ResNet-50 batch 16 421.1 -> 419.3, no more than that
// difference (batch 4 267.5 -> 268.3, batch 1 204.4 -> 205.9: the launch is 1.7 us shorter, the softmax, which fetches the parts from other XCDs' L2s, 0.7 us longer).
constexpr int kFcWaves = 8, kFcPartsMaxOut = 1024;
constexpr bool fc_in_parts(int64_t B, int64_t in, int64_t out) {
    return out <= kFcPartsMaxOut && in % (32 * kFcWaves) == 0 && (in <= 1024 || (B >= 8 && in <= 4096)) && (B + 15) / 16 * ((out + 15) / 16) <= 256;
}

struct SoftmaxArgs {
    const float *z;
    float *p;
    int32_t B, D;
    unsigned *done;   // gets `seq` as the launch begins (launch_wait_done), or nullptr
    unsigned seq;
    const float *partial;   // the FC's parts instead of z, which is then written (FcArgs::partial), or nullptr
    const float *bias;
};

// Tile shapes the conv kernel is instantiated for (fixed at plan time per layer).
// (pixels x channels per workgroup; "wN" = N waves when not 4, each wave then owning 64x64;
// "k128" = K slices of 128 instead of 64, for Cin % 128 == 0; "gN" = N groups of waves that split
// every K slice between them and add up at the end; the four from 256x128w8 on are for large GEMMs:
// 8 waves of 64x64 or 64x128 each, and 256x128 on 4 waves of 128x64; "k256": K slices of 256 for
// long K and few tiles, Cin % 256 == 0; the last five: a 32x32 tile in parts on workgroups of their own,
// "q" quarters, "n" halves of its channels, "m" halves of its pixels, on 16x16x32 matrix instructions)
enum ConvTile : int32_t {
    T128x128 = 0, T128x64, T64x64, T64x32, T32x64, T32x32, T128x64w2, T64x128w2, T256x64, T128x128w8,
    T128x64k128, T64x64k128, T64x32k128, T32x64k128, T32x32k128,
    T128x64k128g2, T64x64k128g2, T64x64k128g4, T64x32k128g4, T32x64k128g4, T32x32k128g4,
    T32x32k128g8, T128x64g2, T64x64g2, T32x32g4,
    T256x128w8, T128x256w8, T256x256w8, T256x128,
    T32x32k256g4, T32x32k256g8, T64x32k256g4, T64x32k256g8, T32x64k256g4, T32x64k256g8, T64x64k256g4,
    T32x32k128g4q, T32x32k128g4n, T32x32k128g4m, T32x32k256g4q, T32x32k256g4n, N_CONV_TILES
};
struct TileDim {
    int bm, bn, threads, bk, kg;   // threads: of the waves that multiply; those that only load (conv_loader_threads) come on top
    int pm = bm, pn = bn;   // what one workgroup computes of it
    int parts() const { return (bm / pm) * (bn / pn); }
};
TileDim conv_tile_dim(ConvTile t);
// Split-K arrival counters of an output tile: one, or one per wave where the wave groups finish the tile together.
inline int conv_counters_per_tile(ConvTile t) { const TileDim d = conv_tile_dim(t); return d.kg >= 4 ? d.parts() * (d.threads / 64) : 1; }
// The same tile with K slices of 64 (for shapes a k128 tile cannot take).
ConvTile conv_tile_k64(ConvTile t);
// The same tile with one group of waves (split-K needs that).
ConvTile conv_tile_one_group(ConvTile t);
// The largest tile of the register-staged kernel that is no larger than t (that kernel has the ten
// basic shapes only; it serves what conv_uses_dlds does not name).
ConvTile conv_tile_staged(ConvTile t);
// The tile of the 1x1 form that ends in part of a K slice (which has some of the one-group shapes) nearest to t.
ConvTile conv_tile_tail(ConvTile t);
// Whether a convolution runs on the direct-to-LDS kernel (else on the register-staged one).
bool conv_uses_dlds(const ConvArgs &a, bool stem);

// Tiles in parts (kernels_conv_small.hip): a launch has grid.x * grid.z workgroups, grid.z = parts of a tile.
inline bool conv_tile_small(ConvTile t) { return t >= T32x32k128g4q && t < N_CONV_TILES; }

// Threads of a convolution launch (of a pair with a1) that only load, beside conv_grid's; 0 where its waves load for themselves.
int conv_loader_threads(ConvTile tile, bool stem, const ConvArgs &a, const ConvArgs *a1 = nullptr);

// Launchers (kernels_*.hip).  All only enqueue; they return the launch's error state.
hipError_t launch_conv(DType dt, ConvTile tile, bool stem, const ConvArgs &a, hipStream_t s);
// The direct-to-LDS kernel for Cin % 64 == 0, for 1x1 stride-1 convolutions over any Cin % 32 == 0 and for a first
// convolution in its stem form (called by launch_conv after its checks); mode = the kernel's addressing mode.
hipError_t launch_conv_dlds(DType dt, ConvTile tile, int bk, int mode, const ConvArgs &a, hipStream_t s);
// Its 1x1 form whose K ends in part of a slice (kernels_conv_tail.hip) and its K slices of 256 (kernels_conv_k256.hip;
// both called by launch_conv_dlds).
hipError_t launch_conv_tiles_f16(ConvTile tile, int bk, int mode, const ConvArgs &a, hipStream_t s);    // its tiles by storage type
hipError_t launch_conv_tiles_bf16(ConvTile tile, int bk, int mode, const ConvArgs &a, hipStream_t s);
hipError_t launch_conv_dlds_small(DType dt, ConvTile tile, int mode, bool splitk, const ConvArgs &a, hipStream_t s);
hipError_t launch_conv_dlds_tail(DType dt, ConvTile tile, bool splitk, const ConvArgs &a, hipStream_t s);
hipError_t launch_conv_dlds_k256(DType dt, ConvTile tile, int mode, bool splitk, const ConvArgs &a, hipStream_t s);
// A convolution (Cin % 64 == 0, Cout 64 or 128) and the 1x1 convolution that consumes it, in one
// launch (kernels_conv_dlds.hip).  bm = pixels per workgroup (64 or 128).
hipError_t launch_conv_fused(DType dt, int bm, int kg, const ConvArgs &a, hipStream_t s);
// Workgroups of that launch.
void conv_fused_grid(int bm, int kg, const ConvArgs &a, dim3 *grid, int *block);
bool conv_fused_ok(int bm, int kg, int cout, int cout2);   // a (pixels per workgroup, wave groups) form exists for these widths
// Two convolutions over the same input tensor in one launch (kernels_conv_dlds.hip), both on `tile`
// (one of conv_pair_tile_ok), neither split along K.
hipError_t launch_conv_pair(DType dt, ConvTile tile, const ConvArgs &a0, const ConvArgs &a1, hipStream_t s);
bool conv_pair_tile_ok(ConvTile tile);
void conv_pair_grid(ConvTile tile, const ConvArgs &a0, const ConvArgs &a1, dim3 *grid, int *block);
hipError_t launch_cast_input(DType dt, const CastArgs &a, hipStream_t s);
bool head_form_ok(int kh, int cout, bool pool, int n1);
int head_tile_rows(const HeadArgs &a);     // rows of a workgroup's tile of the result, 8 (pooled) or 16 columns wide
unsigned head_tiles(const HeadArgs &a, int32_t *tiles_h, int32_t *tiles_w);   // workgroups; 0: too many for a launch
// One image's planes are read through one descriptor of the launch, whose out-of-range offset is 2 GiB.
constexpr bool head_image_ok(int64_t c, int64_t h, int64_t w) { return c * h * w * 4 < (1ll << 31); }
hipError_t launch_head(DType dt, const HeadArgs &a, hipStream_t s);
hipError_t launch_maxpool(DType dt, const PoolArgs &a, hipStream_t s);
hipError_t launch_gavgpool(DType dt, const PoolArgs &a, hipStream_t s);
// A 3x3 max pool over 64 channels and the 1x1 stride-1 convolution 64 -> 64 or 128 that reads it, in one launch;
// c = that convolution's arguments (its x is not read), bm = pooled pixels per workgroup (64 or 128).
hipError_t launch_maxpool_conv(DType dt, const PoolArgs &a, const ConvArgs &c, int bm, hipStream_t s);
hipError_t launch_fc(DType dt, const FcArgs &a, hipStream_t s);
hipError_t launch_softmax(const SoftmaxArgs &a, hipStream_t s);
// Copies of `bytes` (a multiple of 4) into pinned host memory, 16-byte aligned like the sources; host_logits: nullptr for none.
hipError_t launch_copy_out(void *host_probs, const void *probs, void *host_logits, const void *logits, size_t bytes, hipStream_t s);
// A launch of one wave that ends once *done has reached `seq`, or after `us` microseconds.
hipError_t launch_wait_done(const unsigned *done, unsigned seq, unsigned us, hipStream_t s);
hipError_t launch_dwconv(DType dt, const DwArgs &a, hipStream_t s);
// A depthwise 3x3 convolution over c channels (no residual) and the 1x1 stride-1 convolution c -> n that reads it, in
// one launch (channel counts of dwconv_conv_ok); cv = the 1x1's arguments (its x is not read).
hipError_t launch_dwconv_conv(DType dt, const DwArgs &a, const ConvArgs &cv, hipStream_t s);
bool dwconv_conv_ok(int c, int n);
// A 1x1 convolution to 128 channels and the 3x3 pad-1 convolution to 32 over its result (its x is not read), as in a densely connected block, in one launch;
// the 1x1's result is not stored.
struct DenseTile { int th, tw; };   // rows and columns of the 3x3's result that a workgroup computes
bool dense_pick(const ConvArgs &c1, const ConvArgs &c2, DenseTile *best, double *us);   // the tile predicted to be fastest and its time; false: not for this kernel
hipError_t launch_dense_layer(DType dt, const ConvArgs &c1, const ConvArgs &c2, const DenseTile &t, hipStream_t s);
dim3 dense_grid(const ConvArgs &c1, const DenseTile &t);
// A 3x3 stride-1 pad-1 convolution 64 -> 64, the 1x1 to 256 over its result with a residual and (w3) the 1x1 back to 64 over that, dense tensors, in one launch;
// the 3x3's result is not stored.
struct TailArgs {
    const void *x, *w1, *w2, *res, *w3;
    const float *bias1, *bias2, *bias3;
    void *y, *y3;
    int32_t M, H, W, act1, act2, act3;
    FastDiv w_div, h_div;   // filled in by the launcher
    int32_t tiles;          // as these; launch_tail_walk
    const void *x2, *wd;    // launch_tail_walk: a projection from 64 channels instead of the residual, or nullptr
    const float *biasd;
};
bool tail_shape_ok(int64_t M, int32_t H, int32_t W);
int tail_bm(int64_t M);   // pixels a workgroup
hipError_t launch_tail(DType dt, const TailArgs &a, hipStream_t s);
// The same for many pixels.
constexpr int kTailWalkThreads = 512;
bool tail_walk_ok(int64_t M, int32_t H, int32_t W);
int tail_walk_bm(int64_t M);
hipError_t launch_tail_walk(DType dt, const TailArgs &a, hipStream_t s);
// A 1x1 stride-1 convolution (dense tensors) and the depthwise 3x3 pad-1 convolution over its result (its x is not read) in one launch;
// keep: the 1x1's result is stored too.
struct PwDwTile { int waves, pf, nf, rows; };   // pf x 16 pixels a wave, nf x 16 channels and `rows` rows of the depthwise result a workgroup
bool pw_dw_pick(const ConvArgs &c, const DwArgs &d, bool keep, PwDwTile *tile, double *us);   // whether it may be worth it, and its predicted time
dim3 pw_dw_grid(const ConvArgs &c, const DwArgs &d, const PwDwTile &t);
hipError_t launch_pw_dw(DType dt, const ConvArgs &c, const DwArgs &d, bool keep, const PwDwTile &t, hipStream_t s);
int dwconv_conv_bm(int c, long long M);   // output pixels per workgroup of that launch
hipError_t launch_copy_channels(const CopyArgs &a, hipStream_t s);   // 2-byte elements, C % 8 == 0
hipError_t launch_resident(DType dt, const ResidentArgs &a, hipStream_t s);   // + the epoch bump behind it
// Host-side check of one program layer against what the resident kernel assumes (shapes, sizes,
// tile counts); ws_bytes = size of the workspace its offsets must stay inside.
bool resident_layer_ok(const ResLayer &l, size_t ws_bytes);
hipError_t launch_wino_input(DType dt, const WinoArgs &a, hipStream_t s);
hipError_t launch_wino_output(DType dt, const WinoArgs &a, hipStream_t s);
// LOAD-time: canonical W[cout][cin][3][3] -> U[16][cout'][cin] = G g G^T per (cout, cin), rows in the
// conv kernel's accumulator order, computed in fp32 and rounded once to the storage type
hipError_t launch_pack_winograd(DType dt, const void *src, void *dst, int cout, int cin, hipStream_t s);
// Workgroups of a LOAD-side launch (weight packing and Winograd's transform of weights): at most four per compute unit, which is what the
// pack kernel's LDS lets run at once, each striding over its work.  ResNet-50's 51 MB behind the copy: 53 us with one per CU, 37
// with four, the same with eight.  A batch-8 EXEC beside back-to-back LOADs, six processes each: +1.2 to +3.1 % at the median with
// four, +1.5 to +3.3 % with one; it is the copy that disturbs.
constexpr unsigned kLoadGridCap = 1024;
// LOAD-time re-layout of one tensor and its bias: canonical W[cout][cin][kh][kw] -> [cout'][khp][kwp][cinp] (zero padded);
// permute = rows in the conv kernel's MFMA accumulator order (conv weights), else plain (FC);
// depthwise = W[C][1][kh][kw] -> [kh][kw][C].  The launcher fills in mode and first_chunk.
struct PackItem {
    const uint16_t *src;
    uint16_t *dst;
    const float *bias_src;
    float *bias_dst;
    int32_t cout, cin, cinp;
    uint16_t kh, kw, khp, kwp;
    uint8_t permute, depthwise, mode;
    uint32_t first_chunk;
};
constexpr int kPackItems = 60;
struct PackArgs {
    PackItem items[kPackItems];
    int32_t n;
    uint32_t chunks;
};
static_assert(sizeof(PackArgs) <= 4096, "kernel arguments");
hipError_t launch_pack_model(PackItem *items, int n, hipStream_t s);
// debug read-back: NHWC storage type (ld elements per pixel) -> fp32 NCHW
hipError_t launch_nhwc_to_nchw_f32(DType dt, const void *src, float *dst, int B, int C, int H,
                                   int W, int ld, hipStream_t s);
hipError_t launch_fill_zero(void *dst, size_t bytes, hipStream_t s);

// K-slice width the conv kernel uses for a shape under a tile: the tile's (256, 128 or 64) when Cin is a multiple of it or,
// 128 in a 1x1 stride-1 convolution, more than twice as large; else 64; 32 on the register-staged kernel.
int conv_bk(const ConvArgs &a, bool stem, ConvTile tile);
// How many of them it walks.  The direct-to-LDS kernel ends a first convolution's walk at the last pair of real filter rows.
int conv_slices(const ConvArgs &a, bool stem, ConvTile tile);
// Bytes at the start of the workspace reserved for split-K arrival counters (one int per tile).
constexpr size_t kCounterBytes = 256 * 1024;
// Grid and block of a conv launch (pure function of tile and shape).
void conv_grid(ConvTile tile, const ConvArgs &a, dim3 *grid, int *block);

}  // namespace cw
