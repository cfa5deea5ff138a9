// The head of a network in one launch: input cast, first convolution and, where a 3x3 max pool follows, the pool and the
// 1x1 convolution behind that.
// As launches of their own these are bound by launches and round trips, not by their work: at batch 16 the cast writes and
// the convolution reads a padded copy of the images, the convolution writes and the pool reads 25 MB, and at
// batch 1 each of the three takes 2-3.5 us from its first workgroup to its last store for well under a microsecond of work.
// Here a workgroup computes a tile of the result from the image: it loads the tile's patch of the fp32 planes, rounds it
// once and puts it into LDS as 4-channel pixels (out of the image: zeros), and its four waves run the convolution on the
// matrix cores straight out of that patch, two taps x 4 channels being 16 consecutive bytes of it (the stride is 2).  With a pool the rounded
// convolution tile goes to LDS, -inf outside the convolution's map, and is pooled from there; a pooled tile of 7 x 8 needs
// 15 x 17 = 255 convolution pixels, eight MFMA tiles of 32, of which an eighth is computed twice by neighbours.  K runs in the order of
// the launches of their own and every tensor is rounded as when it is stored: same bits.  (A filter row is padded with weights of
// zero, to 8 taps of a 7x7 and 4 of a 3x3, which has 8 in a launch of its own: an infinite or NaN pixel also makes NaN of the
// outputs whose row ends that far before it.)
// What bounds it: the chain image load, matrix cores, pool, at batch 16 3.5 times per CU side by side (first workgroup's
// start to last store, 224x224: ResNet-50 batch 16 12.6 us, batch 1 4.1, ResNet-18 batch 8 7.7, MobileNet batch 16 5.5), hence the 40 KB of LDS:
// with 56 KB, two workgroups a CU, and the weights loaded as fragments, 32 rows to an instruction, batch 16 took 21.1.  Whole
// EXECs against three launches: ResNet-50 batch 16 440.6 -> 422.0 us, batch 1 219.4 -> 212.0, ResNet-18 batch 8 163.6 -> 147.2, DenseNet
// batch 6 238.2 -> 224.1, Inception 127x127 batch 5 104.5 -> 100.2.
#include "conv_common.h"

namespace cw {

template <typename T>
struct MaxOf8 {   // eight values of the storage type, element-wise maximum that ignores NaN like fmaxf
    float m[8];
    __device__ __forceinline__ void start() {
#pragma unroll
        for (int e = 0; e < 8; ++e) m[e] = -INFINITY;
    }
    __device__ __forceinline__ void take(const u32x4 &raw) {
        const T *v = reinterpret_cast<const T *>(&raw);
#pragma unroll
        for (int e = 0; e < 8; ++e) m[e] = fmaxf(m[e], (float)v[e]);
    }
    __device__ __forceinline__ u32x4 get() const {
        T out[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e] = (T)m[e];  // exact: the max is one of the inputs
        return *reinterpret_cast<const u32x4 *>(out);
    }
};
template <>
struct MaxOf8<f16> {
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    h8 m;
    __device__ __forceinline__ void start() { m = (h8)(_Float16)-INFINITY; }
    __device__ __forceinline__ void take(const u32x4 &raw) { m = __builtin_elementwise_max(m, *reinterpret_cast<const h8 *>(&raw)); }
    __device__ __forceinline__ u32x4 get() const { return *reinterpret_cast<const u32x4 *>(&m); }
};

// Channels 16q + 8*(lane/32) .. +7 of an accumulator: + bias, activation, one rounding.
template <typename T>
static __device__ __forceinline__ u32x4 head_out(const f32x16 &acc, int q, const u32x4 (&bias)[2], int act) {
    float v[8];
    T out[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = acc[8 * q + k] + __uint_as_float(bias[k / 4][k % 4]);
    if (act == ACT_HSWISH) {
#pragma unroll
        for (int k = 0; k < 8; ++k) out[k] = (T)(v[k] * fminf(fmaxf(v[k] + 3.f, 0.f), 6.f) * (1.f / 6.f));
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) out[k] = (T)(act ? fmaxf(v[k], 0.f) : v[k]);
    }
    return *reinterpret_cast<const u32x4 *>(out);
}

// Elements from one pixel to the next of the LDS tile that is pooled: 144 bytes.  A store has 16 consecutive pixels at one
// 16-byte chunk in a clock and, 36 words apart, they cover the 64 banks; a pool read has two pixels 8 apart at
// all 8 chunks, which are half of the banks apart.  Every address is a base plus a constant.
constexpr int kPoolPitch = 72;

// KH x KH filter, CO output channels.  POOL: a tile is TH x 8 pooled pixels, and N1 > 0: with the 1x1 convolution 64 -> N1
// over them; else TH x 16 pixels of the convolution.
template <typename T, int KH, int CO, bool POOL, int N1, int TH>
__global__ __launch_bounds__(256, 4) void head_kernel(const HeadArgs a) {
    constexpr int TW = POOL ? 8 : 16;
    constexpr int CR = POOL ? 2 * TH + 1 : TH, CC = POOL ? 2 * TW + 1 : TW, PIX = CR * CC;   // the tile of the convolution
    constexpr int TAPS = KH > 4 ? 8 : 4, UPR = TAPS / 4, STEPS = KH * UPR;                   // 16-k steps: four taps of a filter row
    constexpr int PR = 2 * (CR - 1) + KH, PC = 2 * (CC - 1) + TAPS;                          // the patch of the image
    static_assert(PC % 2 == 0 && KH <= TAPS, "16-byte aligned pairs of taps");
    constexpr int WC = CO / 32, WP = 4 / WC, NPW = ((PIX + 31) / 32 + WP - 1) / WP;          // waves over channels, over pixels; tiles of a wave
    static_assert(!POOL || CO == 64, "the pool's LDS layout");
    static_assert(N1 == 0 || (POOL && TH * TW <= 64), "the 1x1 takes one 64-pixel tile");
    constexpr int PER = (PR * PC + 255) / 256;
    typedef typename Mfma<T>::v8 v8;
    // One LDS region for the patch and the weights, then the convolution's tile, then the pooled tile: 40 KB, four workgroups a CU.
    // A filter row of a channel is four 16-byte chunks; an odd number of chunks from channel to channel keeps a fragment's 16 rows apart.
    constexpr int W_CHUNKS = KH * 4, W_PITCH = (W_CHUNKS + 1) * 8, W_PER = (CO * W_CHUNKS + 255) / 256;
    constexpr int IN_ELEMS = PR * PC * 4 + CO * W_PITCH, C_ELEMS = POOL ? NPW * WP * 32 * kPoolPitch : 0, P_ELEMS = N1 ? 64 * 64 : 0;
    constexpr int LDS_ELEMS = IN_ELEMS > C_ELEMS ? (IN_ELEMS > P_ELEMS ? IN_ELEMS : P_ELEMS) : (C_ELEMS > P_ELEMS ? C_ELEMS : P_ELEMS);
    static_assert(PR * PC * 4 % 8 == 0 && LDS_ELEMS * 2 <= 40960, "four workgroups a CU");
    __shared__ __attribute__((aligned(16))) T lds[LDS_ELEMS];
    T *const sW = lds + PR * PC * 4;
    T *const sIn = lds, *const sC = lds, *const sP = lds;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lrow = lane & 31, lhalf = lane >> 5;
    const int wc = wave % WC, wp = wave / WC;
    for (int j = blockIdx.x * 256 + tid; j < a.n_zero; j += gridDim.x * 256) a.zero[j] = 0;

    const unsigned tile = xcd_tile_id(blockIdx.x, gridDim.x);
    const unsigned per_image = (unsigned)a.tiles_h * a.tiles_w;
    const int n = (int)(tile / per_image);
    const int rest = (int)(tile - n * per_image);
    const int p0 = rest / a.tiles_w * TH, q0 = rest % a.tiles_w * TW;
    const int cr0 = POOL ? 2 * p0 - 1 : p0, cc0 = POOL ? 2 * q0 - 1 : q0;                    // the tile's first pixel in the convolution's map

    // ---- the patch, the weights and the biases: every load requested before the first is used, none behind a branch (a value
    // out of the image is a load out of range, which returns zero)
    const int hw = a.H * a.W, ih0 = 2 * cr0 - a.pad, iw0 = 2 * cc0 - a.pad;
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.x + (size_t)n * a.C * hw, (unsigned)(a.C * hw) * 4u);
    unsigned px[PER][4];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = tid + j * 256, row = i / PC, ih = ih0 + row, iw = iw0 + (i - row * PC);
        const bool ok = i < PR * PC && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
        const unsigned o = (unsigned)(ih * a.W + iw) * 4u;
#pragma unroll
        for (int c = 0; c < 4; ++c) px[j][c] = __builtin_amdgcn_raw_buffer_load_b32(rx, ok && c < a.C ? o + (unsigned)(c * hw) * 4u : kOob, 0, 0);
    }
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(a.w, CO * 256u * 2u), rb = make_rsrc(a.bias, CO * 4u);
    u32x4 wr[W_PER], bias[2][2];
#pragma unroll
    for (int j = 0; j < W_PER; ++j) {   // packed [CO][8][8][4]: the first KH rows of every channel, in memory order
        const unsigned i = tid + j * 256u, c = i / W_CHUNKS;
        wr[j] = __builtin_amdgcn_raw_buffer_load_b128(rw, i < CO * W_CHUNKS ? c * 512u + (i - c * W_CHUNKS) * 16u : kOob, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int h = 0; h < 2; ++h) bias[q][h] = __builtin_amdgcn_raw_buffer_load_b128(rb, (unsigned)(wc * 32 + 16 * q + 8 * lhalf + 4 * h) * 4u, 0, 0);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = tid + j * 256;
        T v[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = (T)__uint_as_float(px[j][c]);
        if (i < PR * PC) *reinterpret_cast<uint2 *>(sIn + i * 4) = *reinterpret_cast<const uint2 *>(v);
    }
#pragma unroll
    for (int j = 0; j < W_PER; ++j) {
        const int i = tid + j * 256, c = i / W_CHUNKS;
        if (i < CO * W_CHUNKS) *reinterpret_cast<u32x4 *>(sW + c * W_PITCH + (i - c * W_CHUNKS) * 8) = wr[j];
    }
    __syncthreads();

    // ---- the convolution
    f32x16 acc[NPW];
    int at[NPW];
#pragma unroll
    for (int t = 0; t < NPW; ++t) {
        const int p = min((wp * NPW + t) * 32 + lrow, PIX - 1), cr = p / CC, cc = p - cr * CC;
        at[t] = (2 * cr * PC + 2 * cc + 2 * lhalf) * 4;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
    }
    const T *wrow = sW + (wc * 32 + lrow) * W_PITCH + 8 * lhalf;
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        const v8 wf = *reinterpret_cast<const v8 *>(wrow + s / UPR * 32 + s % UPR * 16);
#pragma unroll
        for (int t = 0; t < NPW; ++t) acc[t] = Mfma<T>::mma(wf, *reinterpret_cast<const v8 *>(sIn + at[t] + (s / UPR * PC + s % UPR * 4) * 4), acc[t]);
    }

    if constexpr (!POOL) {
#pragma unroll
        for (int t = 0; t < NPW; ++t) {
            const int p = (wp * NPW + t) * 32 + lrow, cr = p / CC, cc = p - cr * CC;
            if (p >= PIX || cr0 + cr >= a.Ho || cc0 + cc >= a.Wo) continue;
            T *y = static_cast<T *>(a.y) + ((size_t)(n * a.Ho + cr0 + cr) * a.Wo + cc0 + cc) * a.ldy + wc * 32 + 8 * lhalf;
#pragma unroll
            for (int q = 0; q < 2; ++q) *reinterpret_cast<u32x4 *>(y + 16 * q) = head_out<T>(acc[t], q, bias[q], a.act);
        }
    } else {
        const bool inside = cr0 >= 0 && cc0 >= 0 && cr0 + CR <= a.Ho && cc0 + CC <= a.Wo;   // uniform: the whole tile is in the map
        __syncthreads();   // every wave is done with the patch
#pragma unroll
        for (int t = 0; t < NPW; ++t) {
            const int p = (wp * NPW + t) * 32 + lrow;
#pragma unroll
            for (int q = 0; q < 2; ++q) *reinterpret_cast<u32x4 *>(sC + p * kPoolPitch + wc * 32 + 16 * q + 8 * lhalf) = head_out<T>(acc[t], q, bias[q], a.act);
            if (!inside) {
                const int cr = p / CC, cc = p - cr * CC;
                T lowest[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) lowest[k] = (T)-INFINITY;
                if ((unsigned)(cr0 + cr) >= (unsigned)a.Ho || (unsigned)(cc0 + cc) >= (unsigned)a.Wo) {
#pragma unroll
                    for (int q = 0; q < 2; ++q) *reinterpret_cast<u32x4 *>(sC + p * kPoolPitch + wc * 32 + 16 * q + 8 * lhalf) = *reinterpret_cast<const u32x4 *>(lowest);
                }
            }
        }
        constexpr int TN = N1 ? N1 / 64 : 1;
        const int wm = (wave >> 1) * 32, wn = (wave & 1) * (N1 / 2);   // the 1x1: waves 2 x 2 over pixels x channels
        u32x4 w1[TN][4];
        if constexpr (N1 > 0) {   // its weights arrive behind the pool
            const __amdgpu_buffer_rsrc_t rw1 = make_rsrc(a.w1, N1 * 64u * 2u);
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) w1[j][kk] = __builtin_amdgcn_raw_buffer_load_b128(rw1, (unsigned)(wn + j * 32 + lrow) * 128u + 32u * kk + 16u * lhalf, 0, 0);
        }
        __syncthreads();
        // Piece i of the pooled tile: chunk i % 8 of pixel column i/8 % 2 * 4 + i/16 % 4, row i / 64.
        constexpr int ITEMS = TH * TW * 8, IPER = (ITEMS + 255) / 256;
        static_assert(TW == 8, "the order of the pieces");
        u32x4 out[IPER];
#pragma unroll
        for (int j = 0; j < IPER; ++j) {
            const int i = tid + j * 256, c8 = i & 7, pr = i >> 6, pc = ((i >> 3) & 1) * 4 + ((i >> 4) & 3);
            if (i >= ITEMS) continue;
            const T *src = sC + (2 * pr * CC + 2 * pc) * kPoolPitch + c8 * 8;
            MaxOf8<T> m;
            m.start();
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int s = 0; s < 3; ++s) m.take(*reinterpret_cast<const u32x4 *>(src + (r * CC + s) * kPoolPitch));
            out[j] = m.get();
            if (p0 + pr < a.Po && q0 + pc < a.Qo)
                *reinterpret_cast<u32x4 *>(static_cast<T *>(a.y) + ((size_t)(n * a.Po + p0 + pr) * a.Qo + q0 + pc) * a.ldy + c8 * 8) = out[j];
        }
        if constexpr (N1 > 0) {
            // ---- the 1x1 over the pooled tile (rows TH*TW.. hold what was there; never stored)
            __syncthreads();
#pragma unroll
            for (int j = 0; j < IPER; ++j) {
                const int i = tid + j * 256, c8 = i & 7, pr = i >> 6, pc = ((i >> 3) & 1) * 4 + ((i >> 4) & 3);
                if (i < ITEMS) *reinterpret_cast<u32x4 *>(sP + swz<64>(pr * TW + pc, c8)) = out[j];
            }
            u32x4 bias1[TN][2][2];
            const __amdgpu_buffer_rsrc_t rb1 = make_rsrc(a.bias1, N1 * 4u);
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int h = 0; h < 2; ++h) bias1[j][q][h] = __builtin_amdgcn_raw_buffer_load_b128(rb1, (unsigned)(wn + j * 32 + 16 * q + 8 * lhalf + 4 * h) * 4u, 0, 0);
            __syncthreads();
            f32x16 acc1[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc1[j][e] = 0.f;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const v8 fx = *reinterpret_cast<const v8 *>(sP + swz<64>(wm + lrow, kk * 2 + lhalf));
#pragma unroll
                for (int j = 0; j < TN; ++j) acc1[j] = Mfma<T>::mma(*reinterpret_cast<const v8 *>(&w1[j][kk]), fx, acc1[j]);
            }
            const int i = wm + lrow, p = p0 + i / TW, q0i = q0 + i % TW;
            if (i < TH * TW && p < a.Po && q0i < a.Qo) {
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        *reinterpret_cast<u32x4 *>(static_cast<T *>(a.y1) + ((size_t)(n * a.Po + p) * a.Qo + q0i) * a.ldy1 + wn + j * 32 + 16 * q + 8 * lhalf) =
                            head_out<T>(acc1[j], q, bias1[j][q], a.act1);
            }
        }
    }
}

bool head_form_ok(int kh, int cout, bool pool, int n1) {
    return pool ? kh == 7 && cout == 64 && (n1 == 0 || n1 == 64 || n1 == 128) : kh == 3 && cout == 32 && n1 == 0;
}

int head_tile_rows(const HeadArgs &a) {
    return !a.pool ? 8 : a.n1 > 0 || (long long)a.B * ((a.Po + 6) / 7) * ((a.Qo + 7) / 8) >= kHeadTallFrom ? 7 : 3;
}

unsigned head_tiles(const HeadArgs &a, int32_t *tiles_h, int32_t *tiles_w) {
    const int th = head_tile_rows(a);
    *tiles_h = ((a.pool ? a.Po : a.Ho) + th - 1) / th;
    *tiles_w = a.pool ? (a.Qo + 7) / 8 : (a.Wo + 15) / 16;
    const long long tiles = (long long)a.B * *tiles_h * *tiles_w;
    return tiles < (1ll << 31) ? (unsigned)tiles : 0;
}

hipError_t launch_head(DType dt, const HeadArgs &a_in, hipStream_t s) {
    HeadArgs a = a_in;
    if (!head_form_ok(a.kh, a.cout, a.pool, a.n1) || a.B < 1 || a.C < 1 || a.C > 4 || a.H < 1 || a.W < 1 || a.pad < 0 || !a.x || !a.w || !a.bias || !a.y)
        return hipErrorInvalidValue;
    if (a.H + 2 * a.pad < a.kh || a.W + 2 * a.pad < a.kh || a.Ho != (a.H + 2 * a.pad - a.kh) / 2 + 1 || a.Wo != (a.W + 2 * a.pad - a.kh) / 2 + 1) return hipErrorInvalidValue;
    if (a.pool && (a.Po != (a.Ho - 1) / 2 + 1 || a.Qo != (a.Wo - 1) / 2 + 1)) return hipErrorInvalidValue;
    if (a.ldy < a.cout || (a.n1 > 0 && (!a.w1 || !a.bias1 || !a.y1 || a.ldy1 < a.n1)) || a.n_zero < 0 || (a.n_zero > 0 && !a.zero)) return hipErrorInvalidValue;
    if (!head_image_ok(a.C, a.H, a.W) || (long long)a.B * a.Ho * a.Wo >= (1ll << 31)) return hipErrorInvalidValue;
    const int th = head_tile_rows(a);
    const unsigned tiles = head_tiles(a, &a.tiles_h, &a.tiles_w);
    if (tiles == 0) return hipErrorInvalidValue;
#define CW_HEAD(KH_, CO_, POOL_, N1_, TH_)                                                                              \
    do {                                                                                                                \
        if (dt == DT_F16) head_kernel<f16, KH_, CO_, POOL_, N1_, TH_><<<dim3(tiles), 256, 0, s>>>(a);         \
        else head_kernel<bf16, KH_, CO_, POOL_, N1_, TH_><<<dim3(tiles), 256, 0, s>>>(a);                     \
    } while (0)
    if (!a.pool) CW_HEAD(3, 32, false, 0, 8);
    else if (a.n1 == 64) CW_HEAD(7, 64, true, 64, 7);
    else if (a.n1 == 128) CW_HEAD(7, 64, true, 128, 7);
    else if (th == 7) CW_HEAD(7, 64, true, 0, 7);
    else CW_HEAD(7, 64, true, 0, 3);
#undef CW_HEAD
    return hipGetLastError();
}

}  // namespace cw
