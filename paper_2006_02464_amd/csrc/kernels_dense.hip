// A densely connected layer in one launch: a 1x1 convolution to 128 channels and the 3x3 convolution to 32 that reads it.
// As two launches the tensor between them, 128 channels for the 32 that stay, goes to memory and back, and at DenseNet's sizes each launch is its fixed
// time and one wait for operands (28x28, batch 6: 2.8 to 4.3 us and 4.3 for 0.3 and 0.2 us of matrix instructions).  Here a workgroup computes a tile of the
// result: the 1x1 over the tile and a border of one pixel, rounded as when it is stored, into LDS, and the 3x3 from there.
// What bounds it: what a CU has to fetch, 256 bytes x K of the 1x1's weights, 72 KB of the 3x3's and the pixels, then
// two contractions one behind the other with one wave a SIMD.  By counters at batch 6 a wave lives 12.0k to 16.9k clocks at 28x28 and waits 35 to 40 % of them; a stage of 64
// channels of K is 800 clocks for 26 KB (33 bytes a clock of the 58 to 64 that the load path sustains), 1800 at 56x56 with twice the pixels a wave.  What made it faster than the two launches:
// - All operands go to LDS by direct loads whose neighbouring lanes read neighbouring bytes.  A load into the registers of an
//   MFMA operand has its 16 lowest lanes in 16 rows and takes 41 clocks a KB for 14 (28x28, K 256, batch 6 6.4 -> 5.7 us; K 480 8.9 -> 7.0).
// - A wave reads its own quarter of the 3x3's weights, 32 of the 128 channels, into registers once; the four partial sums meet in LDS.
// - Two by two waves over pixels x middle channels: each operand is read from LDS twice, not four times.
// - The border outside the image is stored as zeros, so the 3x3's reads are one base and constants.
// Graph replay, one launch against the two: batch 6, 56x56, K 64 / 160 / 224 7.0 / 8.2 / 8.9 us for 11.4 / 11.5 / 12.4; 28x28, K 128 / 256 / 352 / 480
// 5.0 / 5.7 / 6.4 / 7.0 for 7.1 / 7.5 / 8.2 / 8.5; batch 1 4.7 / 5.4 / 6.1 / 6.7 for 5.7 / 5.9 / 7.2 / 7.6.

#include "conv_dlds_body.h"

namespace cw {

constexpr int kMid = 128, kOut = 32, kTaps = 9;   // channels between the two and behind them

struct alignas(64) DenseRest {
    const float *bias1, *bias2;
    void *y;
    int32_t B, ldy, act1, act2;
    FastDiv halo_div, tw_div;
};

constexpr unsigned kMidPitch = kMid * 2 + 16;   // bytes of a pixel of the middle tensor: 16 consecutive ones start on different banks

// What a workgroup loads: K in stages of 64, weights of the 1x1 [128][64] and pixels [64 PF][64], into a ring of slots, and the 3x3's
// weights in 72 pieces [tap][half of the rows][wave] of 16 rows x 32 channels, `fresh` of a wave's 18 into space of their own and the rest into a slot that is
// done with.  A wave issues, in this order: the ring's first fill, its fresh pieces, and behind the barrier of every stage from the second on what goes
// into the slot that this barrier frees: the stage that comes R - 1 later, or once, when there is none, the rest of the pieces.
template <int PF, int NS>
struct DenseLoads {
    static constexpr int L = 4 + 2 * PF, SLOT = 16384 + 8192 * PF, MOST = PF == 1 ? 4 : 3, R = NS < MOST ? NS : MOST;
    static constexpr int PIECES = 2 * kTaps, FRESH = R < MOST ? PIECES : 15, LATE = PIECES - FRESH;
    static constexpr int late_at = NS - R + 1;   // the stage behind whose barrier the rest of the pieces is issued
    static_assert(LATE == 0 || (late_at >= 1 && late_at < NS && LATE * 4096 <= SLOT), "");
    // Loads issued before the barrier of stage s.
    static constexpr int issued(int s) {
        int n = R * L + FRESH;
        for (int q = 1; q < s; ++q) n += q - 1 + R < NS ? L : q == late_at ? LATE : 0;
        return n;
    }
    // Loads issued up to the last one of stage s.
    static constexpr int upto(int s) { return s < R ? (s + 1) * L : issued(s - R + 1) + L; }
    static constexpr int younger(int s) { return issued(s) - upto(s); }
    static constexpr unsigned ring = R * SLOT, fresh_bytes = FRESH * 4096u;
};

static int dense_pf(const DenseTile &t) { return ((t.th + 2) * (t.tw + 2) + 63) / 64; }
// LDS: ring, later the middle tensor and behind it the waves' sums | fresh pieces
static unsigned dense_sums(const DenseTile &t) { return (unsigned)(t.th + 2) * (t.tw + 2) * kMidPitch; }
static unsigned dense_front(const DenseTile &t, unsigned ring) { return std::max(ring, dense_sums(t) + (unsigned)(t.th * t.tw + 15) / 16 * 8192u); }

// Until stage s has landed, for every wave.
template <int PF, int NS, int S = 0>
static __device__ __forceinline__ void dense_wait(int s) {
    if constexpr (S < NS) {
        if (s == S) wait_lds_loads_and_barrier<DenseLoads<PF, NS>::younger(S) + (S == 0 ? 6 : 0)>();   // 6: the biases, behind the first stage
        else dense_wait<PF, NS, S + 1>(s);
    }
}

template <typename T, int PF, int NS>
__global__ __launch_bounds__(256) void dense_layer_kernel(const void *x, const void *w1, const void *w2, int K_ldx, int H_W, int TH_TW, int tiles_w, int tiles, unsigned o_fresh, const DenseRest a) {
    typedef MfmaTile<T, 16> MF;
    typedef typename Mfma<T>::v8 v8;
    typedef DenseLoads<PF, NS> D;
    constexpr int XF = 2 * PF, NF = 4;   // of a wave, which has half of the pixels and half of the middle channels: 16 each
    const int K = K_ldx & 0xffff, H = H_W & 0xffff, W = (unsigned)H_W >> 16, TH = TH_TW & 0xffff, TW = (unsigned)TH_TW >> 16;
    const unsigned ldx2 = ((unsigned)K_ldx >> 16) * 2u;
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)cw_dyn_lds;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 15, lhalf = lane >> 4;
    const int tile = xcd_tile_id(blockIdx.x, gridDim.x);
    const int n = tile_div(tile, tiles), tt = tile - n * tiles, ti = tile_div(tt, tiles_w);
    const int i0 = ti * TH, j0 = (tt - ti * tiles_w) * TW;
    const int HW = TW + 2, HP = (TH + 2) * HW;
    const u32x4 dw = make_desc(w1, (unsigned)kMid * K * 2u), dx = make_desc(x, ((unsigned)a.B * H * W - 1u) * ldx2 + (unsigned)K * 2u), dw2 = make_desc(w2, kOut * kTaps * kMid * 2u);
    const unsigned row8 = lane >> 3, c8 = lane & 7;   // of a piece of 8 rows x 128 bytes; chunk c of row r lies at c ^ (r / 2) % 8
    unsigned w_off = row8 * (unsigned)K * 2u + ((c8 ^ ((((wave & 1) * 8 + row8) >> 1) & 7)) << 4), x_off[XF];   // a wave's pieces of the weights: all odd or all even
    const bool odd = K & 32;   // the last stage has 32 of its 64: chunks 4 to 7 are zeros
    auto load_w = [&](int s) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int piece = wave + q * 4;
            const bool none = s == NS - 1 && odd && ((c8 ^ (((wave & 1) * 8 + row8) >> 1)) & 4);
            load_to_lds(dw, none ? kOob : w_off, (unsigned)piece * 8u * K * 2u + (unsigned)s * 128u, lds_base + (unsigned)(s % D::R) * D::SLOT + (unsigned)piece * 1024u);
        }
    };
    auto load_x = [&](int s) {
#pragma unroll
        for (int p = 0; p < XF; ++p) {
            const bool none = s == NS - 1 && odd && ((c8 ^ ((((wave + p * 4) * 8 + row8) >> 1))) & 4);
            load_to_lds(dx, none ? kOob : x_off[p], (unsigned)s * 128u, lds_base + (unsigned)(s % D::R) * D::SLOT + 16384u + (unsigned)(wave + p * 4) * 1024u);
        }
    };
    load_w(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < XF; ++p) {
        const int h = (wave + p * 4) * 8 + (int)row8;
        const int hr = (int)fast_div((unsigned)h, a.halo_div), ih = i0 - 1 + hr, iw = j0 - 1 + h - hr * HW;
        x_off[p] = h < HP && (unsigned)ih < (unsigned)H && (unsigned)iw < (unsigned)W ? ((unsigned)(n * H + ih) * W + iw) * ldx2 + ((c8 ^ ((h >> 1) & 7)) << 4) : kOob;
    }
    load_x(0);
    const unsigned nl = 8 * (lhalf & 1) + 4 * (lhalf >> 1);   // the channel of a lane's first row (packed weights)
    const int wp = wave >> 1, wn = wave & 1;
    const __amdgpu_buffer_rsrc_t rb1 = make_rsrc(a.bias1, kMid * 4u), rb2 = make_rsrc(a.bias2, kOut * 4u);
    u32x4 bv[NF];
#pragma unroll
    for (int j = 0; j < NF; ++j) bv[j] = __builtin_amdgcn_raw_buffer_load_b128(rb1, (nl + 16 * j) * 4u, (unsigned)wn * 256u, 0);
    const u32x4 b2[2] = {__builtin_amdgcn_raw_buffer_load_b128(rb2, nl * 4u, 0, 0), __builtin_amdgcn_raw_buffer_load_b128(rb2, (nl + 16) * 4u, 0, 0)};
    __builtin_amdgcn_sched_barrier(0);
    const unsigned p_row = lane >> 2, p_off = p_row * (kTaps * kMid * 2u) + (((lane & 3) ^ ((p_row >> 2) & 3)) << 4);
    auto load_piece = [&](int i) {   // tap i / 2, rows 16 (i % 2) on, this wave's channels
        const unsigned at = i < D::FRESH ? o_fresh + (unsigned)i * 4096u : (unsigned)((D::late_at - 1) % D::R) * D::SLOT + (unsigned)(i - D::FRESH) * 4096u;
        load_to_lds(dw2, p_off, (unsigned)(i & 1) * 16u * (kTaps * kMid * 2u) + (unsigned)(i >> 1) * (kMid * 2u) + (unsigned)wave * 64u, lds_base + at + (unsigned)wave * 1024u);
    };
#pragma unroll
    for (int s = 1; s < D::R; ++s) { load_w(s); load_x(s); }
#pragma unroll
    for (int i = 0; i < D::FRESH; ++i) load_piece(i);
    typename MF::acc acc[XF][NF];
#pragma unroll
    for (int f = 0; f < XF; ++f)
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[f][j] = typename MF::acc{0.f, 0.f, 0.f, 0.f};
    const unsigned key = (lrow >> 1) & 7, rd = (unsigned)lrow * 128u;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        dense_wait<PF, NS>(s);
        if (s > 0 && s - 1 + D::R < NS) { load_w(s - 1 + D::R); load_x(s - 1 + D::R); }
        if (D::LATE && s == D::late_at)
#pragma unroll
            for (int i = D::FRESH; i < D::PIECES; ++i) load_piece(i);
        const unsigned char *at = cw_dyn_lds + (unsigned)(s % D::R) * D::SLOT + rd;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const unsigned c = ((unsigned)(t * 4 + lhalf) ^ key) << 4;
            v8 fw[NF], fx[XF];
#pragma unroll
            for (int j = 0; j < NF; ++j) fw[j] = *reinterpret_cast<const v8 *>(at + (unsigned)(wn * NF + j) * 2048u + c);
#pragma unroll
            for (int f = 0; f < XF; ++f) fx[f] = *reinterpret_cast<const v8 *>(at + 16384u + (unsigned)(wp * XF + f) * 2048u + c);
#pragma unroll
            for (int f = 0; f < XF; ++f)
#pragma unroll
                for (int j = 0; j < NF; ++j) acc[f][j] = MF::mma(fw[j], fx[f], acc[f][j]);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");   // this wave's pieces, which nobody else reads
    u32x4 fw2[kTaps][2];
    const unsigned p_rd = (unsigned)wave * 1024u + (unsigned)lrow * 64u + ((lhalf ^ ((lrow >> 2) & 3)) << 4);
#pragma unroll
    for (int i = 0; i < D::PIECES; ++i) {
        const unsigned at = i < D::FRESH ? o_fresh + (unsigned)i * 4096u : (unsigned)((D::late_at - 1) % D::R) * D::SLOT + (unsigned)(i - D::FRESH) * 4096u;
        fw2[i >> 1][i & 1] = *reinterpret_cast<const u32x4 *>(cw_dyn_lds + at + p_rd);
    }
    wait_lds_and_barrier();   // the ring is done with
    auto middle = [&](auto act) {
#pragma unroll
        for (int f = 0; f < XF; ++f) {
            const int h = (wp * XF + f) * 16 + lrow;
            const int hr = (int)fast_div((unsigned)h, a.halo_div), ih = i0 - 1 + hr, iw = j0 - 1 + h - hr * HW;
            const bool in = (unsigned)ih < (unsigned)H && (unsigned)iw < (unsigned)W;   // the 3x3 has zeros outside the image
#pragma unroll
            for (int j = 0; j < NF; ++j) {
                T o[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (T)act(acc[f][j][e] + __uint_as_float(bv[j][e]));
                const u32x2 v = *reinterpret_cast<const u32x2 *>(o);
                if (h < HP) *reinterpret_cast<u32x2 *>(cw_dyn_lds + (unsigned)h * kMidPitch + (wn * 64 + nl) * 2u + j * 32u) = in ? v : u32x2{0u, 0u};
            }
        }
    };
    if (a.act1 == ACT_RELU) middle([](float v) { return fmaxf(v, 0.f); });
    else if (a.act1 == ACT_HSWISH) middle([](float v) { return v * fminf(fmaxf(v + 3.f, 0.f), 6.f) * (1.f / 6.f); });
    else middle([](float v) { return v; });
    const int OUT = TH * TW, frags = (OUT + 15) >> 4;
    const unsigned o_sums = (unsigned)HP * kMidPitch;
    const unsigned rowb = (unsigned)HW * kMidPitch;
    wait_lds_and_barrier();
    v8 pa[2][kTaps], pb[2][kTaps];
    auto read = [&](v8 (&p)[2][kTaps], int g) {
        unsigned at[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int o = min((g + u) * 16 + lrow, OUT - 1);
            const int orow = (int)fast_div((unsigned)o, a.tw_div);
            at[u] = (unsigned)(orow * HW + o - orow * TW) * kMidPitch + (unsigned)wave * 64u + lhalf * 16u;
        }
#pragma unroll
        for (int t = 0; t < kTaps; ++t)
#pragma unroll
            for (int u = 0; u < 2; ++u) p[u][t] = *reinterpret_cast<const v8 *>(cw_dyn_lds + at[u] + (unsigned)(t / 3) * rowb + (t % 3) * kMidPitch);
    };
    auto product = [&](const v8 (&p)[2][kTaps], int g) {
        typename MF::acc s[2][2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int j = 0; j < 2; ++j) s[u][j] = typename MF::acc{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < kTaps; ++t)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int j = 0; j < 2; ++j) s[u][j] = MF::mma(__builtin_bit_cast(v8, fw2[t][j]), p[u][t], s[u][j]);
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (g + u < frags)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    *reinterpret_cast<typename MF::acc *>(cw_dyn_lds + o_sums + (unsigned)(((g + u) * 4 + wave) * 2 + j) * 1024u + lane * 16u) = s[u][j];
    };
    read(pa, 0);
    for (int g = 0; g < frags; g += 4) {
        if (g + 2 < frags) read(pb, g + 2);
        product(pa, g);
        if (g + 2 < frags) {
            if (g + 4 < frags) read(pa, g + 4);
            product(pb, g + 2);
        }
    }
    wait_lds_and_barrier();
    for (int g = wave; g < frags; g += 4) {
        const int o = g * 16 + lrow, orow = (int)fast_div((unsigned)o, a.tw_div), i = i0 + orow, j = j0 + o - orow * TW;
        float v[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            typename MF::acc p[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) p[w] = *reinterpret_cast<const typename MF::acc *>(cw_dyn_lds + o_sums + (unsigned)((g * 4 + w) * 2 + h) * 1024u + lane * 16u);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[h][e] = (p[0][e] + p[1][e]) + (p[2][e] + p[3][e]) + __uint_as_float(b2[h][e]);
        }
        if (o < OUT && i < H && j < W) {
            char *y = static_cast<char *>(a.y) + ((size_t)((unsigned)(n * H + i) * W + j) * a.ldy + nl) * 2;
            *reinterpret_cast<u32x2 *>(y) = activate<T>(v[0], a.act2);
            *reinterpret_cast<u32x2 *>(y + 32) = activate<T>(v[1], a.act2);
        }
    }
}

// Shapes that the kernel's indexing relies on.
static bool dense_shape_ok(const ConvArgs &c1, const ConvArgs &c2) {
    if (c1.kh != 1 || c1.kw != 1 || c1.stride != 1 || c1.pad != 0 || c1.Cout != kMid || c1.K != c1.Cin || c1.K % 32 != 0 || c1.K < 32 || c1.K > 512) return false;
    if (c2.kh != 3 || c2.kw != 3 || c2.stride != 1 || conv_pad_h(c2) != 1 || conv_pad_w(c2) != 1 || c2.Cin != kMid || c2.Cout != kOut || c2.K != kTaps * kMid) return false;
    if (c1.B < 1 || c1.H < 1 || c1.W < 1 || c1.H > 32767 || c1.W > 32767 || c1.Ho != c1.H || c1.Wo != c1.W || c2.H != c1.H || c2.W != c1.W || c2.Ho != c1.H || c2.Wo != c1.W || c2.B != c1.B) return false;
    if (conv_ldx(c1) < c1.K || conv_ldx(c1) > 65535 || conv_ldx(c1) % 8 != 0 || conv_ldy(c2) < kOut || conv_ldy(c2) % 8 != 0) return false;
    return (int64_t)c1.B * c1.H * c1.W * std::max(conv_ldx(c1), conv_ldy(c2)) < (1ll << 30) && (int64_t)c1.B * c1.H * c1.W < (1 << 21);
}

static int64_t dense_wgs(const ConvArgs &c, const DenseTile &t) { return (int64_t)c.B * ((c.H + t.th - 1) / t.th) * ((c.W + t.tw - 1) / t.tw); }

// The prediction is a fit to graph replay of a DenseNet's 56x56 and 28x28 layers, 40x40 and 16x16 at batch 1 and 6; one workgroup fits a
// compute unit, so every 256 of them are a round.
bool dense_pick(const ConvArgs &c1, const ConvArgs &c2, DenseTile *best, double *us) {
    *us = 1e30;
    if (!dense_shape_ok(c1, c2)) return false;
    const int ns = (c1.K + 63) / 64;
    for (int th = 1; th <= std::min(c1.H, 124); ++th) {
        if ((c1.H + (c1.H + th - 1) / th - 1) / ((c1.H + th - 1) / th) != th) continue;   // as many strips with fewer rows
        for (int tw = std::min(c1.W, 128 / (th + 2) - 2); tw >= 1; --tw) {
            if ((c1.W + (c1.W + tw - 1) / tw - 1) / ((c1.W + tw - 1) / tw) != tw) continue;
            const DenseTile t{th, tw};
            if ((th + 2) * (tw + 2) < 24 && (th < c1.H || tw < c1.W)) break;   // mostly border
            const int pf = dense_pf(t), frags = (th * tw + 15) / 16;
            const int64_t wgs = dense_wgs(c1, t), rounds = (wgs + 255) / 256;
            const double body = (pf == 1 ? 1.65 + 0.33 * ns : 2.0 + 0.6 * ns) + 0.65 * ((frags + 1) / 2) + 0.25 * ((frags + 3) / 4) + 0.0015 * std::min<int64_t>(wgs, 256);
            const double v = 1.5 + body * rounds + 0.8 * (rounds - 1);
            if (v < *us) { *us = v; *best = t; }
        }
    }
    return *us < 1e30;
}

dim3 dense_grid(const ConvArgs &c, const DenseTile &t) { return dim3((unsigned)dense_wgs(c, t)); }

template <typename T, int PF, int NS>
static hipError_t launch_one(const ConvArgs &c1, const ConvArgs &c2, const DenseTile &t, const DenseRest &a, hipStream_t s) {
    typedef DenseLoads<PF, NS> D;
    auto k = dense_layer_kernel<T, PF, NS>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return attr;
    const unsigned front = dense_front(t, D::ring), lds = front + D::fresh_bytes;
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    const int th = (c1.H + t.th - 1) / t.th, tw = (c1.W + t.tw - 1) / t.tw;
    k<<<(unsigned)dense_wgs(c1, t), 256, lds, s>>>(c1.x, c1.w, c2.w, c1.K | conv_ldx(c1) << 16, c1.H | c1.W << 16, t.th | t.tw << 16, tw, th * tw, front, a);
    return hipGetLastError();
}

hipError_t launch_dense_layer(DType dt, const ConvArgs &c1, const ConvArgs &c2, const DenseTile &t, hipStream_t s) {
    if (!dense_shape_ok(c1, c2) || t.th < 1 || t.tw < 1 || (t.th + 2) * (t.tw + 2) > 128) return hipErrorInvalidValue;
    if (!c1.x || !c1.w || !c1.bias || !c2.w || !c2.bias || !c2.y) return hipErrorInvalidValue;
    DenseRest a{};
    a.bias1 = c1.bias; a.bias2 = c2.bias; a.y = c2.y; a.B = c1.B; a.ldy = conv_ldy(c2); a.act1 = c1.relu; a.act2 = c2.relu;
    a.halo_div = make_fast_div(t.tw + 2); a.tw_div = make_fast_div(t.tw);
    const int pf = dense_pf(t), ns = (c1.K + 63) / 64;
#define CW_DENSE(P_, N_) if (pf == P_ && ns == N_) return dt == DT_F16 ? launch_one<f16, P_, N_>(c1, c2, t, a, s) : launch_one<bf16, P_, N_>(c1, c2, t, a, s)
#define CW_DENSE_N(P_) CW_DENSE(P_, 1); CW_DENSE(P_, 2); CW_DENSE(P_, 3); CW_DENSE(P_, 4); CW_DENSE(P_, 5); CW_DENSE(P_, 6); CW_DENSE(P_, 7); CW_DENSE(P_, 8)
    CW_DENSE_N(1);
    CW_DENSE_N(2);
#undef CW_DENSE_N
#undef CW_DENSE
    return hipErrorInvalidValue;
}

}  // namespace cw
