// A 1x1 convolution and the depthwise 3x3 convolution that reads it, in one launch that keeps what is between them in LDS.
//
// Bound: at small batches a launch of either is a chain of latencies (dispatch, arguments, one round trip to memory, stores: 3.2 us within
// an EXEC of MobileNet at batch 1, of which the arithmetic is a tenth) and on a slow host the 2.8 us that the host needs to
// issue it, so what pays is one chain and one launch less.  Depthwise channels do not meet, so a workgroup takes 16 to 64 of them and some rows
// of the result, computes the 1x1 for those channels over the rows and the one row above and below them that the filter
// reaches (whole rows: the pixels are one run of memory), and filters them out of LDS.  Of the 1x1 only the border rows are computed twice;
// the other way round (the depthwise result inside the 1x1 that reads it) every channel tile filters all channels again: 8.1 us against 5.3
// for the two launches at 14x14x512.
// The 1x1: weights in LDS, loaded directly and swizzled as in the convolution kernel; the pixels go straight to registers, as the
// 16x16x32 matrix instruction's operand is 16 contiguous bytes a lane and no two waves share a pixel; two runs of KS steps of K are in
// flight.  Its result is rounded to the storage type as if stored, and stored where another op reads it.
// MobileNet 224x224: 29 launches -> 20 at batch 1; EXEC by plain launches 92.1 -> 87.9 us, a pass of back-to-back calls 107..115 -> 87..89 where
// the host is slow; 128x128 batch 1 by graph replay 88.4 -> 78.6, batch 16 of 64x64 99.5 -> 90.7.
#include <cmath>

#include "conv_dlds_body.h"

namespace cw {

struct alignas(64) PwDwRest {
    const void *res;
    void *y, *d;
    const float *bias, *bias_d;
    const void *wt;
    int32_t act, act_d;
    FastDiv wo_div, k8_div;
    int32_t B, Wo;
};

// LDS: weights of the 1x1 [BN][K] | taps [9][BN] | bias of the depthwise convolution [BN] | 16 zero bytes | result of the 1x1 [pixels][BN + 8]
constexpr unsigned pw_dw_pitch(int nf) { return 16 * nf * 2 + 16; }   // bytes of a pixel: 16 consecutive ones start on different banks
static unsigned pw_dw_lds(const PwDwTile &t, int K, int pixels) {
    const unsigned bn = 16 * t.nf;
    return bn * K * 2 + 9 * bn * 2 + bn * 4 + 16 + (unsigned)pixels * pw_dw_pitch(t.nf);
}

template <typename T, int WAVES, int PF, int NF, int KS>
__global__ __launch_bounds__(64 * WAVES) void pw_dw_kernel(const void *x, const void *w, int K_N, int H_W, int Ho_rows, int slices, int strips, int stride, const PwDwRest a) {
    const int K = K_N & 0xffff, N = (unsigned)K_N >> 16, H = H_W & 0xffff, W = (unsigned)H_W >> 16, Ho = Ho_rows & 0xffff, rows = (unsigned)Ho_rows >> 16;
    typedef MfmaTile<T, 16> MF;
    typedef typename Mfma<T>::v8 v8;
    constexpr int NT = 64 * WAVES, BN = 16 * NF, C8 = BN / 8;
    constexpr unsigned PITCH = pw_dw_pitch(NF);
    static_assert(NT % C8 == 0 && 2 * PF * KS < 64, "");
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)cw_dyn_lds;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 15, lhalf = lane >> 4;
    const int tile = xcd_tile_id(blockIdx.x, gridDim.x);
    const int t1 = tile_div(tile, slices), slice = tile - t1 * slices, n = tile_div(t1, strips), strip = t1 - n * strips;
    const int n0 = slice * BN, r0 = strip * rows, r1 = min(r0 + rows, Ho);
    const int ia = max(r0 * stride - 1, 0), ib = min((r1 - 1) * stride + 2, H);
    const int px0 = (n * H + ia) * W, P = (ib - ia) * W;
    const unsigned K2 = (unsigned)K * 2u;
    const u32x4 dw = make_desc(static_cast<const char *>(w) + (size_t)n0 * K2, BN * K2);
    // weights into LDS, swizzled like the convolution kernel's operands
    const unsigned k8 = (unsigned)K >> 3, ks = K >= 128 ? 0 : K == 64 ? 1 : 2, km = K >= 128 ? 15 : K == 64 ? 7 : 3;
    for (unsigned c0 = wave * 64u; c0 < BN * k8; c0 += NT) {
        const unsigned cid = c0 + lane, row = fast_div(cid, a.k8_div), pc = cid - row * k8;
        load_to_lds(dw, row * K2 + ((pc ^ ((row >> ks) & km)) << 4), 0u, lds_base + c0 * 16u);
    }
    const unsigned M = (unsigned)a.B * H * W;
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(x, M * K2);
    // pixels straight to registers: the lane's operand is 8 channels of one pixel
    unsigned xo[PF];
    u32x4 xa[PF][KS], xb[PF][KS];
#pragma unroll
    for (int f = 0; f < PF; ++f) {
        const int m = (wave + f * WAVES) * 16 + lrow;
        xo[f] = m < P ? (unsigned)(px0 + m) * K2 + lhalf * 16u : kOob;
    }
    const int chunks = K / (32 * KS);
    auto load = [&](u32x4 (&b)[PF][KS], int kc) {
#pragma unroll
        for (int f = 0; f < PF; ++f)
#pragma unroll
            for (int t = 0; t < KS; ++t) b[f][t] = __builtin_amdgcn_raw_buffer_load_b128(rx, (kc < chunks ? xo[f] : kOob) + t * 64u, (unsigned)kc * (KS * 64u), 0);
    };
    const unsigned o_taps = BN * K2, o_bias = o_taps + 9 * BN * 2, o_zero = o_bias + BN * 4, o_y = o_zero + 16;
    // taps and bias of the depthwise convolution, the zeros
    u32x4 small = {0u, 0u, 0u, 0u};
    if (tid < 9 * C8) small = *reinterpret_cast<const u32x4 *>(static_cast<const T *>(a.wt) + (tid / C8) * N + n0 + (tid % C8) * 8);
    else if (tid < 9 * C8 + BN / 4) small = *reinterpret_cast<const u32x4 *>(a.bias_d + n0 + (tid - 9 * C8) * 4);
    const unsigned nl = n0 + 8 * (lhalf & 1) + 4 * (lhalf >> 1);   // first of the lane's four output channels of channel tile 0
    u32x4 bv[NF];
    u32x2 rv[PF][NF];
    {
        const __amdgpu_buffer_rsrc_t rb = make_rsrc(a.bias, N * 4u), rr = make_rsrc(a.res ? a.res : x, M * N * 2u);
#pragma unroll
        for (int j = 0; j < NF; ++j) bv[j] = __builtin_amdgcn_raw_buffer_load_b128(rb, (nl + 16 * j) * 4u, 0, 0);
#pragma unroll
        for (int f = 0; f < PF; ++f) {
            const int m = (wave + f * WAVES) * 16 + lrow;
#pragma unroll
            for (int j = 0; j < NF; ++j)
                rv[f][j] = __builtin_amdgcn_raw_buffer_load_b64(rr, a.res && m < P ? ((unsigned)(px0 + m) * N + nl + 16 * j) * 2u : kOob, 0, 0);
        }
    }
    load(xa, 0);
    load(xb, 1);
    if (tid < 9 * C8 + BN / 4 + 1) *reinterpret_cast<u32x4 *>(cw_dyn_lds + o_taps + tid * 16) = small;
    typename MF::acc acc[PF][NF];
#pragma unroll
    for (int f = 0; f < PF; ++f)
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[f][j] = typename MF::acc{0.f, 0.f, 0.f, 0.f};
    const unsigned key = (lrow >> ks) & km;
    auto compute = [&](const u32x4 (&b)[PF][KS], int kc) {
        v8 fw[KS][NF];
#pragma unroll
        for (int t = 0; t < KS; ++t) {
            const unsigned c = ((unsigned)(kc * KS + t) * 4u + lhalf) ^ key;
#pragma unroll
            for (int j = 0; j < NF; ++j) fw[t][j] = *reinterpret_cast<const v8 *>(cw_dyn_lds + (unsigned)(16 * j + lrow) * K2 + (c << 4));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < KS; ++t)
#pragma unroll
            for (int f = 0; f < PF; ++f)
#pragma unroll
                for (int j = 0; j < NF; ++j) acc[f][j] = MF::mma(fw[t][j], __builtin_bit_cast(v8, b[f][t]), acc[f][j]);
    };
    wait_lds_loads_and_barrier<2 * PF * KS>();   // the weights have landed: younger are the loads of pixels alone
    for (int kc = 0; kc < chunks; kc += 2) {
        compute(xa, kc);
        load(xa, kc + 2);
        if (kc + 1 < chunks) compute(xb, kc + 1);
        load(xb, kc + 3);
    }
    // the 1x1's epilogue into LDS
#pragma unroll
    for (int f = 0; f < PF; ++f) {
        const int m = (wave + f * WAVES) * 16 + lrow;
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            const float *b = reinterpret_cast<const float *>(&bv[j]);
            const T *r = reinterpret_cast<const T *>(&rv[f][j]);
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = acc[f][j][e] + b[e] + (float)r[e];
            if (m < P) *reinterpret_cast<u32x2 *>(cw_dyn_lds + o_y + (unsigned)m * PITCH + (nl - n0 + 16 * j) * 2u) = activate<T>(v, a.act);
        }
    }
    wait_lds_and_barrier();
    const int c = tid % C8;
    u32x4 taps[9];
    float bd[8];
#pragma unroll
    for (int k = 0; k < 9; ++k) taps[k] = *reinterpret_cast<const u32x4 *>(cw_dyn_lds + o_taps + (k * C8 + c) * 16);
#pragma unroll
    for (int e = 0; e < 8; ++e) bd[e] = *reinterpret_cast<const float *>(cw_dyn_lds + o_bias + c * 32 + e * 4);
    const int px_out = (r1 - r0) * a.Wo;
    for (int o = tid / C8; o < px_out; o += NT / C8) {
        const int orow = (int)fast_div((unsigned)o, a.wo_div), ocol = o - orow * a.Wo;
        const int ih0 = (r0 + orow) * stride - 1, iw0 = ocol * stride - 1;
        float s[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] = bd[e];
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const int ih = ih0 + k / 3, iw = iw0 + k % 3;
            const bool ok = (unsigned)ih < (unsigned)H && (unsigned)iw < (unsigned)W;
            const v8 f = __builtin_bit_cast(v8, ok ? taps[k] : u32x4{0u, 0u, 0u, 0u});   // outside the image 0 * 0, also where the tap is infinite
            const v8 v = *reinterpret_cast<const v8 *>(cw_dyn_lds + (ok ? o_y + (unsigned)((ih - ia) * W + iw) * PITCH + c * 16u : o_zero));
#pragma unroll
            for (int e = 0; e < 8; ++e) s[e] += (float)v[e] * (float)f[e];
        }
        *reinterpret_cast<u32x4 *>(static_cast<T *>(a.d) + ((size_t)(n * Ho + r0 + orow) * a.Wo + ocol) * N + n0 + c * 8) = activate<T>(s, a.act_d);
    }
    if (a.y) {   // the rows of the 1x1's result that this strip owns
        const int ya = r0 * stride, yb = strip + 1 == strips ? H : r1 * stride;
        for (int o = tid / C8; o < (yb - ya) * W; o += NT / C8)
            *reinterpret_cast<u32x4 *>(static_cast<T *>(a.y) + ((size_t)(n * H + ya) * W + o) * N + n0 + c * 8) =
                *reinterpret_cast<const u32x4 *>(cw_dyn_lds + o_y + (unsigned)((ya - ia) * W + o) * PITCH + c * 16u);
    }
}

static int pw_dw_pixels(const PwDwTile &t, int H, int W, int stride) { return std::min((t.rows - 1) * stride + 3, H) * W; }

// 32-deep steps of K that a wave requests at a time, as far as the registers go (0: no such kernel).
static constexpr int pw_dw_ks(int pf, int nf, int K) {
    return pf * nf > 8 ? 0 : K % 256 == 0 && pf <= 2 && nf <= 2 ? 8 : K % 128 == 0 ? 4 : K == 64 && pf >= 2 ? 2 : K == 32 && pf == 4 ? 1 : 0;
}

// Shapes that the kernel's indexing relies on.
static bool pw_dw_shape_ok(const ConvArgs &c, const DwArgs &d) {
    if (c.K != 32 && c.K != 64 && c.K % 128 != 0) return false;   // the swizzle of the weights' rows
    if (c.K < 32 || c.Cout < 32 || c.Cout % 32 != 0 || c.Cout > 32767 || c.K > 32767 || d.H > 32767 || d.W > 32767 || d.H < 1 || d.W < 1 || d.B < 1) return false;
    if (d.kh != 3 || d.kw != 3 || d.pad != 1 || d.res || (d.stride != 1 && d.stride != 2)) return false;
    if (d.Ho != (d.H - 1) / d.stride + 1 || d.Wo != (d.W - 1) / d.stride + 1 || d.C != c.Cout || (int64_t)c.M != (int64_t)d.B * d.H * d.W) return false;
    return (int64_t)d.B * d.H * d.W * std::max(c.K, c.Cout) < (1ll << 30);
}

// The line between one launch and two: a launch that fills the chip once at most, and is predicted to take no more than 8 us and
// less than the two.  The prediction is a fit to the shapes of MobileNet's maps at batch 1, 2, 4 and 16 by graph replay (10 % mean
// error; the tile it takes costs 3 % over the best one in the mean, 10 % at batch 1 to 4 at worst), and 0.9 us that a launch takes
// longer within an EXEC, where its operands are in no near cache: with 0.6 EXEC of MobileNet batch 3 was 3 us longer than with the two
// launches, with 1.2 batch 1 3 us longer than with 0.9.  By graph replay, this launch against the two on their best tiles: 14x14, 256 -> 512 channels,
// batch 1 4.2 / 5.1 us, batch 4 5.8 / 5.7; 512 -> 512 with a residual 5.0 / 5.4, batch 4 7.2 / 6.2; 56x56, 64 -> 128, batch 1 4.7 / 5.2, batch 4
// 7.5 / 7.6; 7x7, 512 -> 1024, batch 4 4.7 / 5.8.
bool pw_dw_pick(const ConvArgs &c, const DwArgs &d, bool keep, PwDwTile *best, double *us) {
    if (!pw_dw_shape_ok(c, d)) return false;
    *us = 1e30;
    PwDwTile t;
    for (t.waves = 4; t.waves <= 8; t.waves *= 2)
        for (t.pf = 1; t.pf <= 4; t.pf *= 2)
            for (t.nf = 1; t.nf <= (t.waves == 8 ? 4 : 2); t.nf *= 2)
                for (int strips = 1; strips <= d.Ho; ++strips) {
                    t.rows = (d.Ho + strips - 1) / strips;
                    const int px = pw_dw_pixels(t, d.H, d.W, d.stride), bn = 16 * t.nf, slots = 16 * t.waves * t.pf;
                    const int64_t wgs = (int64_t)d.B * ((d.Ho + t.rows - 1) / t.rows) * (c.Cout / bn);
                    if (wgs > 256) break;
                    if (px > slots || c.Cout % bn != 0 || !pw_dw_ks(t.pf, t.nf, c.K) || pw_dw_lds(t, c.K, px) > 160 * 1024) continue;
                    const double w4 = t.waves / 4.0, out_kb = px * bn * 2 / 1024.0;
                    const double v = 3.32 + 0.01246 * (slots + bn) * c.K * 2 / 1024.0 + 0.256 * ((t.rows * d.Wo * bn / 8 + 64 * t.waves - 1) / (64 * t.waves)) * w4 +
                                     (keep || c.res ? 0.098 : 0.0) * out_kb + 0.0047 * t.pf * t.nf * c.K / 32 * w4 + 0.1 * out_kb + 0.116 * t.pf * w4;
                    if (v < *us) { *us = v; *best = t; }
                }
    *us += 0.9;
    return *us <= 8.0;
}

template <int WAVES, int PF, int NF, int KS>
static hipError_t launch_one(DType dt, const ConvArgs &c, const DwArgs &d, bool keep, const PwDwTile &t, hipStream_t s) {
    PwDwRest a{};
    a.wt = d.w; a.bias = c.bias; a.bias_d = d.bias; a.res = c.res; a.y = keep ? c.y : nullptr; a.d = d.y;
    a.B = d.B; a.Wo = d.Wo; a.act = c.relu; a.act_d = d.act;
    a.wo_div = make_fast_div(d.Wo); a.k8_div = make_fast_div(c.K / 8);
    const int slices = c.Cout / (16 * NF), strips = (d.Ho + t.rows - 1) / t.rows;
    const unsigned lds = pw_dw_lds(t, c.K, pw_dw_pixels(t, d.H, d.W, d.stride));
    auto kern = dt == DT_F16 ? pw_dw_kernel<f16, WAVES, PF, NF, KS> : pw_dw_kernel<bf16, WAVES, PF, NF, KS>;
    static const hipError_t attr[2] = {hipFuncSetAttribute(reinterpret_cast<const void *>(pw_dw_kernel<f16, WAVES, PF, NF, KS>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024),
                                       hipFuncSetAttribute(reinterpret_cast<const void *>(pw_dw_kernel<bf16, WAVES, PF, NF, KS>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)};
    if (attr[0] != hipSuccess || attr[1] != hipSuccess) return attr[0] != hipSuccess ? attr[0] : attr[1];
    kern<<<a.B * strips * slices, 64 * WAVES, lds, s>>>(c.x, c.w, c.K | c.Cout << 16, d.H | d.W << 16, d.Ho | t.rows << 16, slices, strips, d.stride, a);
    return hipGetLastError();
}

dim3 pw_dw_grid(const ConvArgs &c, const DwArgs &d, const PwDwTile &t) { return dim3(d.B * ((d.Ho + t.rows - 1) / t.rows) * (c.Cout / (16 * t.nf))); }

hipError_t launch_pw_dw(DType dt, const ConvArgs &c, const DwArgs &d, bool keep, const PwDwTile &t, hipStream_t s) {
    if (!pw_dw_shape_ok(c, d) || t.rows < 1 || t.rows > d.Ho || t.nf < 1 || c.Cout % (16 * t.nf) != 0) return hipErrorInvalidValue;
    const int px = pw_dw_pixels(t, d.H, d.W, d.stride);
    if (px > 16 * t.waves * t.pf || pw_dw_lds(t, c.K, px) > 160 * 1024) return hipErrorInvalidValue;
    if (c.Cin != c.K || conv_ldx(c) != c.K || conv_ldy(c) != c.Cout || d.ldx != d.C || d.ldy != d.C) return hipErrorInvalidValue;   // dense tensors only
    if (!c.x || !c.w || !c.bias || !d.w || !d.bias || !d.y || (keep && !c.y)) return hipErrorInvalidValue;
    const int ks = pw_dw_ks(t.pf, t.nf, c.K);
#define CW_PW_DW(W_, P_, N_, K_) if (t.waves == W_ && t.pf == P_ && t.nf == N_ && ks == K_) return launch_one<W_, P_, N_, K_>(dt, c, d, keep, t, s)
#define CW_PW_DW_N(P_, K_) CW_PW_DW(4, P_, 1, K_); CW_PW_DW(4, P_, 2, K_); CW_PW_DW(8, P_, 1, K_); CW_PW_DW(8, P_, 2, K_)
    CW_PW_DW_N(1, 4); CW_PW_DW(8, 1, 4, 4); CW_PW_DW_N(1, 8);
    CW_PW_DW_N(2, 2); CW_PW_DW(8, 2, 4, 2); CW_PW_DW_N(2, 4); CW_PW_DW(8, 2, 4, 4); CW_PW_DW_N(2, 8);
    CW_PW_DW_N(4, 1); CW_PW_DW_N(4, 2); CW_PW_DW_N(4, 4);
#undef CW_PW_DW_N
#undef CW_PW_DW
    return hipErrorInvalidValue;
}

}  // namespace cw
