// The tail of a narrow bottleneck over few pixels in one launch: a 3x3 convolution 64 -> 64, the 1x1 to 256 with its residual and, where that is the
// result's only reader as an input, the 1x1 back to 64 of the block behind it.
// What bounds it: a chain of latencies around what a CU has to fetch, 72 KB + 32 KB (+ 32 KB) of weights.  By counters (three layers, 3136 pixels) a wave lives 11.2k clocks, in
// which 152 KB come from L2, waits 46 % of them and has a matrix instruction in the pipe for 5 %.
// So all of it is requested at the start, in the order in which it is needed, and nothing waits for more than its own part:
// - 16 or 32 pixels a workgroup, so that these few pixels still are a workgroup a CU; with 136 KB of weights in LDS there is room for one.
// - A wave has 16 of the 64 channels of the first and the third layer and 64 of the 256, and fetches their weights itself: only pixels and what a layer
//   hands to the next pass a barrier.
// - With 32 pixels the third layer's weights come into the place of the wave's own of the first, once it has read them.
// Back to back, 56x56 at batch 1 and 49x41 at batch 3 (3136 and 6027 pixels): three layers 9.3 -> 5.0 us and 10.7 -> 6.2, two layers 6.6 -> 4.3 and 7.5 -> 5.7 (with LDS
// reads left to the compiler and a branch per activation 5.6, 7.0, 4.6 and 6.2). The 64-pixel form of the
// convolution kernel, which walks the layers in chunks with two barriers each, takes 10.0 and 8.6 at 6272 pixels.
#include "conv_dlds_body.h"

namespace cw {

constexpr int kTailC = 64, kTailWide = 256, kTailTaps = 9;

template <int F>   // 16-pixel groups of a workgroup
struct TailLds {
    static constexpr unsigned W1 = 0, XS = 4 * 18432, W2 = XS + F * 18432, W3 = F == 1 ? W2 + 32768 : 0, P = (F == 1 ? W3 : W2) + 32768;
    static constexpr unsigned P_PITCH = kTailC * 2 + 16, Q_PITCH = kTailWide * 2 + 16;   // 16 consecutive pixels start on different banks
    static constexpr unsigned Q = XS;          // over the first layer's pixels
    static constexpr unsigned BIAS = P + 16 * F * P_PITCH, BYTES = BIAS + 3 * 1024;
    static_assert(16 * F * Q_PITCH <= F * 18432 && BYTES <= 160 * 1024, "");
};

// Without a branch: with one around every four values a tile was a chain of small blocks.
template <typename T>
static __device__ __forceinline__ u32x2 relu_or_none(const float (&v)[4], int act) {
    T o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (T)(act ? fmaxf(v[e], 0.f) : v[e]);
    return *reinterpret_cast<const u32x2 *>(o);
}

// The same for every activation, one branch around all of `body`, which gets the activation.
template <typename T, typename F>
static __device__ __forceinline__ void with_activation(int act, F body) {
    if (act == ACT_HSWISH) body([](const float (&v)[4]) { return activate<T>(v, ACT_HSWISH); });
    else body([act](const float (&v)[4]) { return relu_or_none<T>(v, act); });
}

template <typename T, int F, bool THIRD>
__global__ __launch_bounds__(256) void tail_kernel(const TailArgs a) {
    typedef MfmaTile<T, 16> MF;
    typedef typename Mfma<T>::v8 v8;
    typedef TailLds<F> L;
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)cw_dyn_lds;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 15, lhalf = lane >> 4;
    const unsigned row8 = lane >> 3, c8 = lane & 7;   // of a piece of 8 rows x 128 bytes; chunk c of row r lies at c ^ (r / 2) % 8
    const int m0 = xcd_tile_id(blockIdx.x, gridDim.x) * 16 * F;
    const u32x4 dx = make_desc(a.x, (unsigned)a.M * (kTailC * 2u)), dw1 = make_desc(a.w1, kTailC * kTailTaps * kTailC * 2u), dw2 = make_desc(a.w2, kTailWide * kTailC * 2u);
    const u32x4 dw3 = make_desc(THIRD ? a.w3 : a.w2, kTailC * kTailWide * 2u);
    const unsigned key_l = row8 >> 1;   // (r / 2) % 8 of row 8h + row8: key_l + 4h
    const unsigned cs[2] = {(c8 ^ key_l) << 4, (c8 ^ (key_l + 4)) << 4};
    auto load_w1 = [&](int tap) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            load_to_lds(dw1, row8 * (kTailTaps * kTailC * 2u) + cs[h], (unsigned)(wave * 16 + h * 8) * (kTailTaps * kTailC * 2u) + (unsigned)tap * (kTailC * 2u),
                        lds_base + L::W1 + (unsigned)wave * 18432u + (unsigned)(tap * 2 + h) * 1024u);
    };
    load_w1(0);
    __builtin_amdgcn_sched_barrier(0);
    // A wave's pieces of the pixels: always the same 8 of the workgroup's, of taps 0 and 2 or 1 of a filter row (16 pixels), or of all three (32)
    const int xp = F == 1 ? wave & 1 : wave;
    const int pm = m0 + xp * 8 + (int)row8;
    const unsigned x_cs = cs[xp & 1];
    const unsigned pt = fast_div((unsigned)min(pm, a.M - 1), a.w_div), pn = fast_div(pt, a.h_div);
    const int pj = min(pm, a.M - 1) - (int)pt * a.W, pi = (int)(pt - pn * (unsigned)a.H);
    const bool p_in = pm < a.M;
    auto load_x = [&](int r, int s) {
        const bool in = p_in && (unsigned)(pi + r - 1) < (unsigned)a.H && (unsigned)(pj + s - 1) < (unsigned)a.W;
        load_to_lds(dx, in ? (unsigned)(pm + (r - 1) * a.W + s - 1) * (kTailC * 2u) + x_cs : kOob, 0u, lds_base + L::XS + (unsigned)((r * 3 + s) * 2 * F + xp) * 1024u);
    };
    auto load_x_row = [&](int r) {
        if constexpr (F == 2) { load_x(r, 0); load_x(r, 1); load_x(r, 2); }
        else if (wave < 2) { load_x(r, 0); load_x(r, 2); }   // uniform
        else load_x(r, 1);
    };
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        load_x_row(r);
#pragma unroll
        for (int s = 0; s < 3; ++s)
            if (r + s > 0) load_w1(r * 3 + s);
    }
    {   // biases: wave 0 the first layer's, wave 1 the second's, the others the third's (twice the same bytes to the same place)
        const u32x4 db = make_desc(wave == 0 ? a.bias1 : wave == 1 || !THIRD ? a.bias2 : a.bias3, wave == 0 || (wave > 1 && THIRD) ? kTailC * 4u : kTailWide * 4u);
        load_to_lds(db, (unsigned)lane * 16u, 0u, lds_base + L::BIAS + (unsigned)min(wave, 2) * 1024u);
    }
    // the residual: 4 channels of each of a lane's four 16-channel tiles
    const unsigned nl = 8 * (lhalf & 1) + 4 * (lhalf >> 1);   // the channel of a lane's first row (packed weights)
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(a.res, (unsigned)a.M * (kTailWide * 2u)), ry = make_rsrc(a.y, (unsigned)a.M * (kTailWide * 2u));
    unsigned y_off[F];
    u32x2 res[F][4];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int f = 0; f < F; ++f) {
        const int m = m0 + f * 16 + lrow;
        y_off[f] = m < a.M ? (unsigned)m * (kTailWide * 2u) + (unsigned)(wave * 64 + nl) * 2u : kOob;
#pragma unroll
        for (int j = 0; j < 4; ++j) res[f][j] = __builtin_amdgcn_raw_buffer_load_b64(rr, y_off[f], j * 32, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 8; ++q)
        load_to_lds(dw2, row8 * (kTailC * 2u) + cs[q & 1], (unsigned)(wave * 64 + q * 8) * (kTailC * 2u), lds_base + L::W2 + (unsigned)(wave * 8 + q) * 1024u);
    auto load_w3 = [&] {
#pragma unroll
        for (int q = 0; q < 8; ++q)   // 64 of the 256 channels, half of the rows
            load_to_lds(dw3, row8 * (kTailWide * 2u) + cs[q & 1], (unsigned)(wave * 16 + (q & 1) * 8) * (kTailWide * 2u) + (unsigned)(q >> 1) * 128u,
                        lds_base + L::W3 + (unsigned)wave * (F == 1 ? 8192u : 18432u) + (unsigned)q * 1024u);
    };
    if (THIRD && F == 1) load_w3();
    // Loads behind the last of filter row r
    constexpr int N3 = THIRD ? 8 : 0, AFTER = 1 + 4 * F + 8 + (F == 1 ? N3 : 0);
    typename MF::acc acc[F][2];
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
        for (int k = 0; k < 2; ++k) acc[f][k] = typename MF::acc{0.f, 0.f, 0.f, 0.f};
    const unsigned key = (lrow >> 1) & 7, rd = (unsigned)lrow * 128u;
    const unsigned ck[2] = {((unsigned)lhalf ^ key) << 4, ((unsigned)(4 + lhalf) ^ key) << 4};
    auto row = [&](int r) {   // all reads, then the products: left to the compiler two or three are in flight
        v8 fw[6], fx[6][F];
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const int tap = r * 3 + (q >> 1);
            fw[q] = *reinterpret_cast<const v8 *>(cw_dyn_lds + L::W1 + (unsigned)wave * 18432u + tap * 2048u + rd + ck[q & 1]);
#pragma unroll
            for (int f = 0; f < F; ++f) fx[q][f] = *reinterpret_cast<const v8 *>(cw_dyn_lds + L::XS + (unsigned)(tap * F + f) * 2048u + rd + ck[q & 1]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int f = 0; f < F; ++f) acc[f][q & 1] = MF::mma(fw[q], fx[q][f], acc[f][q & 1]);
    };
    // (16 pixels: waves 0 and 1 have one load of pixels a filter row more)
    if (F == 2) wait_lds_loads_and_barrier<AFTER + 2 * 9>();
    else if (wave < 2) wait_lds_loads_and_barrier<AFTER + 2 * 8>();
    else wait_lds_loads_and_barrier<AFTER + 2 * 7>();
    row(0);
    if (F == 2) wait_lds_loads_and_barrier<AFTER + 9>();
    else if (wave < 2) wait_lds_loads_and_barrier<AFTER + 8>();
    else wait_lds_loads_and_barrier<AFTER + 7>();
    row(1);
    wait_lds_loads_and_barrier<AFTER - 1>();   // the biases too
    row(2);
    // first layer's result: 4 channels of a pixel, rounded as when it is stored
    with_activation<T>(a.act1, [&](auto activation) {
        const typename MF::acc b = *reinterpret_cast<const typename MF::acc *>(cw_dyn_lds + L::BIAS + (wave * 16 + nl) * 4u);
#pragma unroll
        for (int f = 0; f < F; ++f) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = acc[f][0][e] + acc[f][1][e] + b[e];
            *reinterpret_cast<u32x2 *>(cw_dyn_lds + L::P + (unsigned)(f * 16 + lrow) * L::P_PITCH + (wave * 16 + nl) * 2u) = activation(v);
        }
    });
    if (THIRD && F == 2) {
        // this wave's reads of its first weights have returned (their products are in the sums just stored)
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
        load_w3();
    }
    wait_lds_loads_and_barrier<N3>();   // the second layer's weights (and the residual); everyone's part of the first layer's result
    {
        v8 fp[F][2];
#pragma unroll
        for (int f = 0; f < F; ++f)
#pragma unroll
            for (int k = 0; k < 2; ++k) fp[f][k] = *reinterpret_cast<const v8 *>(cw_dyn_lds + L::P + (unsigned)(f * 16 + lrow) * L::P_PITCH + (unsigned)(k * 4 + lhalf) * 16u);
        typename MF::acc s[F][4], b[4];
        v8 fw[4][2];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int k = 0; k < 2; ++k) fw[j][k] = *reinterpret_cast<const v8 *>(cw_dyn_lds + L::W2 + (unsigned)wave * 8192u + j * 2048u + rd + ck[k]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) b[j] = *reinterpret_cast<const typename MF::acc *>(cw_dyn_lds + L::BIAS + 1024u + (wave * 64 + j * 16 + nl) * 4u);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int f = 0; f < F; ++f) s[f][j] = MF::mma(fw[j][k], fp[f][k], k == 0 ? typename MF::acc{0.f, 0.f, 0.f, 0.f} : s[f][j]);
        with_activation<T>(a.act2, [&](auto activation) {
#pragma unroll
            for (int f = 0; f < F; ++f)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const T *r = reinterpret_cast<const T *>(&res[f][j]);
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = s[f][j][e] + b[j][e] + (float)r[e];
                    const u32x2 o = activation(v);
                    __builtin_amdgcn_raw_buffer_store_b64(o, ry, y_off[f], j * 32, 0);
                    if (THIRD) *reinterpret_cast<u32x2 *>(cw_dyn_lds + L::Q + (unsigned)(f * 16 + lrow) * L::Q_PITCH + (unsigned)(wave * 64 + j * 16 + nl) * 2u) = o;
                }
        });
    }
    if constexpr (THIRD) {
        wait_lds_loads_and_barrier<4 * F>();   // older than the stores are the third layer's weights; everyone's part of the second's result
        const typename MF::acc b = *reinterpret_cast<const typename MF::acc *>(cw_dyn_lds + L::BIAS + 2048u + (wave * 16 + nl) * 4u);
        typename MF::acc s[F][2];
#pragma unroll
        for (int f = 0; f < F; ++f)
#pragma unroll
            for (int k = 0; k < 2; ++k) s[f][k] = typename MF::acc{0.f, 0.f, 0.f, 0.f};
        v8 fw[8], fq[8][F];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            fw[k] = *reinterpret_cast<const v8 *>(cw_dyn_lds + L::W3 + (unsigned)wave * (F == 1 ? 8192u : 18432u) + (k >> 1) * 2048u + rd + ck[k & 1]);
#pragma unroll
            for (int f = 0; f < F; ++f) fq[k][f] = *reinterpret_cast<const v8 *>(cw_dyn_lds + L::Q + (unsigned)(f * 16 + lrow) * L::Q_PITCH + (unsigned)(k * 4 + lhalf) * 16u);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int f = 0; f < F; ++f) s[f][k & 1] = MF::mma(fw[k], fq[k][f], s[f][k & 1]);
        with_activation<T>(a.act3, [&](auto activation) {
#pragma unroll
            for (int f = 0; f < F; ++f) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = s[f][0][e] + s[f][1][e] + b[e];
                const int m = m0 + f * 16 + lrow;
                if (m < a.M) *reinterpret_cast<u32x2 *>(static_cast<char *>(a.y3) + (size_t)m * (kTailC * 2) + (wave * 16 + nl) * 2u) = activation(v);
            }
        });
    }
}

// The same for many pixels, also with the projection shortcut of a stage's first block (x2, 64 channels, instead of a residual).  Workgroups of the form for few pixels, in
// several rounds, would fetch the weights again each time; here a wave holds its own in registers, 104 to 168 of the 256 that it has, and the workgroup, one
// a CU, walks its range of pixels 32 at a time: four waves by channels for each half of the 32.  The next tile's pixels and residual are on their way meanwhile.
// What bounds it: up to three tiles the start, 5.0 to 6.0 us with the first tile; each further one takes 1.8 to 3.0 us for 5.6 (projection) to 8.0 MB over the chip, 2.2 to
// 3.9 TB/s where a large copy reaches 4.7, and a wave waits 42 to 47 % of its life (kernel trace and counters at one to four tiles on 196 CUs).  Where two waves a SIMD took
// 2.1 us a tile, one took 2.6, and two with the reads of LDS left to the compiler 3.6.
// Against the convolution kernel's fused form, back to back, with projection and third layer / with the third / alone: 6272 pixels 10.5 -> 6.2 us / 9.9 -> 6.2 / 8.6 -> 5.4,
// 12544 11.0 -> 8.5 / 10.4 -> 8.5 / 9.0 -> 7.3, 25088 14.2 -> 12.9 / 13.2 -> 13.0 / 11.2 -> 11.2, 50176 in bf16 20.8 -> 19.2 / 19.4 -> 19.5 / 16.5 -> 17.0.

template <bool PROJ>
struct WalkLds {
    static constexpr unsigned X = 36864, XR = X + (PROJ ? 4096 : 16384);   // a tile's pixels and its residual or shortcut
    // W1, later W2 and W3 of the same wave, later the odd tiles | the even tiles | first layer's result | Wd, later the second layer's | biases
    static constexpr unsigned ODD = 0, EVEN = 4 * 18432, P = EVEN + XR, Q = P + 32 * TailLds<2>::P_PITCH;
    static constexpr unsigned BIAS = Q + (PROJ ? 32768 : 32 * TailLds<2>::Q_PITCH), BYTES = BIAS + 4096;
    static_assert(XR <= EVEN && 32 * TailLds<2>::Q_PITCH <= BIAS - Q && BYTES <= 160 * 1024, "");
};

template <typename T, bool THIRD, bool PROJ>
__global__ __launch_bounds__(kTailWalkThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void tail_walk_kernel(const TailArgs a) {
    typedef MfmaTile<T, 16> MF;
    typedef typename MF::acc acc_t;
    typedef typename Mfma<T>::v8 v8;
    typedef WalkLds<PROJ> L;
    constexpr unsigned P_PITCH = TailLds<2>::P_PITCH, Q_PITCH = TailLds<2>::Q_PITCH;
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)cw_dyn_lds;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6), wave = wave8 & 3, g = wave8 >> 2;   // its channels, its half of the tile
    const int lrow = lane & 15, lhalf = lane >> 4;
    const unsigned row8 = lane >> 3, c8 = lane & 7;   // as above
    const int wg0 = xcd_tile_id(blockIdx.x, gridDim.x) * a.tiles * 32;
    const int tiles = min(a.tiles, (a.M - wg0 + 31) >> 5);   // at least one
    const u32x4 dx = make_desc(a.x, (unsigned)a.M * (kTailC * 2u)), dw1 = make_desc(a.w1, kTailC * kTailTaps * kTailC * 2u), dw2 = make_desc(a.w2, kTailWide * kTailC * 2u);
    const u32x4 dw3 = make_desc(THIRD ? a.w3 : a.w2, kTailC * kTailWide * 2u), dwd = make_desc(PROJ ? a.wd : a.w2, kTailWide * kTailC * 2u);
    const u32x4 dr = make_desc(PROJ ? a.x2 : a.res, (unsigned)a.M * (PROJ ? kTailC * 2u : kTailWide * 2u));
    const unsigned key_l = row8 >> 1;
    const unsigned cs[2] = {(c8 ^ key_l) << 4, (c8 ^ (key_l + 4)) << 4};
    const unsigned own = (unsigned)wave * 18432u;   // of both waves with these channels
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const int q = i * 2 + g;
        load_to_lds(dw1, row8 * (kTailTaps * kTailC * 2u) + ((c8 ^ (key_l + 4u * (unsigned)g)) << 4), (unsigned)(wave * 16 + g * 8) * (kTailTaps * kTailC * 2u) + (unsigned)i * (kTailC * 2u),
                    lds_base + own + (unsigned)q * 1024u);
    }
    auto load_tile = [&](int t) {
        const unsigned at = lds_base + (t & 1 ? L::ODD : L::EVEN);
        const int pm = wg0 + t * 32 + wave * 8 + (int)row8, pc = min(pm, a.M - 1);
        const unsigned pt = fast_div((unsigned)pc, a.w_div), pn = fast_div(pt, a.h_div);
        const int pj = pc - (int)pt * a.W, pi = (int)(pt - pn * (unsigned)a.H);
        const unsigned x_cs = (c8 ^ (key_l + 4u * (unsigned)(wave & 1))) << 4, px = (unsigned)pm * (kTailC * 2u) + x_cs;
        const bool p_in = pm < a.M;
        auto load_x = [&](int r, int s) {
            const bool in = p_in & ((unsigned)(pi + r - 1) < (unsigned)a.H) & ((unsigned)(pj + s - 1) < (unsigned)a.W);
            load_to_lds(dx, in ? px + (unsigned)(((r - 1) * a.W + s - 1) * (kTailC * 2)) : kOob, 0u, at + (unsigned)((r * 3 + s) * 4 + wave) * 1024u);
        };
        if (g == 0) { load_x(0, 0); load_x(0, 1); load_x(0, 2); load_x(1, 0); load_x(1, 1); }   // uniform
        else {
            load_x(1, 2); load_x(2, 0); load_x(2, 1); load_x(2, 2);
            if (PROJ) load_to_lds(dr, p_in ? px : kOob, 0u, at + L::X + (unsigned)wave * 1024u);
        }
        if constexpr (!PROJ) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {   // two pixels; chunk c of pixel p lies at c ^ p % 16
                const int p = (wave8 * 2 + q) * 2 + (lane >> 5), m = wg0 + t * 32 + p;
                load_to_lds(dr, m < a.M ? (unsigned)m * (kTailWide * 2u) + (((unsigned)(lane & 31) ^ (unsigned)(p & 15)) << 4) : kOob, 0u, at + L::X + (unsigned)(wave8 * 2 + q) * 1024u);
            }
        }
    };
    load_tile(0);
    {   // (both waves the same bytes to the same place)
        const float *b = wave == 0 ? a.bias1 : wave == 1 ? a.bias2 : wave == 2 ? (THIRD ? a.bias3 : a.bias2) : PROJ ? a.biasd : a.bias2;
        const u32x4 db = make_desc(b, wave == 0 || (wave == 2 && THIRD) ? kTailC * 4u : kTailWide * 4u);
        load_to_lds(db, (unsigned)lane * 16u, 0u, lds_base + L::BIAS + (unsigned)wave * 1024u);
    }
    if constexpr (PROJ)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            load_to_lds(dwd, row8 * (kTailC * 2u) + cs[i & 1], (unsigned)(wave * 64 + (g * 4 + i) * 8) * (kTailC * 2u), lds_base + L::Q + (unsigned)(wave * 8 + g * 4 + i) * 1024u);
    const unsigned key = (lrow >> 1) & 7, rd = (unsigned)lrow * 128u;
    const unsigned ck[2] = {((unsigned)lhalf ^ key) << 4, ((unsigned)(4 + lhalf) ^ key) << 4};
    // the first layer's weights: behind them a tile's loads (5 and, with the projection, 5 a wave, or 7 and 6), the biases and the projection's weights
    if (PROJ) wait_lds_loads_and_barrier<5 + 1 + 4>();
    else if (g == 0) wait_lds_loads_and_barrier<7 + 1>();
    else wait_lds_loads_and_barrier<6 + 1>();
    v8 fw1[18], fw2[8], fw3[8], fwd[8];
#pragma unroll
    for (int k = 0; k < 18; ++k) fw1[k] = *reinterpret_cast<const v8 *>(cw_dyn_lds + own + (k >> 1) * 2048u + rd + ck[k & 1]);
    wait_lds_and_barrier();   // both waves have them
#pragma unroll
    for (int i = 0; i < 4; ++i)
        load_to_lds(dw2, row8 * (kTailC * 2u) + cs[i & 1], (unsigned)(wave * 64 + (g * 4 + i) * 8) * (kTailC * 2u), lds_base + own + (unsigned)(g * 4 + i) * 1024u);
    if constexpr (THIRD)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int q = g * 4 + i;
            load_to_lds(dw3, row8 * (kTailWide * 2u) + cs[i & 1], (unsigned)(wave * 16 + (i & 1) * 8) * (kTailWide * 2u) + (unsigned)(q >> 1) * 128u, lds_base + own + 8192u + (unsigned)q * 1024u);
        }
    const unsigned nl = 8 * (lhalf & 1) + 4 * (lhalf >> 1);   // the channel of a lane's first row (packed weights)
    const __amdgpu_buffer_rsrc_t ry = make_rsrc(a.y, (unsigned)a.M * (kTailWide * 2u)), ry3 = make_rsrc(THIRD ? a.y3 : a.y, (unsigned)a.M * (kTailC * 2u));
    const acc_t zero = {0.f, 0.f, 0.f, 0.f};
    const int half = g * 16 + lrow;   // a lane's pixel of a tile
    unsigned char *const p_at = cw_dyn_lds + L::P + (unsigned)half * P_PITCH, *const q_at = cw_dyn_lds + L::Q + (unsigned)half * Q_PITCH;
    // Reads stand before the products that use them, many at once: left to the compiler two are in flight.
    auto first = [&](int t) {
        const unsigned char *x = cw_dyn_lds + (t & 1 ? L::ODD : L::EVEN) + rd + (unsigned)g * 2048u;
        acc_t acc[2] = {zero, zero};
        v8 xa[6], xb[6];   // a filter row
        auto read = [&](v8 (&v)[6], int r) {
#pragma unroll
            for (int k = 0; k < 6; ++k) v[k] = *reinterpret_cast<const v8 *>(x + (r * 3 + (k >> 1)) * 4096u + ck[k & 1]);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto product = [&](const v8 (&v)[6], int r) {
#pragma unroll
            for (int k = 0; k < 6; ++k) acc[k & 1] = MF::mma(fw1[r * 6 + k], v[k], acc[k & 1]);
            __builtin_amdgcn_sched_barrier(0);
        };
        read(xa, 0);
        read(xb, 1);
        product(xa, 0);
        read(xa, 2);
        const acc_t b = *reinterpret_cast<const acc_t *>(cw_dyn_lds + L::BIAS + (wave * 16 + nl) * 4u);
        product(xb, 1);
        product(xa, 2);
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[0][e] + acc[1][e] + b[e];
        *reinterpret_cast<u32x2 *>(p_at + (wave * 16 + nl) * 2u) = relu_or_none<T>(v, a.act1);
    };
    auto rest = [&](int t) {
        const unsigned char *r_at = cw_dyn_lds + (t & 1 ? L::ODD : L::EVEN) + L::X;
        v8 fp[2], fd[2];
        acc_t b[4];
        u32x2 raw[4];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            fp[k] = *reinterpret_cast<const v8 *>(p_at + (unsigned)(k * 4 + lhalf) * 16u);
            if (PROJ) fd[k] = *reinterpret_cast<const v8 *>(r_at + g * 2048u + rd + ck[k]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            b[j] = *reinterpret_cast<const acc_t *>(cw_dyn_lds + L::BIAS + 1024u + (wave * 64 + j * 16 + nl) * 4u);
            if (PROJ) b[j] += *reinterpret_cast<const acc_t *>(cw_dyn_lds + L::BIAS + 3072u + (wave * 64 + j * 16 + nl) * 4u);
            const unsigned c = (unsigned)(wave * 8 + j * 2) + (nl >> 3);
            if (!PROJ) raw[j] = *reinterpret_cast<const u32x2 *>(r_at + (unsigned)half * 512u + ((c ^ (unsigned)lrow) << 4) + (nl & 4) * 2u);
        }
        __builtin_amdgcn_sched_barrier(0);
        acc_t s2[4];
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) s2[j] = MF::mma(fw2[2 * j + k], fp[k], k == 0 ? zero : s2[j]);
        if (PROJ)
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j) s2[j] = MF::mma(fwd[2 * j + k], fd[k], s2[j]);
        const int m = wg0 + t * 32 + half;
        const unsigned y_off = m < a.M ? (unsigned)m * (kTailWide * 2u) + (unsigned)(wave * 64 + nl) * 2u : kOob;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = s2[j][e] + b[j][e];
            if constexpr (!PROJ) {
                const T *r = reinterpret_cast<const T *>(&raw[j]);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += (float)r[e];
            }
            const u32x2 o = relu_or_none<T>(v, a.act2);
            __builtin_amdgcn_raw_buffer_store_b64(o, ry, y_off, j * 32, 0);
            if (THIRD) *reinterpret_cast<u32x2 *>(q_at + (unsigned)(wave * 64 + j * 16 + nl) * 2u) = o;
        }
        if constexpr (THIRD) {
            wait_lds_and_barrier();
            acc_t s[2] = {zero, zero};
            v8 fq[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) fq[k] = *reinterpret_cast<const v8 *>(q_at + (unsigned)(k * 4 + lhalf) * 16u);
            const acc_t b3 = *reinterpret_cast<const acc_t *>(cw_dyn_lds + L::BIAS + 2048u + (wave * 16 + nl) * 4u);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < 8; ++k) s[k & 1] = MF::mma(fw3[k], fq[k], s[k & 1]);
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = s[0][e] + s[1][e] + b3[e];
            __builtin_amdgcn_raw_buffer_store_b64(relu_or_none<T>(v, a.act3), ry3, m < a.M ? (unsigned)m * (kTailC * 2u) + (wave * 16 + nl) * 2u : kOob, 0, 0);
        }
    };
    wait_lds_loads_and_barrier<4 + (THIRD ? 4 : 0)>();   // the first tile and the biases
    first(0);
    wait_lds_loads_and_barrier<0>();   // the other weights; everyone's part of the first layer's result
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        fw2[k] = *reinterpret_cast<const v8 *>(cw_dyn_lds + own + (k >> 1) * 2048u + rd + ck[k & 1]);
        if (THIRD) fw3[k] = *reinterpret_cast<const v8 *>(cw_dyn_lds + own + 8192u + (k >> 1) * 2048u + rd + ck[k & 1]);
        if (PROJ) fwd[k] = *reinterpret_cast<const v8 *>(cw_dyn_lds + L::Q + (unsigned)wave * 8192u + (k >> 1) * 2048u + rd + ck[k & 1]);
    }
    wait_lds_and_barrier();   // their places are free
    if (tiles > 1) load_tile(1);
    rest(0);
    for (int t = 1; t < tiles; ++t) {
        // tile t has landed: younger than it are only the last one's stores.  The other buffer is free: everyone has read the last tile.
        wait_lds_loads_and_barrier<4 + (THIRD ? 1 : 0)>();
        if (t + 1 < tiles) load_tile(t + 1);
        first(t);
        wait_lds_and_barrier();
        rest(t);
    }
}

int tail_bm(int64_t M) { return M <= 16 * 256 ? 16 : 32; }

// Up to a round of 32 pixels a workgroup.  From 96 tiles of 64 pixels on the plan has the convolution kernel's own form, so that this one sees less.
bool tail_shape_ok(int64_t M, int32_t H, int32_t W) { return M >= 1 && M <= 32 * 256 && H >= 1 && W >= 1 && M % ((int64_t)H * W) == 0; }

template <typename T, int F, bool THIRD>
static hipError_t launch_one(const TailArgs &a, hipStream_t s) {
    auto k = tail_kernel<T, F, THIRD>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)TailLds<F>::BYTES);
    if (attr != hipSuccess) return attr;
    k<<<(unsigned)((a.M + 16 * F - 1) / (16 * F)), 256, TailLds<F>::BYTES, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_tail(DType dt, const TailArgs &a_in, hipStream_t s) {
    TailArgs a = a_in;
    if (!tail_shape_ok(a.M, a.H, a.W) || !a.x || !a.w1 || !a.bias1 || !a.w2 || !a.bias2 || !a.res || !a.y) return hipErrorInvalidValue;
    if (a.w3 && (!a.bias3 || !a.y3)) return hipErrorInvalidValue;
    a.w_div = make_fast_div((uint32_t)a.W);
    a.h_div = make_fast_div((uint32_t)a.H);
#define CW_TAIL(T_, F_) (a.w3 ? launch_one<T_, F_, true>(a, s) : launch_one<T_, F_, false>(a, s))
    if (tail_bm(a.M) == 16) return dt == DT_F16 ? CW_TAIL(f16, 1) : CW_TAIL(bf16, 1);
    return dt == DT_F16 ? CW_TAIL(f16, 2) : CW_TAIL(bf16, 2);
#undef CW_TAIL
}

// Pixels a workgroup: as many tiles of 32 as leave no CU more than one workgroup.
int tail_walk_bm(int64_t M) { return 32 * (int)((M + 32 * 256 - 1) / (32 * 256)); }

bool tail_walk_ok(int64_t M, int32_t H, int32_t W) { return M >= 1 && M < (1 << 21) && H >= 1 && W >= 1 && M % ((int64_t)H * W) == 0; }

template <typename T, bool THIRD, bool PROJ>
static hipError_t launch_walk_one(const TailArgs &a, hipStream_t s) {
    auto k = tail_walk_kernel<T, THIRD, PROJ>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)WalkLds<PROJ>::BYTES);
    if (attr != hipSuccess) return attr;
    k<<<(unsigned)((a.M + 32 * a.tiles - 1) / (32 * a.tiles)), kTailWalkThreads, WalkLds<PROJ>::BYTES, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_tail_walk(DType dt, const TailArgs &a_in, hipStream_t s) {
    TailArgs a = a_in;
    if (!tail_walk_ok(a.M, a.H, a.W) || !a.x || !a.w1 || !a.bias1 || !a.w2 || !a.bias2 || !a.y) return hipErrorInvalidValue;
    if (a.wd ? !a.x2 || !a.biasd : !a.res) return hipErrorInvalidValue;
    if (a.w3 && (!a.bias3 || !a.y3)) return hipErrorInvalidValue;
    if (a.act1 > ACT_RELU || a.act2 > ACT_RELU || a.act3 > ACT_RELU) return hipErrorInvalidValue;   // as the plan fuses
    a.w_div = make_fast_div((uint32_t)a.W);
    a.h_div = make_fast_div((uint32_t)a.H);
    a.tiles = tail_walk_bm(a.M) / 32;
#define CW_WALK(T_) (a.w3 ? (a.wd ? launch_walk_one<T_, true, true>(a, s) : launch_walk_one<T_, true, false>(a, s)) : (a.wd ? launch_walk_one<T_, false, true>(a, s) : launch_walk_one<T_, false, false>(a, s)))
    return dt == DT_F16 ? CW_WALK(f16) : CW_WALK(bf16);
#undef CW_WALK
}

}  // namespace cw
