// Shared pieces of the convolution kernels: MFMA wrappers, buffer descriptors, the LDS swizzle
// and the fused epilogue (bias + residual + ReLU + store, and the in-kernel split-K reduction).
#pragma once
#include <type_traits>

#include "common.h"

namespace cw {
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr unsigned kOob = 0x80000000u;  // byte offset beyond any buffer (buffers are < 2 GiB)

// MODE_TAIL: MODE_GEMM whose K ends in part of a slice (a form of its own: the masks cost the plain one 1.5 %)
enum ConvMode : int { MODE_CONV = 0, MODE_GEMM = 1, MODE_STEM = 2, MODE_TAIL = 3 };

// LDS stages of a tile's ring: 4 where that still lets two workgroups share a CU's 160 KiB, else 3.
constexpr int conv_ring_stages(int stage_bytes) { return stage_bytes * 4 <= 80 * 1024 ? 4 : stage_bytes * 3 <= 160 * 1024 ? 3 : 2; }

// Waves of a workgroup that only load (conv_loader_body.h).
constexpr int kLoaderWaves = 4;
// Forms that have them: tiles of one or two wave groups whose waves' registers fit beside the loaders'.  Four groups put a multiplying wave of every
// group on a SIMD already, and with one step a slice and group the loaders' own chain from barrier to barrier is the longer one: ResNet-18 64x64 batch 1
// 97.1 us without, 101.4 with them (its 32x32 tiles on slices of 64 4.0 -> 4.6 us a launch), ResNet-50 batch 1 187 and 189.
// Registers: a wave's 512 a lane and SIMD are shared with the loaders, and a tile of MFMA tiles of 32x32 takes 16 accumulators, about 24 of operands and 8 of
// residual for each.  On eight multiplying waves (three a SIMD then) waves of 64x64 do not fit, nor do waves of 128x64 and 64x128 anywhere: they spilled in the
// loop over the slices, 256x128 and 128x256 on eight waves 29.1 -> 32.9 us for 1x7 of 256 channels at 56x56 batch 8 and 9.8 -> 15.2 for 1x1 256 -> 128 there
// at batch 16, 256x256 3-10 times as slow.
// Not with split K: in two and four splits launches took 0.73-2.1 times the time, by tile (80-97 shapes each) 0.87-1.07 in the median and 1.3 for 1x1 on
// 32x32 with slices of 128; and a ticket a wave, which two groups that finish a tile together draw, takes eight times the arrival counters.
constexpr bool conv_has_loaders(int mode, bool splitk, bool fused, int bm, int bn, int waves, int kg) {
    return mode != MODE_STEM && !splitk && !fused && kg <= 2 && 48 * (bm * bn * kg / (waves * 1024)) + 16 <= 512 / ((waves + kLoaderWaves + 3) / 4) &&
           !(mode == MODE_GEMM && bm * bn * kg >= waves * 4096);   // 1x1 in waves of 64x64: 1.04 times the time in the median of 340 launches
}
// The launches of such a form that are issued with them: those whose workgroups are on the CUs all at once.  Loaders take workgroups' places: with them
// two fit a CU, one of eight multiplying waves or of a larger tile, where up to five of the same tile would.  Behind that a workgroup's set-up and epilogue
// stand alone: 1x1 64 -> 256 at 56x56 batch 16 13.2 -> 17.3 us on 64x64, 32 -> 64 at 112x112 10.7 -> 27.8 on 32x32, 7x1 of 256 channels at 56x56 66 -> 78 on
// 128x64 in two groups.  One slice on a CU of its own has nothing to overlap and pays for the longer start: 128x128 on eight waves 4.1 -> 4.4.
// More of them gain with general addressing where the ring leaves a CU no room for more workgroups either: 0.85-1.0 of the time, 3x3 of 512 channels at 56x56 batch
// 16 388 -> 352 us on 64x64 with slices of 128 and 276 -> 251 on 128x128 on eight waves, both with rings of 96 KB.  1x1s gain on four multiplying waves where K is long
// enough beside the tile's pixels.  Whole EXECs without and with: MobileNet batch 16 at 224x224 196.2 -> 192.5 and at 208x208 190.0 -> 187.2 (128 channels at
// 128x64, 784 and 676 workgroups), batch 12 186.7 -> 185.1 (one slice of 128 at 64x64, 1176; ResNet-50 208x208 batch 7, 592: 306.7 -> 309.0), DenseNet 193x193
// batch 14 234.2 -> 233.0; Inception 224x224 batch 16 410 -> 408.5 (512 channels at 128x64, 1568), but 161x161 batch 12 193.0 -> 196.5 (632) and, by its
// pairs, 177x177 batch 9 215.0 -> 216.8; 2048 channels at 56x56, 12544 workgroups of 128x64, 606 -> 641 a launch.
// Over 7900 pairs of shape and tile inside EXECs, whole K, launches take 0.74-1.0 times the time in the mean by tile and form, without the rule 0.72-1.04.
constexpr bool conv_loads_apart(int mode, bool pair, int bm, int bn, int bk, int waves, int K, long long workgroups) {
    const int fit = waves < 8 && bm * bn * bk <= waves * 131072 ? 2 : 1, slices = (K + bk - 1) / bk, stage = (bm + bn) * bk * 2;
    if (workgroups <= 256 * fit) return fit == 2 || slices > 1;
    if (pair || waves < 4) return false;
    if (mode == MODE_CONV) return (slices < conv_ring_stages(stage) ? slices : conv_ring_stages(stage)) * stage * (fit + 1) > 160 * 1024;
    if (waves > 4 || fit == 1) return false;
    return slices == 1 ? bk == 128 && workgroups >= 1024 : bm * K >= 16384 && K <= 512 && (workgroups >= 768 || K <= 256);
}

// n / d for a divisor prepared on the host (round-up multiplier; exact for every 32-bit n).
static __device__ __forceinline__ unsigned fast_div(unsigned n, const FastDiv &d) {
    const unsigned t = __umulhi(d.magic, n);
    return (t + ((n - t) >> d.sh1)) >> d.sh2;
}

static __device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *p, unsigned bytes) {
    // raw buffer (stride 0), 32-bit data format word as on every CDNA part
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000);
}

template <typename T>
struct Mfma;
template <>
struct Mfma<f16> {
    typedef _Float16 v8 __attribute__((ext_vector_type(8)));
    static __device__ __forceinline__ f32x16 mma(v8 rows, v8 cols, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(rows, cols, c, 0, 0, 0);
    }
};
template <>
struct Mfma<bf16> {
    typedef __bf16 v8 __attribute__((ext_vector_type(8)));
    static __device__ __forceinline__ f32x16 mma(v8 rows, v8 cols, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows, cols, c, 0, 0, 0);
    }
};

// One MFMA tile of MT pixels x MT channels: 32 (16-deep steps, 16 accumulators a lane) or 16 (32-deep, 4).
template <typename T, int MT>
struct MfmaTile {
    typedef f32x16 acc;
    static constexpr int K = 16, REGS = 16;
    static __device__ __forceinline__ acc mma(typename Mfma<T>::v8 rows, typename Mfma<T>::v8 cols, acc c) { return Mfma<T>::mma(rows, cols, c); }
};
template <typename T>
struct MfmaTile<T, 16> {
    typedef float acc __attribute__((ext_vector_type(4)));
    static constexpr int K = 32, REGS = 4;
    static __device__ __forceinline__ acc mma(typename Mfma<T>::v8 rows, typename Mfma<T>::v8 cols, acc c) {
        if constexpr (std::is_same<T, f16>::value) return __builtin_amdgcn_mfma_f32_16x16x32_f16(rows, cols, c, 0, 0, 0);
        else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(rows, cols, c, 0, 0, 0);
    }
};

// Element offset of 16-byte chunk c of `row` inside a [rows][BK] LDS stage.  A 16-byte-per-lane
// LDS access is served 16 lanes (256 bytes, all 64 banks) per clock, and an MFMA operand read
// has 16 consecutive rows at one chunk index in such a group.  With 128-byte rows two rows
// share 256 bytes, so the chunk index is XORed with (row/2)%8: rows of equal parity then land
// on 8 different chunk positions and the two parities on the two halves.  With 64-byte rows
// four rows share 256 bytes and the key is (row/4)%4; with 256-byte rows every row covers all
// banks and the key is row%16.
template <int BK>
static __device__ __forceinline__ int swz_key(int row) {
    return BK >= 128 ? (row & 15) : BK == 64 ? ((row >> 1) & 7) : ((row >> 2) & 3);
}
template <int BK>
static __device__ __forceinline__ int swz(int row, int c) {
    return row * BK + ((c ^ swz_key<BK>(row)) << 3);
}

// ---- epilogue ------------------------------------------------------------------------------
// Accumulator layout (weights are the MFMA row operand, pixels the column operand): the lane
// holds pixel m0+wm0+32i+lane%32; of channel tile j its registers 8q..8q+7 are channels
// n0+wn0+32j+16q+8*(lane/32) .. +7  (q = 0, 1).
struct EpiPos {
    int m0, n0, wm0, wn0, lrow, lhalf;
};

// Split-K: every workgroup of a tile stores its raw fp32 partial tile, then takes a ticket.
// The one that draws the last ticket adds the partial tiles of all splits in split order (its
// own included, re-read like the others, so the sum does not depend on which workgroup came
// last) and returns true; the others return false and are done.
// Workgroups of one tile may sit on different XCDs, whose L2s are not coherent for plain
// accesses.  The partial sums therefore travel as device-scope accesses (sc1: stores write
// through, loads do not hit a stale local line), which costs no cache-wide write-back or
// invalidate; a store is complete once vmcnt has counted it.
template <int TM, int TN>
static __device__ __forceinline__ bool splitk_exchange(f32x16 (&acc)[TM][TN], const ConvArgs &a, const EpiPos &p, int tile_id) {
    constexpr int kDeviceScope = 16;  // cache-policy operand: sc1
    __shared__ int s_last;
    const unsigned mn = (unsigned)a.M * a.Cout;
    {
        const __amdgpu_buffer_rsrc_t rp = make_rsrc(a.partial + (size_t)blockIdx.y * a.M * a.Cout, mn * 4u);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const unsigned m = p.m0 + p.wm0 + i * 32 + p.lrow;
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const unsigned n = p.n0 + p.wn0 + j * 32 + q * 16 + p.lhalf * 8;
                    const unsigned o = (m < (unsigned)a.M && n < (unsigned)a.Cout) ? (m * a.Cout + n) * 4u : kOob;
                    const f32x16 &v = acc[i][j];
                    __builtin_amdgcn_raw_buffer_store_b128(
                        u32x4{__float_as_uint(v[8 * q + 0]), __float_as_uint(v[8 * q + 1]), __float_as_uint(v[8 * q + 2]),
                              __float_as_uint(v[8 * q + 3])},
                        rp, o, 0, kDeviceScope);
                    __builtin_amdgcn_raw_buffer_store_b128(
                        u32x4{__float_as_uint(v[8 * q + 4]), __float_as_uint(v[8 * q + 5]), __float_as_uint(v[8 * q + 6]),
                              __float_as_uint(v[8 * q + 7])},
                        rp, o + 16u, 0, kDeviceScope);
                }
        }
    }
    __builtin_amdgcn_s_waitcnt(0);  // vmcnt(0): this thread's partial sums have been written
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __syncthreads();  // ... and so have those of the whole workgroup
    if (threadIdx.x == 0) {
        const int ticket = __hip_atomic_fetch_add(&a.counters[tile_id], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int last = ticket == a.split_k - 1;
        if (last) __hip_atomic_store(&a.counters[tile_id], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // for the next launch
        s_last = last;
    }
    __syncthreads();
    if (!s_last) return false;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    for (int z = 0; z < a.split_k; ++z) {
        const __amdgpu_buffer_rsrc_t rp = make_rsrc(a.partial + (size_t)z * a.M * a.Cout, mn * 4u);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const unsigned m = p.m0 + p.wm0 + i * 32 + p.lrow;
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const unsigned n = p.n0 + p.wn0 + j * 32 + q * 16 + p.lhalf * 8;
                    const unsigned o = (m < (unsigned)a.M && n < (unsigned)a.Cout) ? (m * a.Cout + n) * 4u : kOob;
                    const u32x4 p0 = __builtin_amdgcn_raw_buffer_load_b128(rp, o, 0, kDeviceScope);
                    const u32x4 p1 = __builtin_amdgcn_raw_buffer_load_b128(rp, o + 16u, 0, kDeviceScope);
                    acc[i][j][8 * q + 0] += __uint_as_float(p0.x);
                    acc[i][j][8 * q + 1] += __uint_as_float(p0.y);
                    acc[i][j][8 * q + 2] += __uint_as_float(p0.z);
                    acc[i][j][8 * q + 3] += __uint_as_float(p0.w);
                    acc[i][j][8 * q + 4] += __uint_as_float(p1.x);
                    acc[i][j][8 * q + 5] += __uint_as_float(p1.y);
                    acc[i][j][8 * q + 6] += __uint_as_float(p1.z);
                    acc[i][j][8 * q + 7] += __uint_as_float(p1.w);
                }
        }
    }
    return true;
}

// Bias and residual operands of the epilogue, as 16-byte vectors.  Loading them is separate
// from using them so that a kernel can issue the loads before its last MFMAs.
template <int TM, int TN>
struct EpiOperands {
    u32x4 bv[TN][2][2], rv[TM][TN][2];
};

template <int TM, int TN>
static __device__ __forceinline__ void epilogue_load(EpiOperands<TM, TN> &e, const ConvArgs &a, const EpiPos &p) {
    const unsigned mn = (unsigned)a.M * a.Cout;
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(a.res ? a.res : a.y, mn * 2u);
    // without a bias (the batched form) every bias load is out of range and returns zeros
    const bool has_bias = a.bias != nullptr;
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(has_bias ? static_cast<const void *>(a.bias) : a.y, (unsigned)a.Cout * 4u);
    const bool has_res = a.res != nullptr;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const unsigned n = p.n0 + p.wn0 + j * 32 + q * 16 + p.lhalf * 8;
            const unsigned o = (has_bias && n < (unsigned)a.Cout) ? n * 4u : kOob;
            e.bv[j][q][0] = __builtin_amdgcn_raw_buffer_load_b128(rb, o, 0, 0);
            e.bv[j][q][1] = __builtin_amdgcn_raw_buffer_load_b128(rb, has_bias ? o + 16u : kOob, 0, 0);
        }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const unsigned m = p.m0 + p.wm0 + i * 32 + p.lrow;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const unsigned n = p.n0 + p.wn0 + j * 32 + q * 16 + p.lhalf * 8;
                const unsigned o = (has_res && m < (unsigned)a.M && n < (unsigned)a.Cout) ? (m * a.Cout + n) * 2u : kOob;
                e.rv[i][j][q] = __builtin_amdgcn_raw_buffer_load_b128(rr, o, 0, 0);  // zeros without a residual
            }
    }
}

// Values through the activation and one rounding.  The choice is one branch of the wave around all N: both activations and a choice
// for every value are 8 instructions each.
template <typename T, int N, typename V>
static __device__ __forceinline__ V activate_as(const float (&v)[N], int act) {
    static_assert(sizeof(V) == N * sizeof(T), "");
    T o[N];
    if (act == ACT_HSWISH) {
#pragma unroll
        for (int e = 0; e < N; ++e) o[e] = (T)(v[e] * fminf(fmaxf(v[e] + 3.f, 0.f), 6.f) * (1.f / 6.f));
    } else if (act == ACT_RELU) {
#pragma unroll
        for (int e = 0; e < N; ++e) o[e] = (T)fmaxf(v[e], 0.f);
    } else {
#pragma unroll
        for (int e = 0; e < N; ++e) o[e] = (T)v[e];
    }
    return *reinterpret_cast<const V *>(o);
}
template <typename T> static __device__ __forceinline__ u32x4 activate(const float (&v)[8], int act) { return activate_as<T, 8, u32x4>(v, act); }
template <typename T> static __device__ __forceinline__ u32x2 activate(const float (&v)[4], int act) { return activate_as<T, 4, u32x2>(v, act); }

// + bias, + residual, activation, one round-to-nearest-even to the storage type, 16-byte stores.
// The activation code is uniform, so the hard-swish arithmetic sits behind a scalar branch and the
// ReLU / identity form runs the instructions it always ran.
template <typename T, int TM, int TN, bool HSWISH>
static __device__ __forceinline__ void epilogue_store_act(const f32x16 (&acc)[TM][TN], const EpiOperands<TM, TN> &e, const ConvArgs &a,
                                                          const EpiPos &p) {
    // y may be a channel range of a wider tensor: ldy elements from one pixel to the next
    const unsigned ldy = (unsigned)conv_ldy(a);
    const __amdgpu_buffer_rsrc_t ry = make_rsrc(a.y, (((unsigned)a.M - 1u) * ldy + (unsigned)a.Cout) * 2u);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const unsigned m = p.m0 + p.wm0 + i * 32 + p.lrow;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const unsigned n = p.n0 + p.wn0 + j * 32 + q * 16 + p.lhalf * 8;
                const unsigned o = (m < (unsigned)a.M && n < (unsigned)a.Cout) ? (m * ldy + n) * 2u : kOob;
                const T *r = reinterpret_cast<const T *>(&e.rv[i][j][q]);
                const float *b = reinterpret_cast<const float *>(&e.bv[j][q][0]);
                T out[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const float v = acc[i][j][8 * q + k] + b[k] + (float)r[k];
                    if (HSWISH) out[k] = (T)(v * fminf(fmaxf(v + 3.f, 0.f), 6.f) * (1.f / 6.f));
                    else out[k] = (T)(a.relu ? fmaxf(v, 0.f) : v);
                }
                __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4 *>(out), ry, o, 0, 0);
            }
    }
}

template <typename T, int TM, int TN>
static __device__ __forceinline__ void epilogue_store(const f32x16 (&acc)[TM][TN], const EpiOperands<TM, TN> &e, const ConvArgs &a,
                                                      const EpiPos &p) {
    if (a.relu == ACT_HSWISH) epilogue_store_act<T, TM, TN, true>(acc, e, a, p);
    else epilogue_store_act<T, TM, TN, false>(acc, e, a, p);
}

// ---- epilogue of a tile whose K was split over groups of waves ---------------------------------
// The groups' accumulators meet in LDS in units of four registers: a unit is four consecutive channels of the
// lane's pixel, 64 lanes = 1 KiB, so every access is 16 bytes a lane and runs of lanes are consecutive.  Every wave
// writes all its units, and after one barrier group g adds up units g*UPG .. g*UPG+UPG-1 of the tile (over the groups
// in group order: the sum is the one a single finishing group would make) and carries them through bias, residual,
// activation and store.  With one finishing group its waves read KG-1 times 16 single registers and convert and
// store 16 values, 0.64 us from the last matrix instruction to the last store of a 32x32 tile in four groups, a quarter
// of a 1x1 launch at batch 1.  EXEC of ResNet-50 batch 1 253.3 -> 244.8 us, 193x161 batch 3 272.1 -> 265.8, MobileNet batch 1
// 135.7 -> 131.2.
template <int MT, int TM, int TN, int KG>
struct GroupUnits {
    static constexpr int PER_TILE = MT == 32 ? 4 : 1;
    static constexpr int UNITS = TM * TN * PER_TILE;           // per wave
    static constexpr int UPG = (UNITS + KG - 1) / KG;          // finished by each group; groups beyond UNITS / UPG have none
    static constexpr int W = MT == 32 && UPG % 2 == 0 ? 2 : 1;   // units per load and store: two make eight consecutive channels
};

// Pixel and first channel of unit u (see EpiPos for the accumulator layout).  In a 16x16 tile the lane's four
// accumulators are weight rows 4*(lane/16) .. +3, which the packed order makes channels 8*h + 4*g .. +3 for lane/16 = 2g + h.
template <int MT, int TN>
static __device__ __forceinline__ void unit_pos(const EpiPos &p, int u, unsigned *m, unsigned *n) {
    constexpr int PT = MT == 32 ? 4 : 1;
    const int t = u / PT, r = u - t * PT, i = t / TN, j = t - i * TN;
    *m = p.m0 + p.wm0 + i * MT + p.lrow;
    *n = p.n0 + p.wn0 + j * MT + (MT == 32 ? 16 * (r >> 1) + 8 * p.lhalf + 4 * (r & 1) : 8 * (p.lhalf & 1) + 4 * (p.lhalf >> 1));
}

template <int MT, int TM, int TN, int KG>
struct GroupOperands {
    typedef GroupUnits<MT, TM, TN, KG> G;
    u32x4 bv[G::UPG];
    u32x2 rv[G::UPG];
};

template <int MT, int TM, int TN, int KG>
static __device__ __forceinline__ void group_epilogue_load(GroupOperands<MT, TM, TN, KG> &e, const ConvArgs &a, const EpiPos &p, int kg) {
    typedef GroupUnits<MT, TM, TN, KG> G;
    const bool has_bias = a.bias != nullptr, has_res = a.res != nullptr;
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(has_res ? a.res : a.y, (unsigned)a.M * a.Cout * 2u);
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(has_bias ? static_cast<const void *>(a.bias) : a.y, (unsigned)a.Cout * 4u);
#pragma unroll
    for (int k = 0; k < G::UPG; k += G::W) {
        unsigned m, n;
        unit_pos<MT, TN>(p, kg * G::UPG + k, &m, &n);
        const bool n_ok = kg * G::UPG + k < G::UNITS && n < (unsigned)a.Cout;   // Cout % 32 == 0: all of a unit or none
        const unsigned ob = has_bias && n_ok ? n * 4u : kOob;
        const unsigned orr = has_res && n_ok && m < (unsigned)a.M ? (m * a.Cout + n) * 2u : kOob;
        if constexpr (G::W == 2) {
            e.bv[k] = __builtin_amdgcn_raw_buffer_load_b128(rb, ob, 0, 0);
            e.bv[k + 1] = __builtin_amdgcn_raw_buffer_load_b128(rb, has_bias ? ob + 16u : kOob, 0, 0);
            const u32x4 r = __builtin_amdgcn_raw_buffer_load_b128(rr, orr, 0, 0);
            e.rv[k] = u32x2{r.x, r.y};
            e.rv[k + 1] = u32x2{r.z, r.w};
        } else {
            e.bv[k] = __builtin_amdgcn_raw_buffer_load_b128(rb, ob, 0, 0);
            e.rv[k] = __builtin_amdgcn_raw_buffer_load_b64(rr, orr, 0, 0);
        }
    }
}

// xch: KG * WAVES * UNITS KiB of LDS that no wave reads any more; wq = the wave's place in its group.
template <int MT, int TM, int TN, int KG, int WAVES, typename ACC>
static __device__ __forceinline__ void group_exchange_write(const ACC (&acc)[TM][TN], float *xch, int kg, int wq, int lane) {
    typedef GroupUnits<MT, TM, TN, KG> G;
    float *dst = xch + (kg * WAVES + wq) * (G::UNITS * 256) + lane * 4;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < G::PER_TILE; ++r)
                *reinterpret_cast<float4 *>(dst + ((i * TN + j) * G::PER_TILE + r) * 256) =
                    make_float4(acc[i][j][4 * r], acc[i][j][4 * r + 1], acc[i][j][4 * r + 2], acc[i][j][4 * r + 3]);
}

// This group's units, added up over the groups in group order.
template <int MT, int TM, int TN, int KG, int WAVES>
static __device__ __forceinline__ void group_sum(const float *xch, float4 (&s)[GroupUnits<MT, TM, TN, KG>::UPG], int kg, int wq, int lane) {
    typedef GroupUnits<MT, TM, TN, KG> G;
    float4 v[G::UPG][KG];
#pragma unroll
    for (int k = 0; k < G::UPG; ++k)
#pragma unroll
        for (int g = 0; g < KG; ++g)
            v[k][g] = *reinterpret_cast<const float4 *>(xch + ((g * WAVES + wq) * G::UNITS + min(kg * G::UPG + k, G::UNITS - 1)) * 256 + lane * 4);
#pragma unroll
    for (int k = 0; k < G::UPG; ++k) {
        s[k] = v[k][0];
#pragma unroll
        for (int g = 1; g < KG; ++g) { s[k].x += v[k][g].x; s[k].y += v[k][g].y; s[k].z += v[k][g].z; s[k].w += v[k][g].w; }
    }
}

// splitk_exchange for units: every wave's partial sums go out device-scope, the wave that draws its place's last ticket
// adds those of all splits in split order.  false: another workgroup's wave finishes the units.  `counter` is the arrival
// counter of this place: conv_counters_per_tile of them a tile.
template <int MT, int TM, int TN, int KG>
static __device__ __forceinline__ bool group_splitk(const ConvArgs &a, const EpiPos &p, float4 (&s)[GroupUnits<MT, TM, TN, KG>::UPG], int kg, int lane, int32_t *counter) {
    typedef GroupUnits<MT, TM, TN, KG> G;
    constexpr int kDeviceScope = 16;  // cache-policy operand: sc1
    const unsigned mn = (unsigned)a.M * a.Cout;
    unsigned o[G::UPG];
#pragma unroll
    for (int k = 0; k < G::UPG; ++k) {
        unsigned m, n;
        unit_pos<MT, TN>(p, kg * G::UPG + k, &m, &n);
        o[k] = kg * G::UPG + k < G::UNITS && m < (unsigned)a.M && n < (unsigned)a.Cout ? (m * a.Cout + n) * 4u : kOob;
    }
    const __amdgpu_buffer_rsrc_t rp = make_rsrc(a.partial + (size_t)blockIdx.y * mn, mn * 4u);
#pragma unroll
    for (int k = 0; k < G::UPG; ++k)
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{__float_as_uint(s[k].x), __float_as_uint(s[k].y), __float_as_uint(s[k].z), __float_as_uint(s[k].w)}, rp, o[k], 0, kDeviceScope);
    // Each wave draws tickets of its own, for the units it holds: no barrier, and waves without units are long gone.
    __builtin_amdgcn_s_waitcnt(0);  // vmcnt(0): the wave's partial sums have been written
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    int last = 0;
    if (lane == 0) {
        const int ticket = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = ticket == a.split_k - 1;
        if (last) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // for the next launch
    }
    if (!__builtin_amdgcn_readfirstlane(last)) return false;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // Four splits' sums are requested together; this workgroup's own are the registers that it stored.
    float4 own[G::UPG];
#pragma unroll
    for (int k = 0; k < G::UPG; ++k) { own[k] = s[k]; s[k] = make_float4(0.f, 0.f, 0.f, 0.f); }
    for (int z0 = 0; z0 < a.split_k; z0 += 4) {
        u32x4 v[4][G::UPG];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int z = min(z0 + u, a.split_k - 1);
            const __amdgpu_buffer_rsrc_t rz = make_rsrc(a.partial + (size_t)z * mn, mn * 4u);
#pragma unroll
            for (int k = 0; k < G::UPG; ++k) v[u][k] = __builtin_amdgcn_raw_buffer_load_b128(rz, z0 + u < a.split_k && z != (int)blockIdx.y ? o[k] : kOob, 0, kDeviceScope);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < G::UPG; ++k) {   // past the last split: zeros
                const bool mine = z0 + u == (int)blockIdx.y;
                s[k].x += mine ? own[k].x : __uint_as_float(v[u][k].x);
                s[k].y += mine ? own[k].y : __uint_as_float(v[u][k].y);
                s[k].z += mine ? own[k].z : __uint_as_float(v[u][k].z);
                s[k].w += mine ? own[k].w : __uint_as_float(v[u][k].w);
            }
    }
    return true;
}

template <typename T, int MT, int TM, int TN, int KG, bool HSWISH>
static __device__ __forceinline__ void group_epilogue_store_act(const float4 (&s)[GroupUnits<MT, TM, TN, KG>::UPG], const GroupOperands<MT, TM, TN, KG> &e,
                                                                const ConvArgs &a, const EpiPos &p, int kg) {
    typedef GroupUnits<MT, TM, TN, KG> G;
    const unsigned ldy = (unsigned)conv_ldy(a);
    const __amdgpu_buffer_rsrc_t ry = make_rsrc(a.y, (((unsigned)a.M - 1u) * ldy + (unsigned)a.Cout) * 2u);
#pragma unroll
    for (int k = 0; k < G::UPG; k += G::W) {
        unsigned m, n;
        unit_pos<MT, TN>(p, kg * G::UPG + k, &m, &n);
        T out[4 * G::W];
#pragma unroll
        for (int w = 0; w < G::W; ++w) {
            const float *b = reinterpret_cast<const float *>(&e.bv[k + w]);
            const T *r = reinterpret_cast<const T *>(&e.rv[k + w]);
            const float f[4] = {s[k + w].x, s[k + w].y, s[k + w].z, s[k + w].w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float v = f[c] + b[c] + (float)r[c];
                if (HSWISH) out[4 * w + c] = (T)(v * fminf(fmaxf(v + 3.f, 0.f), 6.f) * (1.f / 6.f));
                else out[4 * w + c] = (T)(a.relu ? fmaxf(v, 0.f) : v);
            }
        }
        const unsigned o = kg * G::UPG + k < G::UNITS && m < (unsigned)a.M && n < (unsigned)a.Cout ? (m * ldy + n) * 2u : kOob;
        if constexpr (G::W == 2) __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4 *>(out), ry, o, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b64(*reinterpret_cast<const u32x2 *>(out), ry, o, 0, 0);
    }
}

template <typename T, int MT, int TM, int TN, int KG>
static __device__ __forceinline__ void group_epilogue_store(const float4 (&s)[GroupUnits<MT, TM, TN, KG>::UPG], const GroupOperands<MT, TM, TN, KG> &e,
                                                            const ConvArgs &a, const EpiPos &p, int kg) {
    if (a.relu == ACT_HSWISH) group_epilogue_store_act<T, MT, TM, TN, KG, true>(s, e, a, p, kg);
    else group_epilogue_store_act<T, MT, TM, TN, KG, false>(s, e, a, p, kg);
}

// Workgroups go to the 8 XCDs round-robin; give each XCD a contiguous run of tiles so that
// tiles sharing pixels (same tile_m) meet in one XCD's L2.
static __device__ __forceinline__ int xcd_tile_id(int bid, int nb) {
    const int xcd = bid & 7, idx = bid >> 3;
    const int per = nb >> 3, rem = nb & 7;
    return xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
}
static __device__ __forceinline__ int xcd_tile_id() { return xcd_tile_id(blockIdx.x, gridDim.x); }

}  // namespace cw
