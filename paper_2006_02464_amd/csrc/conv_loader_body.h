// The direct-to-LDS convolution with waves that only load: the per-tile body of those per-layer launches (conv_dlds_launch.h) and
// pair launches (kernels_conv_dlds.hip) that conv_loads_apart (conv_common.h) gives them to.
//
// Same GEMM view, weight layout, LDS stages and swizzle, MFMA roles, K order and epilogues as conv_dlds_body.h, and the same sums
// bit for bit (of a hard swish's results the compiler may round a product to fp16 in one instruction here and in two there).  What differs
// is who does what.  A wave issues its instructions in order, and one that both multiplies and loads pays for each in turn: per 16-k step
// of a 64x64 tile on four waves 32 clocks of matrix core, about 13 for each operand read and 35-40 for a load to LDS, whose issue
// waits for the CU's address path (16 clocks a load, shared by the four SIMDs), 890 clocks a slice of 128 where the load path needs 512
// and the matrix cores 256.  Here kLoaderWaves further waves, one a SIMD, issue all of them, and the others only read and multiply:
// - a slice costs what is longer of the two, not the sum;
// - the set-up of the addresses (0.25 us, 0.5 with general addressing) is the loaders' alone; beside it the others request bias
//   and residual, which used to be requested before the last slice;
// - with no loads of their own to count, the multiplying waves read a slice's first operands while they multiply the last ones of
//   the slice before: one barrier a slice, behind its last operand read, says both that the next slice has arrived and that this one's
//   stage may be loaded again.
// Without -> with them.  Single launches, back to back, weights of 24 layers in turn: 3x3 of 256 channels at 14x14 batch 16 10.1 -> 9.0 us (64x64,
// slices of 128), 1x1 1024 -> 256 there 6.1 -> 5.4, 3x3 of 128 channels at 28x28 batch 8 6.7 -> 5.9, 1x1 128 -> 512 there at batch 1
// 3.15 -> 2.81.  Whole EXECs: ResNet-152 batch 16 1162 -> 1121 us, ResNet-18 batch 8 132.5 -> 127.4, ResNet-50 batch 16 402.3 -> 397.6,
// Inception 127x127 batch 5 115.7 -> 107.9.  Inside EXECs, by a kernel trace of ResNet, MobileNet and Inception: general addressing on 64x64 and 128x64 with
// slices of 128 10.4-12.1 -> 9.2-10.6, 1x1 on 64x64 5.37-5.71 -> 5.36-5.61, on 128x128 on eight waves 6.63 -> 6.49, on 128x64 with slices of 128
// 6.19-6.24 -> 6.35-6.39, though whole EXECs are 0.1-0.3 % faster with them there too (ResNet-50 and ResNet-152, batch 16; MobileNet the same).
// Two loaders are as fast for 1x1 and 0.1-0.9 us slower for 3x3, one is slower everywhere; a higher wave priority for them, or operands
// requested behind the first slice, cost 1-2 %.
#pragma once
#include "conv_dlds_body.h"

namespace cw {

// tile / tiles_n by a reciprocal from the host; 0: none (one channel tile, or too many tiles for it to be exact).
inline uint32_t conv_tile_magic(unsigned tiles, unsigned tiles_n) {
    return tiles_n > 1 && (unsigned long long)tiles * tiles_n < (1ull << 32) ? (uint32_t)((1ull << 32) / tiles_n) + 1u : 0u;
}

template <typename V>
static __device__ __forceinline__ V lds_read(unsigned at) {
    return *reinterpret_cast<const __attribute__((address_space(3))) V *>((size_t)at);
}

template <typename T, int BM, int BN, int WARPS_M, int WARPS_N, int BK, int NS, int MODE, int KG>
static __device__ __forceinline__ void conv_loader_body(const ConvArgs &a, const int bid, const int nb_packed, const unsigned magic) {
    constexpr int MT = 32;
    const int nb = conv_nb_tiles(nb_packed), panel = conv_nb_panel(nb_packed);
    static_assert(MODE == MODE_CONV || MODE == MODE_GEMM || MODE == MODE_TAIL, "");
    typedef MfmaTile<T, MT> MF;
    typedef typename MF::acc acc_t;
    typedef typename Mfma<T>::v8 v8;
    static_assert(KG <= 2, "one or two wave groups");
    constexpr bool GEMM = MODE != MODE_CONV;
    constexpr int CW = WARPS_M * WARPS_N * KG, NT = 64 * kLoaderWaves;
    constexpr int WM = BM / WARPS_M, WN = BN / WARPS_N, TM = WM / MT, TN = WN / MT;
    constexpr int CPR = BK / 8, RSTEP = NT / CPR;   // 16-byte chunks per LDS row; rows the loaders fetch together
    static_assert(BM * CPR % NT == 0 && BN * CPR % NT == 0, "tile/threads mismatch");
    constexpr int X_PER = BM * CPR / NT, W_PER = BN * CPR / NT, LOADS = X_PER + W_PER;   // load instructions per loading thread per slice
    constexpr unsigned STAGE = (BM + BN) * BK * 2u;
    static_assert(NS >= 2 && NS <= 4 && (NS - 2) * LOADS < 64, "ring of 2..4 stages");
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)cw_dyn_lds;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int per = nb >> 3, rem = nb & 7, xcd = bid & 7;
    const int tile_id = xcd * per + min(xcd, rem) + (bid >> 3);   // xcd_tile_id without branches
    const int tiles_n = (a.Cout + BN - 1) / BN;
    int tile_m, tile_n;
    if (panel == 0) {   // uniform
        tile_m = magic ? (int)__umulhi((unsigned)tile_id, magic) : tile_div(tile_id, tiles_n);
        tile_n = tile_id - tile_m * tiles_n;
    } else {
        panel_tile<BM, BM>(tile_id, tiles_n, panel, a.M, &tile_m, &tile_n);
    }
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int nsteps = MODE == MODE_TAIL ? (a.K + BK - 1) / BK : a.K / BK;   // at least one
    // Barriers: both kinds of waves meet at (general addressing) 1 behind the rows' arithmetic, 1 + nsteps around the slices and 1 in
    // the wave groups' exchange.
    constexpr bool ROWS_SHARED = MODE == MODE_CONV && X_PER > 1;

    if (wave >= CW) {
        // ---- the loading waves.  Piece j of a slice is LDS position lt + j*NT of the operand's [rows][CPR chunks] stage: row lt/CPR +
        // j*RSTEP, chunk position lt%CPR, holding logical chunk lt%CPR ^ key(row).
        const int lt = tid - CW * 64, lw = wave - CW;
        const unsigned row = (unsigned)lt / CPR, pc = (unsigned)lt % CPR;
        unsigned chunk[2];   // the key is the same for every other step of RSTEP rows
#pragma unroll
        for (int q = 0; q < 2; ++q) chunk[q] = pc ^ (unsigned)swz_key<BK>((int)row + q * RSTEP);
        const unsigned ldx2 = (unsigned)conv_ldx(a) * 2u, k2 = (unsigned)a.K * 2u;
        // Rows past M (1x1) or Cout begin at or past the buffers' ends, where loads return zeros.
        const u32x4 dw = make_desc(a.w, (unsigned)a.Cout * k2);
        unsigned w_off[W_PER];
        const unsigned w_row0 = (unsigned)n0 * k2 + row * k2;
#pragma unroll
        for (int j = 0; j < W_PER; ++j) w_off[j] = w_row0 + (unsigned)(j * RSTEP) * k2 + (chunk[j & 1] << 4);
        const unsigned dst0 = lds_base + (unsigned)lw * 1024u;
        const int k_last = a.K - (nsteps - 1) * BK;   // K elements of the last slice (MODE_TAIL)
        auto beyond = [&](int j) { return MODE == MODE_TAIL && (int)chunk[j & 1] * 8 >= k_last; };   // piece j is not in the last slice
        unsigned kb = 0;   // byte offset of the next slice within a weight row
        bool part = false; // it is the last, part of a slice (MODE_TAIL)
        auto load_w = [&](int j, unsigned stage_at) { load_to_lds(dw, part && beyond(j) ? kOob : w_off[j], kb, stage_at + BM * BK * 2u + j * (NT * 16u)); };
        // with general addressing the first slice's weights need none of the pixel arithmetic
        if constexpr (!GEMM) {
#pragma unroll
            for (int j = 0; j < W_PER; ++j) load_w(j, dst0);
        }
        // The activation buffer is described from the top-left tap's offset before its start, so that centre offset (per thread) + tap and
        // channel offset (uniform) is never negative.  x may be the first Cin channels of a wider tensor.
        const int pad_h = GEMM ? 0 : conv_pad_h(a), pad_w = GEMM ? 0 : conv_pad_w(a);
        const unsigned x_bytes = ((GEMM ? (unsigned)a.M : (unsigned)a.B * a.H * a.W) - 1u) * ldx2 + (unsigned)a.Cin * 2u;
        const unsigned x_shift = GEMM ? 0u : (unsigned)(pad_h * a.W + pad_w) * ldx2;
        const u32x4 dx = make_desc(static_cast<const char *>(a.x) - x_shift, x_bytes + x_shift);
        unsigned x_off[X_PER], x_mask[X_PER];   // byte offset at the filter's centre pixel; the taps inside the image (bit r*kw+s)
        if constexpr (GEMM) {
            const unsigned x_row0 = (unsigned)m0 * ldx2 + row * ldx2;
#pragma unroll
            for (int j = 0; j < X_PER; ++j) x_off[j] = x_row0 + (unsigned)(j * RSTEP) * ldx2 + (chunk[j & 1] << 4);
        } else {
            auto pixel_row = [&](unsigned m) {
                const unsigned t = fast_div(m, a.wo_div), n = fast_div(t, a.ho_div);
                const int iwc = (int)(m - t * (unsigned)a.Wo) * a.stride, ihc = (int)(t - n * (unsigned)a.Ho) * a.stride;
                const unsigned taps = tap_mask(a, pad_h, pad_w, ihc, iwc);
                return u32x2{(unsigned)((n * a.H + ihc) * a.W + iwc) * ldx2, m < (unsigned)a.M ? taps : 0u};
            };
            if constexpr (!ROWS_SHARED) {
                const u32x2 ri = pixel_row((unsigned)m0 + row);
                x_off[0] = ri.x + (chunk[0] << 4);
                x_mask[0] = ri.y;
            } else {
                // once per tile row, by thread `row`, and through LDS to the threads that load the row's chunks
                __shared__ u32x2 s_row[BM];
                static_assert(NT >= BM, "one thread per tile row");
                if (lt < BM) s_row[lt] = pixel_row((unsigned)(m0 + lt));
                wait_lds_and_barrier();
#pragma unroll
                for (int j = 0; j < X_PER; ++j) {
                    const u32x2 ri = s_row[row + j * RSTEP];
                    x_off[j] = ri.x + (chunk[j & 1] << 4);
                    x_mask[j] = ri.y;
                }
            }
        }
        // (r, s, c0) of the next slice: k0 = kt*BK = (r*kw + s)*Cin + c0
        int fr = 0, fs = 0, fc0 = 0;
        unsigned soff = 0, tbit = 1u;
        int kt = 0;   // slices issued
        auto issue = [&](unsigned stage, bool with_w) {
            const unsigned at = dst0 + stage * STAGE;
            if (MODE == MODE_TAIL) part = kt == nsteps - 1;
#pragma unroll
            for (int j = 0; j < X_PER; ++j)
                load_to_lds(dx, (GEMM ? part && beyond(j) : (x_mask[j] & tbit) == 0u) ? kOob : x_off[j], soff, at + j * (NT * 16u));
            if (with_w) {
#pragma unroll
                for (int j = 0; j < W_PER; ++j) load_w(j, at);
            }
            ++kt;
            kb += BK * 2u;
            if constexpr (GEMM) {
                soff = kb;
            } else {
                fc0 += BK;
                if (fc0 == a.Cin) {
                    fc0 = 0;
                    if (++fs == a.kw) { fs = 0; ++fr; }
                }
                soff = ((unsigned)(fr * a.W + fs) * (unsigned)conv_ldx(a) + (unsigned)fc0) * 2u;
                tbit = 1u << (fr * a.kw + fs);
            }
        };
#pragma unroll
        for (int u = 0; u < NS - 1; ++u)
            if (u < nsteps) issue(u, GEMM || u > 0);
        // Slice i has arrived when at most the loads of the slices behind it are outstanding.  Behind barrier i the stage of slice i - 1
        // (no one's for i = 0) is free for slice i + NS - 1.
        unsigned fill = NS - 1;
        int i = 0;
        for (; i + NS - 1 < nsteps; ++i) {
            wait_loads_and_barrier<(NS - 2) * LOADS>();
            issue(fill, true);
            fill = fill + 1 == NS ? 0 : fill + 1;
        }
        if (NS >= 4 && i + 2 < nsteps) { wait_loads_and_barrier<2 * LOADS>(); ++i; }
        if (NS >= 3 && i + 1 < nsteps) { wait_loads_and_barrier<LOADS>(); ++i; }
        wait_loads_and_barrier<0>();
        wait_lds_and_barrier();   // the last slice is read
        if constexpr (KG > 1) wait_lds_and_barrier();
        return;
    }

    // ---- the multiplying waves
    const int kg = wave / (WARPS_M * WARPS_N), wq = wave - kg * (WARPS_M * WARPS_N);
    const int wm0 = (wq / WARPS_N) * WM, wn0 = (wq % WARPS_N) * WN;
    const int lrow = lane & (MT - 1), lhalf = lane / MT;
    const EpiPos pos{m0, n0, wm0, wn0, lrow, lhalf};
    EpiOperands<TM, TN> eo;
    GroupOperands<MT, TM, TN, KG> go;
    if constexpr (KG > 1) group_epilogue_load<MT, TM, TN, KG>(go, a, pos, kg);
    else epilogue_load<TM, TN>(eo, a, pos);
    acc_t acc[TM][TN];  // [pixel tile][channel tile]; MFMA rows = channels, columns = pixels
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < MF::REGS; ++e) acc[i][j][e] = 0.f;
    // A slice is multiplied in two halves.  While the first is, the second's operands are read, and behind the barrier, while the second is,
    // those of the next slice's first half: every read has half a slice of matrix instructions to arrive in.  The order is pinned: left to the
    // compiler a step waited for the reads just issued for a later one, 9.25 against 9.10 us for 3x3 of 256 channels at 14x14 batch 16, 7.88 and
    // 7.65 of 64 at 56x56 batch 8, 1x1 1024 -> 512 at 14x14 batch 16 (slices of 64) 9.8 and 9.4; two wave groups the same either way.
    constexpr int KK = BK / MF::K / KG, HK = KK / 2;   // steps of a slice that are this wave's: kg, kg + KG, ...
    static_assert(KK % 2 == 0, "halves of whole steps");
    // The key is the same for all of a wave's tiles: MT rows are whole periods of it.
    const unsigned xkey = (unsigned)swz_key<BK>(wm0 + lrow), wkey = (unsigned)swz_key<BK>(wn0 + lrow);
    const unsigned xo = lds_base + (unsigned)(wm0 + lrow) * (BK * 2u), wo = lds_base + (unsigned)(BM + wn0 + lrow) * (BK * 2u);
    unsigned xc[KK], wc[KK];
#pragma unroll
    for (int t = 0; t < KK; ++t) {
        const unsigned c = (unsigned)((kg + t * KG) * (MF::K / 8) + lhalf);
        xc[t] = xo + ((c ^ xkey) << 4);
        wc[t] = wo + ((c ^ wkey) << 4);
    }
    v8 fx[KK][TM], fw[KK][TN];
    auto fetch = [&](unsigned stage, int t) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fx[t][i] = lds_read<v8>(xc[t] + stage * STAGE + i * (MT * BK * 2u));
#pragma unroll
        for (int j = 0; j < TN; ++j) fw[t][j] = lds_read<v8>(wc[t] + stage * STAGE + j * (MT * BK * 2u));
    };
    if constexpr (ROWS_SHARED) wait_lds_and_barrier();
    wait_lds_and_barrier();   // the first slice is there
#pragma unroll
    for (int t = 0; t < HK; ++t) {
        fetch(0, t);
        __builtin_amdgcn_sched_barrier(0);   // in this order: the loop's waits count the reads behind a step's
    }
    unsigned stage = 0;
    for (int kt = 0; kt < nsteps; ++kt) {
        const bool more = kt + 1 < nsteps;   // behind the last slice its first half is read again: no branch, whose two sides would wait for all reads
        const unsigned next = !more ? stage : stage + 1 == NS ? 0 : stage + 1;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h == 1) wait_lds_and_barrier();   // the slice's last operands are in registers: its stage is free, the next slice is there
#pragma unroll
            for (int t = 0; t < HK; ++t) {
                // two steps' reads with one step's instructions, so that the half ends with none just issued
#pragma unroll
                for (int u = 2 * t; u < 2 * t + 2 && u < HK; ++u) fetch(h ? next : stage, h ? u : HK + u);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j] = MF::mma(fw[h * HK + t][j], fx[h * HK + t][i], acc[i][j]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        stage = next;
    }
    // Every wave is behind the last slice's barrier: the ring is free.
    if constexpr (KG > 1) {
        static_assert(KG * BM * BN * 4 <= NS * (int)STAGE, "K-group exchange does not fit the ring");
        float *xch = reinterpret_cast<float *>(cw_dyn_lds);
        group_exchange_write<MT, TM, TN, KG, WARPS_M * WARPS_N>(acc, xch, kg, wq, lane);
        wait_lds_and_barrier();
        typedef GroupUnits<MT, TM, TN, KG> G;
        static_assert(G::UNITS % KG == 0, "a share for every group");
        float4 sum[G::UPG];
        group_sum<MT, TM, TN, KG, WARPS_M * WARPS_N>(xch, sum, kg, wq, lane);
        group_epilogue_store<T, MT, TM, TN, KG>(sum, go, a, pos, kg);
    } else {
        epilogue_store<T, TM, TN>(acc, eo, a, pos);
    }
}

}  // namespace cw
