// LOAD: the canonical weights and biases of a model into the layouts the kernels read.
#include "common.h"

namespace cw {

// A launch packs up to kPackItems tensors, described in its kernel arguments, and their biases.  (One launch per tensor and
// one per bias, as before, took 4 us each: 108 launches and 480 us behind the 930 us of ResNet-50's copy.)
// Bound: HBM (every byte read once, written once).  The tensors are cut into chunks of 256 threads' work and the
// workgroups, at most four per CU, stride over the chunks of all of them: LOAD runs beside EXEC (paper section 5.2), and
// a launch as wide as a large tensor would queue thousands of workgroups behind the EXEC kernels' own.
//
// Row i of every group of 32 output channels of a convolution receives channel sigma(i) of that group,
//     i = 8g + 4h + k  ->  sigma(i) = 16*(g/2) + 8h + 4*(g%2) + k,
// the order in which the conv kernel's MFMA accumulators come out as runs of 8 channels.
__device__ static inline unsigned pack_row(unsigned k, bool permute) {
    if (!permute) return k;
    const unsigned row = k & 31, g = row >> 3, h = (row >> 2) & 1, kk = row & 3;
    return (k & ~31u) + (g >> 1) * 16 + h * 8 + (g & 1) * 4 + kk;
}

constexpr unsigned kUnroll1 = 4;   // 16-byte pieces a thread has in flight in a 1x1 tensor

enum PackMode { PACK_1X1, PACK_3X3, PACK_TAPS, PACK_ANY, PACK_DEPTHWISE };

static unsigned pack_chunks(const PackItem &t) {
    const size_t c8 = (size_t)t.cout * t.cin / 8;
    size_t units = 0;   // of 256
    switch (t.mode) {
        case PACK_1X1: units = (c8 + kUnroll1 - 1) / kUnroll1; break;
        case PACK_3X3: units = c8; break;
        case PACK_TAPS: units = c8 * t.kh * t.kw; break;
        case PACK_ANY: units = (size_t)t.cout * t.khp * t.kwp * t.cinp; break;
        default: units = (size_t)t.cout * t.kh * t.kw; break;
    }
    return (unsigned)((units + 255) / 256);
}

__global__ __launch_bounds__(256) void pack_model_kernel(const PackArgs a) {
    __shared__ uint4 lds[256 * 9];
    const unsigned tid = threadIdx.x;
    int i = 0;
    for (unsigned b = blockIdx.x; b < a.chunks; b += gridDim.x) {
        while (i + 1 < a.n && b >= a.items[i + 1].first_chunk) ++i;
        const PackItem &t = a.items[i];
        const unsigned chunk = b - t.first_chunk;
        const unsigned c8 = (unsigned)t.cin / 8, taps = (unsigned)t.kh * t.kw;
        const unsigned units = (unsigned)t.cout * c8;   // of 8 input channels
        if (chunk == 0)
            for (unsigned j = tid; j < (unsigned)t.cout; j += 256) t.bias_dst[j] = t.bias_src[j];
        switch (t.mode) {
            case PACK_1X1: {   // rows change places
                const uint4 *src = reinterpret_cast<const uint4 *>(t.src);
                uint4 *dst = reinterpret_cast<uint4 *>(t.dst);
                const unsigned first = chunk * kUnroll1 * 256 + tid;
                auto from = [&](unsigned u) {   // the last piece where there is no such one
                    u = u < units ? u : units - 1;
                    const unsigned k = u / c8;
                    return src[(size_t)pack_row(k, t.permute) * c8 + (u - k * c8)];
                };
                const uint4 v0 = from(first), v1 = from(first + 256), v2 = from(first + 512), v3 = from(first + 768);
                if (first < units) dst[first] = v0;
                if (first + 256 < units) dst[first + 256] = v1;
                if (first + 512 < units) dst[first + 512] = v2;
                if (first + 768 < units) dst[first + 768] = v3;
                break;
            }
            case PACK_3X3: {   // 8 channels x 9 taps are 144 contiguous bytes: to LDS in 16-byte pieces, from there transposed
                __syncthreads();
#pragma unroll
                for (unsigned j = 0; j < 9; ++j) {
                    const unsigned p = j * 256 + tid, u = chunk * 256 + p / 9;
                    if (u < units) {
                        const unsigned k = u / c8;
                        lds[p] = reinterpret_cast<const uint4 *>(t.src)[((size_t)pack_row(k, t.permute) * c8 + (u - k * c8)) * 9 + p % 9];
                    }
                }
                __syncthreads();
                const unsigned u = chunk * 256 + tid;
                if (u < units) {
                    uint4 in[9];
#pragma unroll
                    for (int j = 0; j < 9; ++j) in[j] = lds[tid * 9 + j];
                    const uint32_t *w = reinterpret_cast<const uint32_t *>(in);
                    const unsigned k = u / c8, c = u - k * c8;
#pragma unroll
                    for (int tap = 0; tap < 9; ++tap) {
                        uint32_t o[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int e0 = (2 * q) * 9 + tap, e1 = (2 * q + 1) * 9 + tap;
                            const uint32_t lo = (e0 & 1) ? w[e0 / 2] >> 16 : w[e0 / 2] & 0xffffu;
                            const uint32_t hi = (e1 & 1) ? w[e1 / 2] & 0xffff0000u : w[e1 / 2] << 16;
                            o[q] = lo | hi;
                        }
                        reinterpret_cast<uint4 *>(t.dst)[((size_t)k * 9 + tap) * c8 + c] = make_uint4(o[0], o[1], o[2], o[3]);
                    }
                }
                break;
            }
            case PACK_TAPS: {   // any filter: 8 channels of one tap
                const unsigned u = chunk * 256 + tid;
                if (u < units * taps) {
                    const unsigned c = u % c8, kt = u / c8, tap = kt % taps, k = kt / taps;
                    const uint16_t *s = t.src + ((size_t)pack_row(k, t.permute) * t.cin + c * 8) * taps + tap;
                    uint32_t o[4];
#pragma unroll
                    for (unsigned q = 0; q < 4; ++q) o[q] = (uint32_t)s[2 * q * taps] | (uint32_t)s[(2 * q + 1) * taps] << 16;
                    reinterpret_cast<uint4 *>(t.dst)[u] = make_uint4(o[0], o[1], o[2], o[3]);
                }
                break;
            }
            case PACK_ANY: {   // with padded rows, columns and channels (a first convolution)
                const unsigned e = chunk * 256 + tid;
                if (e < (unsigned)t.cout * t.khp * t.kwp * t.cinp) {
                    const unsigned c = e % t.cinp, e1 = e / t.cinp, s = e1 % t.kwp, e2 = e1 / t.kwp, r = e2 % t.khp, k = e2 / t.khp;
                    uint16_t v = 0;
                    if (c < (unsigned)t.cin && s < t.kw && r < t.kh) v = t.src[(((size_t)pack_row(k, t.permute) * t.cin + c) * t.kh + r) * t.kw + s];
                    t.dst[e] = v;
                }
                break;
            }
            default: {   // depthwise: W[C][1][kh][kw] -> [kh][kw][C]
                const unsigned e = chunk * 256 + tid;
                if (e < (unsigned)t.cout * taps) t.dst[e] = t.src[(size_t)(e % (unsigned)t.cout) * taps + e / (unsigned)t.cout];
                break;
            }
        }
    }
}

hipError_t launch_pack_model(PackItem *items, int n, hipStream_t s) {
    for (int at = 0; at < n; at += kPackItems) {
        PackArgs a{};
        a.n = n - at < kPackItems ? n - at : kPackItems;
        unsigned chunks = 0;
        for (int i = 0; i < a.n; ++i) {
            PackItem &t = items[at + i];
            if (t.cout < 1 || t.cin < 1 || t.kh < 1 || t.kw < 1 || (t.permute && t.cout % 32 != 0) || !t.src || !t.dst || !t.bias_src || !t.bias_dst)
                return hipErrorInvalidValue;
            if ((size_t)t.cout * t.khp * t.kwp * t.cinp >= (1ull << 31) || reinterpret_cast<uintptr_t>(t.dst) % 16 != 0) return hipErrorInvalidValue;
            const bool plain = t.khp == t.kh && t.kwp == t.kw && t.cinp == t.cin && t.cin % 8 == 0;
            const bool aligned = reinterpret_cast<uintptr_t>(t.src) % 16 == 0;
            t.mode = t.depthwise ? PACK_DEPTHWISE : !plain ? PACK_ANY : (aligned && t.kh * t.kw == 1) ? PACK_1X1
                   : (aligned && t.kh * t.kw == 9) ? PACK_3X3 : PACK_TAPS;
            t.first_chunk = chunks;
            chunks += pack_chunks(t);
            a.items[i] = t;
        }
        a.chunks = chunks;
        pack_model_kernel<<<dim3(chunks < kLoadGridCap ? chunks : kLoadGridCap), 256, 0, s>>>(a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace cw
