// int8 path (the paper's own precision: int8 weights, activations and zero points, int32 scale; Section 5.1
// footnote, Section 4.2.2) for the per-layer launch mode: dense convolution on the int8 matrix cores with integer
// requantisation, max-pool on codes, exact pooled sums, int64 classifier.  Every step is integer arithmetic with
// one right answer (see include/sushi.h: sushi_load_supernet_int8), so results are compared bit for bit.
//
// Layouts: activations [B][H][W][C] int8, C a multiple of 8 (3 for the network input); weights
// [tap][channel group of 16][filter, padded to 16][16 channels] int8, channels beyond the layer's width zero.
//
// Dense layers run in conv_small.hip, conv_tile.hip and conv_patch.hip.  Zero points: the matrix cores multiply the raw
// codes, sum w * (x - z_x) = sum w * x - z_x * sum w.  Cells outside the image are filled with the code z_x (the real
// value 0), channels beyond the SubNet's width with the code 0, so the correction is z_x times the weight sum
// over the ACTIVE channels and all taps, which the host has as a prefix table per 8 channels.
#include "kernels.h"
#include "device_common.h"

#include <algorithm>

namespace sushi {

// Requantises four accumulators of consecutive filters f .. f+3 of pixel m and stores four codes.
__device__ __forceinline__ void store_codes(const ConvArgs &a, const QuantArgs &q, const int acc[4], int f, long m) {
    if (f >= a.K) return;
    const int lo = a.act == 1 ? q.zy : -128;
    unsigned packed = 0;
    unsigned res = 0;
    if (a.res) res = *reinterpret_cast<const unsigned *>(static_cast<const int8_t *>(a.res) + m * a.K + f);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        long long t = rr64((long long)(acc[i] + q.qbias[f + i]) * (long long)q.qmult[f + i], q.qshift[f + i]);
        if (a.res) t += rr64((long long)((int)(int8_t)(res >> (8 * i)) - q.z_res) * (long long)q.m_res, q.sh_res);
        t += q.zy;
        const int v = (int)(t < lo ? lo : t > 127 ? 127 : t);
        packed |= (unsigned)(v & 0xFF) << (8 * i);
    }
    *reinterpret_cast<unsigned *>(static_cast<int8_t *>(a.y) + m * a.K + f) = packed;  // K is a multiple of 4
}

// Fewer than 8 input channels (the network input): one thread per output pixel, all filters of a group of up to 32;
// the group's weights sit in LDS as int32 [tap * C + channel][32] (every thread reads the same word: a broadcast).
// Bound by the multiply-adds on the vector ALUs: 48 images of 224 x 224 to 32 filters, 3x3/2, 49 us, one image 15.
// (Requesting a patch's 27 codes at once lost at every batch size: 56 and 17 us; the other waves hide the loads' latency.)
__global__ __launch_bounds__(256) void conv_i8_direct_kernel(ConvArgs a, QuantArgs q) {
    __shared__ int wl[49 * 4 * 32];
    const int f0 = blockIdx.y * 32;
    const int nf = min(32, a.K - f0);
    const int taps = a.R * a.R;
    const int8_t *w = static_cast<const int8_t *>(a.w);
    for (int i = threadIdx.x; i < taps * a.C * 32; i += 256) {
        const int f = i & 31, tc = i >> 5;
        const int tap = tc / a.C, ch = tc - tap * a.C;
        wl[i] = f < nf ? (int)w[(((long)tap * a.CG + (ch >> 4)) * a.Kpad + f0 + f) * 16 + (ch & 15)] : 0;
    }
    __syncthreads();
    const long M = (long)a.B * a.P * a.Q;
    const long m = (long)blockIdx.x * 256 + threadIdx.x;
    if (m >= M) return;
    const int qq = (int)(m % a.Q), pp = (int)((m / a.Q) % a.P), n = (int)(m / ((long)a.Q * a.P));
    const int8_t *x = static_cast<const int8_t *>(a.x);
    int acc[32];
#pragma unroll
    for (int f = 0; f < 32; ++f) acc[f] = 0;
    for (int tap = 0; tap < taps; ++tap) {
        const int h = pp * a.stride - a.pad + tap / a.R, v = qq * a.stride - a.pad + tap % a.R;
        if (h < 0 || h >= a.H || v < 0 || v >= a.W) continue;
        const int8_t *xp = x + (((long)n * a.H + h) * a.W + v) * a.C;
        for (int ch = 0; ch < a.C; ++ch) {
            const int xv = (int)xp[ch] - q.zx;
            const int4 *wr = reinterpret_cast<const int4 *>(wl + (tap * a.C + ch) * 32);
#pragma unroll
            for (int g = 0; g < 8; ++g) {
                const int4 wv = wr[g];
                acc[4 * g] += xv * wv.x, acc[4 * g + 1] += xv * wv.y, acc[4 * g + 2] += xv * wv.z, acc[4 * g + 3] += xv * wv.w;
            }
        }
    }
#pragma unroll
    for (int g = 0; g < 8; ++g) {
        const int v[4] = {acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
        store_codes(a, q, v, f0 + 4 * g, m);
    }
}

__global__ __launch_bounds__(256) void maxpool_i8_kernel(PoolArgs a) {
    const int cgs = a.C >> 3;
    const long total = (long)a.B * a.P * a.Q * cgs;
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int cg = (int)(idx % cgs);
    const long m = idx / cgs;
    const int qq = (int)(m % a.Q), pp = (int)((m / a.Q) % a.P), n = (int)(m / ((long)a.Q * a.P));
    const int8_t *x = static_cast<const int8_t *>(a.x);
    int best[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) best[j] = -128;
    for (int r = 0; r < 3; ++r) {
        const int h = pp * 2 - 1 + r;
        if (h < 0 || h >= a.H) continue;
        for (int s = 0; s < 3; ++s) {
            const int v = qq * 2 - 1 + s;
            if (v < 0 || v >= a.W) continue;
            const uint2 q = *reinterpret_cast<const uint2 *>(x + (((long)n * a.H + h) * a.W + v) * a.C + cg * 8);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int c = (int)(int8_t)((j < 4 ? q.x : q.y) >> (8 * (j & 3)));
                best[j] = c > best[j] ? c : best[j];
            }
        }
    }
    uint2 o = make_uint2(0, 0);
#pragma unroll
    for (int j = 0; j < 8; ++j) (j < 4 ? o.x : o.y) |= (unsigned)(best[j] & 0xFF) << (8 * (j & 3));
    *reinterpret_cast<uint2 *>(static_cast<int8_t *>(a.y) + m * a.C + cg * 8) = o;
}

// Exact sums of (code - z_x) over H x W: one thread per (image, group of 8 channels); int32 out.
__global__ __launch_bounds__(256) void gap_i8_kernel(PoolArgs a, QuantArgs q) {
    const int cgs = a.C >> 3;
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long)a.B * cgs) return;
    const int cg = (int)(idx % cgs), n = (int)(idx / cgs);
    const int8_t *x = static_cast<const int8_t *>(a.x) + (long)n * a.H * a.W * a.C + cg * 8;
    int sum[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) sum[j] = 0;
#pragma unroll 8
    for (int p = 0; p < a.H * a.W; ++p) {
        const uint2 v = *reinterpret_cast<const uint2 *>(x + (long)p * a.C);
#pragma unroll
        for (int j = 0; j < 8; ++j) sum[j] += (int)(int8_t)((j < 4 ? v.x : v.y) >> (8 * (j & 3))) - q.zx;
    }
    int *y = static_cast<int *>(a.y) + (long)n * a.C + cg * 8;
#pragma unroll
    for (int j = 0; j < 8; ++j) y[j] = sum[j];
}

// Classifier on the pooled sums: a workgroup serves 64 classes of one image; the image's sums sit in LDS, wave w
// takes the channel cells w, w + 4, ... (eight weight cells requested at a time), and the four partial sums are
// added in LDS (exact: integers).  int64 accumulator, float32 logit.
__global__ __launch_bounds__(256) void fc_i8_kernel(ConvArgs a, QuantArgs q) {
    extern __shared__ int fc_sums[];               // C sums, then 4 x 64 partial sums (two words each)
    const int n = blockIdx.y, kk = threadIdx.x & 63, part = threadIdx.x >> 6;
    const int k = blockIdx.x * 64 + kk;
    const int cpad = (a.C + 15) & ~15;
    const int *sums = static_cast<const int *>(a.x) + (long)n * a.C;
    for (int i = threadIdx.x; i < cpad; i += 256) fc_sums[i] = i < a.C ? sums[i] : 0;
    __syncthreads();
    long long acc = 0;
    if (k < a.K) {
        const uint4 *w = static_cast<const uint4 *>(a.w) + k;
        const int ncell = cpad >> 4;
#pragma unroll 1
        for (int c0 = part; c0 < ncell; c0 += 32) {
            uint4 cell[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) cell[u] = c0 + 4 * u < ncell ? w[(long)(c0 + 4 * u) * a.Kpad] : make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int cb = min(c0 + 4 * u, ncell - 1) * 16;
                const unsigned word[4] = {cell[u].x, cell[u].y, cell[u].z, cell[u].w};
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    acc += (long long)fc_sums[cb + j] * (long long)(int)(int8_t)(word[j >> 2] >> (8 * (j & 3)));
            }
        }
    }
    long long *part_sums = reinterpret_cast<long long *>(fc_sums + cpad);
    part_sums[part * 64 + kk] = acc;
    __syncthreads();
    if (part == 0 && k < a.K) {
        const long long total = part_sums[kk] + part_sums[64 + kk] + part_sums[128 + kk] + part_sums[192 + kk] +
                                (long long)q.pool_hw * (long long)q.qbias[k];
        const double base = (double)__int_as_float(q.qmult[k]);
        static_cast<float *>(a.y)[(long)n * a.K + k] = (float)((double)total * (base / (double)q.pool_hw));
    }
}

// ------------------------------------------------------------------ launchers

static inline unsigned i8_blocks(long total) { return (unsigned)((total + 255) / 256); }

hipError_t launch_conv_i8(const ConvArgs &a, const QuantArgs &q, hipStream_t s, int *kc, long patch_min_pixels) {
    const long M = (long)a.B * a.P * a.Q;
    if ((a.K & 3) || M * a.K >= (1l << 31) - 256 || (long)a.B * a.H * a.W * a.C >= (1l << 31) - 256) return hipErrorInvalidValue;
    if ((long)a.R * a.R * a.CG * a.Kpad * 16 >= (1l << 31) - 256) return hipErrorInvalidValue;
    if (a.C < 8 || (a.C & 7)) {
        if (a.C > 4 || a.R * a.R > 49) return hipErrorInvalidValue;
        *kc = KC_CONV_I8_DIRECT;
        hipLaunchKernelGGL(conv_i8_direct_kernel, dim3(i8_blocks(M), (unsigned)((a.K + 31) / 32)), dim3(256), 0, s, a, q);
        return hipGetLastError();
    }
    const bool chosen = patch_min_pixels != PATCH_AUTO;  // (by the caller: then it decides by itself)
    const bool patch = patch_from(patch_min_pixels, M, (long)a.C * a.R * a.R >= 2048);
    auto picked = [&](hipError_t e, int family) {
        if (e != hipErrorNotSupported) *kc = family;
        return e;
    };
    hipError_t e = chosen && patch ? picked(launch_conv_patch_i8(a, q, s), KC_CONV_PATCH) : hipErrorNotSupported;
    if (e == hipErrorNotSupported) e = picked(launch_conv_ksplit_i8(a, q, s, patch && !chosen), KC_CONV_KSPLIT);
    if (e == hipErrorNotSupported && conv_small_is_faster(a, true)) e = picked(launch_conv_small_i8(a, q, s), KC_CONV_SMALL);
    if (e == hipErrorNotSupported) e = picked(launch_conv_tile_i8(a, q, s, patch && !chosen), KC_CONV_TILE);
    if (e == hipErrorNotSupported && patch && !chosen) e = picked(launch_conv_patch_i8(a, q, s), KC_CONV_PATCH);
    if (e == hipErrorNotSupported) e = picked(launch_conv_small_i8(a, q, s), KC_CONV_SMALL);
    return e;
}

hipError_t launch_fc_i8(const ConvArgs &a, const QuantArgs &q, hipStream_t s) {
    if (a.H * a.W != 1 || q.pool_hw < 1) return hipErrorInvalidValue;
    const size_t lds = (size_t)((a.C + 15) & ~15) * 4 + 4 * 64 * 8;
    if (lds > 60 * 1024) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fc_i8_kernel, dim3((unsigned)((a.K + 63) / 64), (unsigned)a.B), dim3(256), lds, s, a, q);
    return hipGetLastError();
}

hipError_t launch_maxpool_i8(const PoolArgs &a, hipStream_t s) {
    if (a.C & 7) return hipErrorInvalidValue;
    hipLaunchKernelGGL(maxpool_i8_kernel, dim3(i8_blocks((long)a.B * a.P * a.Q * (a.C >> 3))), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_gap_i8(const PoolArgs &a, const QuantArgs &q, hipStream_t s) {
    if (a.C & 7) return hipErrorInvalidValue;
    hipLaunchKernelGGL(gap_i8_kernel, dim3(i8_blocks((long)a.B * (a.C >> 3))), dim3(256), 0, s, a, q);
    return hipGetLastError();
}

}  // namespace sushi
