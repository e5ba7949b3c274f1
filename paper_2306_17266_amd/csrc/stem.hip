// The input layer in bf16: 3x3 convolution of a 3-channel image [B][H][W][3] on the matrix cores.
//
// The 27 values of a pixel's patch are ONE reduction step of v_mfma_f32_16x16x32_bf16 (filters are the rows, 16 output
// pixels the columns).  In channels-last order a patch row is nine consecutive elements of memory, so lane (pixel, kg)
// with kg < 3 takes elements 0 .. 7 of patch row kg and the lanes of kg = 3 take element 8 of all three rows; the
// weight fragment is built in the same order once per wave.  Elements are 2 bytes and a patch row may start on an odd
// one: a lane loads the aligned words around its elements (buffer loads: beyond the tensor they return zeros) and
// shifts them into place; elements outside the image are masked out.
//
// Bound by memory (with stride 2 the output map of 24 filters is twice the input).  One thread per pixel and four filters
// on the vector ALUs (conv_direct_kernel, which keeps every other channel count) took 234 us for 61 images of 224 x 224 to 24
// filters and 151 us for 64 images to 16: every thread read its patch element by element.  Here: 24 us (55 MB, 2.3 TB/s)
// and 21 us (45 MB, 2.2 TB/s).
#include "kernels.h"
#include "device_common.h"

namespace sushi {

constexpr int STEM_OOB = 0x7FFFFFF0;

// FT filter tiles of 16 per workgroup, PT pixel tiles of 16 per wave (all their loads are in flight together).
template <int FT, int PT>
__global__ __launch_bounds__(256) void stem_mfma_kernel(ConvArgs a, int tiles_m) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l16 = lane & 15, kg = lane >> 4;
    const int M = a.B * a.P * a.Q;
    const int f0 = (int)(blockIdx.x / tiles_m) * FT * 16;
    const int m0 = ((int)(blockIdx.x % tiles_m) * 4 + wave) * PT * 16;
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.x), 0, (int)((long)a.B * a.H * a.W * 6), 0x00020000);
    const uint16_t *w = static_cast<const uint16_t *>(a.w);

    // the words around this lane's elements; `odd` has one bit per word group that starts on an odd element
    unsigned xw[PT][5];
    int odd[PT];
    bool left[PT], right[PT];
    int rows[PT];  // bit r: patch row r lies inside the image
#pragma unroll
    for (int t = 0; t < PT; ++t) {
        const int m = min(m0 + t * 16 + l16, M - 1);
        const int q = m % a.Q, pn = m / a.Q, p = pn % a.P, n = pn / a.P;
        const int h0 = p * a.stride - 1, w0 = q * a.stride - 1;
        left[t] = w0 >= 0, right[t] = w0 + 2 < a.W;
        rows[t] = 0;
        odd[t] = 0;
#pragma unroll
        for (int r = 0; r < 3; ++r) rows[t] |= (h0 + r >= 0 && h0 + r < a.H) ? 1 << r : 0;
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            const int r = kg < 3 ? kg : j;
            const int e = ((n * a.H + h0 + r) * a.W + w0) * 3 + (kg < 3 ? 0 : 8);  // first element of the group
            const bool live = r < 3 && (rows[t] >> r & 1);
            odd[t] |= (e & 1) << j;
            xw[t][j] = __builtin_amdgcn_raw_buffer_load_b32(rx, live ? ((e >> 1) + (kg < 3 ? j : 0)) * 4 : STEM_OOB, 0, 0);
        }
    }
    Frag fa[FT];
    float sc[FT][4], sh[FT][4];
#pragma unroll
    for (int i = 0; i < FT; ++i) {
        const int f = min(f0 + i * 16 + l16, a.Kpad - 1);
        uint2 c[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) c[j] = *reinterpret_cast<const uint2 *>(w + ((long)(kg < 3 ? kg * 3 + j : j * 3 + 2) * a.Kpad + f) * 8);
        fa[i].u = kg < 3 ? make_uint4(c[0].x, (c[0].y & 0xFFFFu) | c[1].x << 16, c[1].x >> 16 | c[1].y << 16, c[2].x)
                         : make_uint4((c[0].y & 0xFFFFu) | c[1].y << 16, c[2].y & 0xFFFFu, 0u, 0u);
        const int fs = min(f0 + i * 16 + kg * 4, a.K - 4);
        const float4 s4 = a.scale ? *reinterpret_cast<const float4 *>(a.scale + fs) : make_float4(1.f, 1.f, 1.f, 1.f);
        const float4 h4 = *reinterpret_cast<const float4 *>(a.shift + fs);
        sc[i][0] = s4.x, sc[i][1] = s4.y, sc[i][2] = s4.z, sc[i][3] = s4.w;
        sh[i][0] = h4.x, sh[i][1] = h4.y, sh[i][2] = h4.z, sh[i][3] = h4.w;
    }
#pragma unroll
    for (int t = 0; t < PT; ++t) {
        unsigned g[4];
        if (kg < 3) {
#pragma unroll
            for (int j = 0; j < 4; ++j) g[j] = odd[t] & 1 ? xw[t][j] >> 16 | xw[t][j + 1] << 16 : xw[t][j];
            if (!left[t]) g[0] = 0u, g[1] &= 0xFFFF0000u;  // elements 0 .. 2: the column left of the image
            if (!right[t]) g[3] = 0u;                      // elements 6, 7: the column right of it
        } else {
            unsigned e[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) e[j] = right[t] ? (odd[t] >> j & 1 ? xw[t][j] >> 16 : xw[t][j] & 0xFFFFu) : 0u;
            g[0] = e[0] | e[1] << 16, g[1] = e[2], g[2] = 0u, g[3] = 0u;
        }
        Frag fb;
        fb.u = make_uint4(g[0], g[1], g[2], g[3]);
        const int m = m0 + t * 16 + l16;
#pragma unroll
        for (int i = 0; i < FT; ++i) {
            const f32x4_t d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i].v, fb.v, f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            const int f = f0 + i * 16 + kg * 4;
            float v[4];
            with_activation(a.act, a.hsigmoid, [&](auto act) {
#pragma unroll
                for (int k = 0; k < 4; ++k) v[k] = activate_as<decltype(act)::value>(d[k] * sc[i][k] + sh[i][k]);
            });
            if (m < M && f < a.K)
                *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(a.y) + (long)m * a.K + f) =
                    make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
        }
    }
}

template <int FT, int PT>
static hipError_t launch_stem_ft(const ConvArgs &a, hipStream_t s) {
    const long M = (long)a.B * a.P * a.Q;
    const int tiles_m = (int)((M + 64 * PT - 1) / (64 * PT)), tiles_f = (a.K + 16 * FT - 1) / (16 * FT);
    hipLaunchKernelGGL((stem_mfma_kernel<FT, PT>), dim3(tiles_m * tiles_f), dim3(256), 0, s, a, tiles_m);
    return hipGetLastError();
}

// Returns hipErrorNotSupported (nothing launched) for shapes the kernel does not cover: word loads need a 4-byte
// aligned image of an even number of elements (a word never straddles the tensor's end), 8-byte stores a multiple of
// four filters.
hipError_t launch_stem(const ConvArgs &a, hipStream_t s) {
    if (a.C != 3 || a.R != 3 || a.Rmax != 3 || a.pad != 1 || a.stride < 1 || a.stride > 2 || a.CG != 1) return hipErrorNotSupported;
    if (a.res || a.out_f32 || a.in_f32 || (a.K & 3) || a.K < 4) return hipErrorNotSupported;
    const long elems = (long)a.B * a.H * a.W * 3, M = (long)a.B * a.P * a.Q;
    if ((elems & 1) || elems * 2 >= (1l << 31) - 4096 || M >= (1l << 31) - 4096) return hipErrorNotSupported;
    if ((reinterpret_cast<uintptr_t>(a.x) & 3) || (reinterpret_cast<uintptr_t>(a.y) & 7)) return hipErrorNotSupported;
    // four pixel tiles per wave once every SIMD of the chip still gets a wave, else one
    const bool wide = M >= 4 * 16 * 2048;
    if (a.K <= 16) return wide ? launch_stem_ft<1, 4>(a, s) : launch_stem_ft<1, 1>(a, s);
    return wide ? launch_stem_ft<2, 4>(a, s) : launch_stem_ft<2, 1>(a, s);
}

}  // namespace sushi
