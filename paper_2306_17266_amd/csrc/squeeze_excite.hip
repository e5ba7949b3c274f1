// The two fully connected layers of a squeeze-excite block as one launch (bf16 mode): pooled map -> FC + ReLU -> FC + hard
// sigmoid -> one float32 multiplier per image and channel, which the 1x1 layer behind the block applies to its operands.
//
// A workgroup computes a chunk of the gates of up to eight images and, for that, ALL of their hidden vectors: the hidden
// layer is computed again in every chunk, because handing it from one workgroup to another costs a launch (3.5 us) and the
// weights come out of the XCD's L2.  The matrix cores multiply 16 filters x 16 columns (16x16x32): a column is the upper or
// the lower bf16 term of one image's float32 vector (x = hi + lo, about 16 bits of the mantissa), so the eight images share
// the weight operands.  The sixteen waves share filter tiles and, where there are fewer tiles, the reduction; partial sums
// meet in LDS in a fixed order.
//
// Bound by latency: the weights of both layers are requested before the pooled values have arrived (neither depends on
// them), and by the L2 bandwidth of one compute unit where the hidden layer is large (960 x 240: 460 KB, 3 us).  672
// x 168 takes 8.4 us for 64 images and 8.5 for one; two launches and the pass over the map for the gating that it replaces took a
// query of one image 366 us instead of 337, one of 64 images 1526 instead of 1441.
#include "kernels.h"
#include "device_common.h"

#include <algorithm>

namespace sushi {

constexpr int SE_WAVES = 16, SE_THREADS = 64 * SE_WAVES, SE_IMAGES = 8;
constexpr int SE_U1 = 8, SE_U2 = 4;  // weight operands in flight per wave

struct SeShare {
    int tiles, parts;  // filter tiles of 16; waves that share a tile's reduction
    int steps;         // reduction steps (32 inputs) in all
    int tile, part;    // this wave's
};

static __device__ __forceinline__ SeShare se_share(int filters, int inputs, int wave) {
    SeShare s;
    s.tiles = (filters + 15) >> 4;
    s.parts = s.tiles >= SE_WAVES ? 1 : SE_WAVES / s.tiles;
    s.steps = (inputs + 31) >> 5;
    s.tile = wave / s.parts;
    s.part = wave - s.tile * s.parts;
    return s;
}

// Weight operand of one step: filter f0 + l16, cell step * 4 + kg; zeros past the end.
static __device__ __forceinline__ u32x4_t se_weights(const __amdgpu_buffer_rsrc_t rw, int Kpad, int filter, int cell, int cells) {
    return __builtin_amdgcn_raw_buffer_load_b128(rw, offset_if((cell < cells) & (filter < Kpad), ((unsigned)cell * (unsigned)Kpad + (unsigned)filter) * 16u), 0, 0);
}

// Partial sums of this wave's tiles to LDS: part[(wave or tile) ...][column][filter of the tile]
template <int U>
static __device__ __forceinline__ void se_multiply(const __amdgpu_buffer_rsrc_t rw, int Kpad, int f0, int cells, const SeShare &s, const uint16_t *vec, int pitch,
                                                   const u32x4_t *first, float *out, int wave, int l16, int kg) {
    for (int t = s.tile; t < s.tiles; t += SE_WAVES) {  // (more than one tile only where parts is 1)
        f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
        for (int k = s.part; k < s.steps; k += s.parts * U) {
            u32x4_t w[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                w[u] = t == s.tile && k == s.part ? first[u] : se_weights(rw, Kpad, f0 + t * 16 + l16, (k + u * s.parts) * 4 + kg, cells);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int step = min(k + u * s.parts, s.steps - 1);  // (past the end: zeros times the last step's inputs)
                const bf16x8_t x = *reinterpret_cast<const bf16x8_t *>(vec + l16 * pitch + step * 32 + kg * 8);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w[u]), x, acc, 0, 0, 0);
            }
        }
        *reinterpret_cast<f32x4_t *>(out + ((t * s.parts + s.part) * 16 + l16) * 20 + kg * 4) = acc;
    }
}

// Sum over the parts and both terms of filter f, image j.
static __device__ __forceinline__ float se_sum(const float *out, const SeShare &s, int f, int j) {
    float v = 0.f;
    for (int p = 0; p < s.parts; ++p) {
        const float *o = out + ((f >> 4) * s.parts + p) * 320 + (f & 15);
        v += o[2 * j * 20] + o[(2 * j + 1) * 20];
    }
    return v;
}

static __device__ __forceinline__ void se_split(float x, uint16_t *vec, int pitch, int j, int k) {
    const unsigned h = f2bf(x);
    vec[2 * j * pitch + k] = (uint16_t)h;
    vec[(2 * j + 1) * pitch + k] = (uint16_t)f2bf(x - bf2f(h));
}

__global__ __launch_bounds__(SE_THREADS) void se_gate_kernel(SeGateArgs a, int chunk, int nimg) {
    extern __shared__ float4 se_lds[];  // vectors [column][input] of both layers (bf16), biases, partial sums
    const int p1 = ((a.C + 31) & ~31) + 8, p2 = ((a.red + 31) & ~31) + 8;  // (pitch of a column, in values)
    uint16_t *const v1 = reinterpret_cast<uint16_t *>(se_lds), *const v2 = v1 + 16 * p1;
    float *const consts = reinterpret_cast<float *>(v2 + 16 * p2), *const out = consts + a.red + chunk;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int chunks = (a.C + chunk - 1) / chunk;
    const int group = blockIdx.x / chunks, c0 = (blockIdx.x - group * chunks) * chunk;
    const int n0 = group * nimg, ni = min(nimg, a.B - n0), nc = min(chunk, a.C - c0);
    const __amdgpu_buffer_rsrc_t r1 = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w1), 0, (a.C >> 3) * a.Kpad1 * 16, 0x00020000);
    const __amdgpu_buffer_rsrc_t r2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w2), 0, (a.red >> 3) * a.Kpad2 * 16, 0x00020000);
    const SeShare s1 = se_share(a.red, a.C, wave), s2 = se_share(nc, a.red, wave);
    u32x4_t w1[SE_U1], w2[SE_U2];
#pragma unroll
    for (int u = 0; u < SE_U1; ++u)
        w1[u] = se_weights(r1, a.Kpad1, s1.tile < s1.tiles ? s1.tile * 16 + l16 : a.Kpad1, (s1.part + u * s1.parts) * 4 + kg, a.C >> 3);
#pragma unroll
    for (int u = 0; u < SE_U2; ++u)
        w2[u] = se_weights(r2, a.Kpad2, s2.tile < s2.tiles ? c0 + s2.tile * 16 + l16 : a.Kpad2, (s2.part + u * s2.parts) * 4 + kg, a.red >> 3);
    __builtin_amdgcn_sched_barrier(0);

    // per: threads per image, the rest of an image's values in strides
    const int per = nimg == 1 ? SE_THREADS : SE_THREADS / SE_IMAGES, j = tid / per, t0 = tid - j * per;
    const float bias1 = tid < a.red ? a.b1[tid] : 0.f, bias2 = tid < nc ? a.b2[c0 + tid] : 0.f;
    const float *src = a.pooled + (long)min(n0 + j, a.B - 1) * a.parts * a.C;
    if (a.parts <= 2) {  // eight channels' loads in flight, or sixteen parts of one
        for (int ch = t0; ch < a.C; ch += 8 * per) {
            float x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = src[min(ch + u * per, a.C - 1)];
            if (a.parts == 2)
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] += src[a.C + min(ch + u * per, a.C - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (ch + u * per < a.C && j < ni) se_split(x[u] * a.inv, v1, p1, j, ch + u * per);
        }
    } else {
        for (int ch = t0; ch < a.C; ch += per) {
            float s = 0.f;
            for (int t = 0; t < a.parts; t += 16) {
                float x[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) x[u] = src[(long)min(t + u, a.parts - 1) * a.C + ch];
#pragma unroll
                for (int u = 0; u < 16; ++u) s += t + u < a.parts ? x[u] : 0.f;
            }
            if (j < ni) se_split(s * a.inv, v1, p1, j, ch);
        }
    }
    // Inputs past the end are zeros.  (Columns of images that are not there hold anything: columns do not meet.)
    if (tid < 16 * 32) {
        const int col = tid >> 5, k = tid & 31;
        if (a.C + k < p1) v1[col * p1 + a.C + k] = 0;
        if (a.red + k < p2) v2[col * p2 + a.red + k] = 0;
    }
    if (tid < a.red) consts[tid] = bias1;
    if (tid < nc) consts[a.red + tid] = bias2;
    __syncthreads();
    se_multiply<SE_U1>(r1, a.Kpad1, 0, a.C >> 3, s1, v1, p1, w1, out, wave, l16, kg);
    __syncthreads();
    if (j < ni)
        for (int f = t0; f < a.red; f += per) se_split(fmaxf(se_sum(out, s1, f, j) + consts[f], 0.f), v2, p2, j, f);
    __syncthreads();
    se_multiply<SE_U2>(r2, a.Kpad2, c0, a.red >> 3, s2, v2, p2, w2, out, wave, l16, kg);
    __syncthreads();
    if (j < ni)
        for (int f = t0; f < nc; f += per) a.gate[(long)(n0 + j) * a.C + c0 + f] = activate(se_sum(out, s2, f, j) + consts[a.red + f], 0, 1);
}

static size_t se_lds_bytes(const SeGateArgs &a, int chunk) {
    const size_t p1 = ((a.C + 31) & ~31) + 8, p2 = ((a.red + 31) & ~31) + 8;
    const size_t t1 = (a.red + 15) / 16, t2 = (chunk + 15) / 16;  // (tiles times parts: at most the tiles, or the waves)
    return 32 * (p1 + p2) + (a.red + chunk) * 4 + std::max({t1, t2, (size_t)SE_WAVES}) * 320 * 4;
}

bool se_gate_covers(const SeGateArgs &a) {
    return a.C >= 8 && (a.C & 7) == 0 && a.red >= 8 && (a.red & 7) == 0 && a.C <= 8192 && a.red <= SE_THREADS && se_lds_bytes(a, 256) <= 64 * 1024;
}

hipError_t launch_se_gate(const SeGateArgs &a, hipStream_t s) {
    if (!se_gate_covers(a)) return hipErrorInvalidValue;
    // Images share a workgroup from the number on that fills the chip with one chunk each; 64 gates per workgroup, more where
    // there are more workgroups than compute units (every chunk computes the hidden vector once more).
    const int nimg = (int)std::max(1l, std::min<long>(SE_IMAGES, (long)a.B * ((a.C + 63) / 64) / 256));
    const long groups = (a.B + nimg - 1) / nimg;
    int chunk = 64;
    while (chunk < 256 && groups * ((a.C + chunk - 1) / chunk) > 256) chunk *= 2;
    const long wgs = groups * ((a.C + chunk - 1) / chunk);
    if (wgs >= (1l << 22)) return hipErrorInvalidValue;  // (fewer than 2^32 threads)
    hipLaunchKernelGGL(se_gate_kernel, dim3((unsigned)wgs), dim3(SE_THREADS), se_lds_bytes(a, chunk), s, a, chunk, nimg);
    return hipGetLastError();
}

}  // namespace sushi
