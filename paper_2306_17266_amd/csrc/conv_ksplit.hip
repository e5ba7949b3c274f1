// 3x3 convolution with stride 1 and at least 96 (int8: 120) input channels on the matrix cores, bf16 and int8.  The four waves of a workgroup
// split the REDUCTION, so that every weight operand is loaded by one wave only, from memory straight into registers, the input is
// copied once for all nine taps, and one barrier is passed per nine steps.
//
// A workgroup computes 32 FT filters x 32 PT consecutive output pixels; every wave holds all FT x PT accumulators (32x32x16_bf16,
// 32x32x32_i8).  The input is addressed in a frame around the image (padded coordinates, see conv_patch.hip), so that a tile
// needs one contiguous range of positions.  Channels come in chunks of eight 16-byte cells, double-buffered in LDS as
// [cell][position] planes of odd length; wave w owns cells 2 w, 2 w + 1 of a chunk: nine steps, one per tap.  A step is FT weight
// operands (a ring of three steps in flight, running on across chunks), PT reads from LDS and FT PT matrix instructions.
// The partial tiles are added in LDS, 32 pixels at a time, in the order of the waves, and finished as 16-byte pieces (8 filters).
//
// Bound by the weights' way into a compute unit, 70 clocks a step for each 32 filters (four waves' KiB at 60 B per clock), whatever
// the pixels: a ring of nine steps gains nothing.  us, one layer over and over: 16 x 14 x 14 x 360 14.5 with 96 x 64 tiles (64 x
// 64 tiles whose waves share operands through LDS, conv_tile.hip: 25.1); 16 x 7 x 7 x 720 17.9 (24.4), 61 x 14 x 14 x 256 19.5
// (27.6 in the patch kernel), int8 16 x 14 x 14 x 360 12 (16.5).  Inside a query, its weights not in the caches: 16 x 14 x 14 x 360
// 15.7 (25.9), 16 x 7 x 7 x 720 19.0 (24.5).
#include "kernels.h"
#include "device_common.h"

#include <algorithm>
#include <type_traits>

namespace sushi {

typedef __attribute__((ext_vector_type(16))) float ck_f32x16;
typedef __attribute__((ext_vector_type(16))) int ck_i32x16;
typedef __attribute__((ext_vector_type(4))) int ck_i32x4;
typedef __attribute__((ext_vector_type(2))) unsigned ck_u32x2;

struct KsplitGeom {
    int tiles_f, tiles_m;
    int M;           // B * P * Q
    int hp, wp;      // frame: H + 2 and W + 2
    int ps;          // positions of a plane (odd)
    int nchunks;     // chunks of channels
    int part;        // cell offset of the scale / shift (int8: multiplier, shift, bias) copies in LDS
    FastDiv dq, dp, dwp, dhp;  // division by Q, P, wp, hp
};

constexpr int KSPLIT_LOADS = 7;                    // cells of a chunk that a thread copies
constexpr int KSPLIT_POSITIONS = KSPLIT_LOADS * 32;  // that a tile may need

template <bool I8, int FT, int PT>
__global__ __launch_bounds__(256, 2) void conv_ksplit_kernel(ConvArgs a, KsplitGeom g, QuantArgs q) {
    constexpr int ES = I8 ? 1 : 2, CPC = 16 / ES;  // bytes per element, channels per cell
    constexpr int BN = 32 * FT, BM = 32 * PT, CC = 8, NLD = KSPLIT_LOADS, STEPS = 9, D = 3;
    constexpr int PROW = BN / 4 + 1;               // 16-byte cells per pixel row of a partial tile
    extern __shared__ uint4 ck_lds[];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, kh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntiles = g.tiles_f * g.tiles_m, per_xcd = (ntiles + 7) >> 3;
    const int tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (tile >= ntiles) return;
    const int tf = tile / g.tiles_m, tm = tile - tf * g.tiles_m;
    const int f0 = tf * BN, m0 = tm * BM, cells = (a.C + CPC - 1) / CPC;
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.x), 0, (int)((long)a.B * a.H * a.W * a.C * ES), 0x00020000);
    const __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w), 0, (int)(9l * a.CG * a.Kpad * 16), 0x00020000);
    auto frame = [&](int m) {  // position of output pixel m's first tap
        const int t = fdiv(m, g.dq), qq = m - t * a.Q, n = fdiv(t, g.dp), p = t - n * a.P;
        return (n * g.hp + p) * g.wp + qq;
    };
    const int u0 = frame(m0);

    // ---- weights: lane (filter l32, cell kh of a pair), steps of this wave in order
    const unsigned wlane = ((unsigned)kh * (unsigned)a.Kpad + (unsigned)(f0 + l32)) * 16u;
    u32x4_t wr[D][FT];
    auto load_weights = [&](int chunk, int t, u32x4_t *dst) {
        const int cell = chunk * CC + 2 * wave;
        const unsigned off = (unsigned)(t * a.CG + cell) * (unsigned)a.Kpad * 16u;
        const unsigned o = (unsigned)offset_if(cell + kh < cells, wlane + off);
#pragma unroll
        for (int f = 0; f < FT; ++f) dst[f] = __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(o + f * 512u), 0, 0);
    };
    // ---- patch: thread copies cell tid % 8 of positions tid / 8 + 32 e
    const int ccell = tid & 7, cpos = tid >> 3;
    unsigned poff[NLD];
    bool pok[NLD];
#pragma unroll
    for (int e = 0; e < NLD; ++e) {
        const int u = u0 + cpos + 32 * e, t = fdiv(u, g.dwp), n = fdiv(t, g.dhp), h = t - n * g.hp - 1, w = u - t * g.wp - 1;
        pok[e] = cpos + 32 * e < g.ps && n < a.B && (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W;
        poff[e] = (unsigned)(((n * a.H + h) * a.W + w) * a.C * ES);
    }
    u32x4_t pr[NLD];
    auto load_patch = [&](int chunk, int e) {
        const int cell = chunk * CC + ccell;
        pr[e] = __builtin_amdgcn_raw_buffer_load_b128(rx, offset_if(pok[e] & (cell < cells), poff[e] + (unsigned)cell * 16u), 0, 0);
    };
    // int8: a cell of the frame holds the code of the real value 0 (the input's zero point) in its active channels, the
    // upper half of a cell that straddles the SubNet's channel count zeros
    const unsigned zfill = (unsigned)(q.zx & 0xFF) * 0x01010101u;
    auto store_patch = [&](int chunk) {
        uint4 *const dst = ck_lds + (chunk & 1) * CC * g.ps + ccell * g.ps + cpos;
        const int cell = chunk * CC + ccell;
#pragma unroll
        for (int e = 0; e < NLD; ++e) {
            u32x4_t v = pr[e];
            if (I8) {
                if (!pok[e] && cell < cells) v = u32x4_t{zfill, zfill, zfill, zfill};
                if (cell * CPC + 8 >= a.C) v[2] = 0u, v[3] = 0u;
            }
            if (cpos + 32 * e < g.ps) dst[32 * e] = __builtin_bit_cast(uint4, v);
        }
    };
#pragma unroll
    for (int e = 0; e < NLD; ++e) load_patch(0, e);
#pragma unroll
    for (int d = 0; d < D; ++d) load_weights(0, d, wr[d]);
    // the tile's epilogue constants
    {
        auto rsrc = [&](const void *p) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, p ? a.K * 4 : 0, 0x00020000); };
        const void *const src[4] = {I8 ? (const void *)q.qmult : (const void *)a.scale, I8 ? (const void *)q.qshift : (const void *)a.shift, q.qbias, q.wsum};
        uint4 cst[I8 ? 4 : 2];
#pragma unroll
        for (int i = 0; i < (I8 ? 4 : 2); ++i)
            cst[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc(src[i]), offset_if(tid < BN / 4, (unsigned)(f0 + tid * 4) * 4u), 0, 0));
        __builtin_amdgcn_sched_barrier(0);
        if (I8) {  // (the zero-point term goes to the bias: minus z_x times the sum of the active weights)
            cst[1] = make_uint4(max((int)cst[1].x, 1), max((int)cst[1].y, 1), max((int)cst[1].z, 1), max((int)cst[1].w, 1));  // (filters beyond K: any valid shift)
            cst[I8 ? 2 : 0].x -= q.zx * cst[I8 ? 3 : 0].x, cst[I8 ? 2 : 0].y -= q.zx * cst[I8 ? 3 : 0].y, cst[I8 ? 2 : 0].z -= q.zx * cst[I8 ? 3 : 0].z, cst[I8 ? 2 : 0].w -= q.zx * cst[I8 ? 3 : 0].w;
        } else if (!a.scale) {
            cst[0] = make_uint4(0x3F800000u, 0x3F800000u, 0x3F800000u, 0x3F800000u);
        }
        if (tid < BN / 4)
#pragma unroll
            for (int i = 0; i < (I8 ? 3 : 2); ++i) ck_lds[g.part + i * (BN / 4) + tid] = cst[i];
    }
    // ---- where a lane's pixels stand in a plane
    unsigned brow[PT];
#pragma unroll
    for (int p = 0; p < PT; ++p) {
        const int m = min(m0 + p * 32 + l32, g.M - 1);
        brow[p] = (unsigned)(frame(m) - u0 + (2 * wave + kh) * g.ps);
    }
    typedef typename std::conditional<I8, ck_i32x16, ck_f32x16>::type acc_t;
    acc_t acc[FT][PT];
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int p = 0; p < PT; ++p)
#pragma unroll
            for (int k = 0; k < 16; ++k) acc[f][p][k] = 0;
    store_patch(0);
    __syncthreads();
    for (int chunk = 0; chunk < g.nchunks; ++chunk) {
        const unsigned base = (unsigned)((chunk & 1) * CC * g.ps);
        Frag in[2][PT];
        auto read = [&](int t, Frag *dst) {
            const unsigned add = base + (unsigned)((t / 3) * g.wp + t % 3);
#pragma unroll
            for (int p = 0; p < PT; ++p) dst[p].u = ck_lds[brow[p] + add];
        };
        read(0, in[0]);
#pragma unroll
        for (int t = 0; t < STEPS; ++t) {
            if (t + 1 < STEPS) read(t + 1, in[(t + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int f = 0; f < FT; ++f)
#pragma unroll
                for (int p = 0; p < PT; ++p)
                    if constexpr (I8)
                        acc[f][p] = __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(ck_i32x4, wr[t % D][f]), __builtin_bit_cast(ck_i32x4, in[t & 1][p].u),
                                                                          acc[f][p], 0, 0, 0);
                    else
                        acc[f][p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, wr[t % D][f]), in[t & 1][p].v, acc[f][p], 0, 0, 0);
            // (every load is issued on every path, past the end where there is nothing left)
            if (t + D < STEPS)
                load_weights(chunk, t + D, wr[t % D]);
            else
                load_weights(chunk + 1, t + D - STEPS, wr[t % D]);
#pragma unroll
            for (int e = t * NLD / STEPS; e < (t + 1) * NLD / STEPS; ++e) load_patch(chunk + 1, e);
            __builtin_amdgcn_sched_barrier(0);
        }
        store_patch(chunk + 1);
        __syncthreads();
    }

    // ---- the partial tiles meet, 32 pixels at a time: [wave][pixel][filter] (32-bit), over the patches
    constexpr int PIECES = 32 * (BN / 8), EPT = (PIECES + 255) / 256;
    const int obytes = (int)((long)g.M * a.K * ES);
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.res ? a.res : a.y), 0, obytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(a.y, 0, obytes, 0x00020000);
    auto out_offset = [&](int p, int e) {
        const int idx = tid + 256 * e, px = idx / (BN / 8), f = f0 + (idx - px * (BN / 8)) * 8, m = m0 + p * 32 + px;
        return offset_if((idx < PIECES) & (m < g.M) & (f < a.K), (unsigned)(m * a.K + f) * ES);
    };
    u32x4_t res[PT][EPT];
    if (a.res)
#pragma unroll
        for (int p = 0; p < PT; ++p)
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                if (I8) {
                    const ck_u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rr, out_offset(p, e), 0, 0);
                    res[p][e] = u32x4_t{v[0], v[1], 0u, 0u};
                } else {
                    res[p][e] = __builtin_amdgcn_raw_buffer_load_b128(rr, out_offset(p, e), 0, 0);
                }
            }
    uint4 *const part = ck_lds;
    const uint4 *const ss = ck_lds + g.part;
#pragma unroll
    for (int p = 0; p < PT; ++p) {
        if (p > 0) __syncthreads();
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                typedef typename std::conditional<I8, ck_i32x4, f32x4_t>::type v4;
                const v4 v = {acc[f][p][4 * jj], acc[f][p][4 * jj + 1], acc[f][p][4 * jj + 2], acc[f][p][4 * jj + 3]};
                part[(wave * 32 + l32) * PROW + f * 8 + 2 * jj + kh] = __builtin_bit_cast(uint4, v);
            }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int idx = min(tid + 256 * e, PIECES - 1), px = idx / (BN / 8), cc = idx - px * (BN / 8);
            const uint4 *src = part + px * PROW + 2 * cc;
            const int o = out_offset(p, e);
            if constexpr (I8) {
                int v[8] = {};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint4 lo = src[k * 32 * PROW], hi = src[k * 32 * PROW + 1];
                    v[0] += (int)lo.x, v[1] += (int)lo.y, v[2] += (int)lo.z, v[3] += (int)lo.w;
                    v[4] += (int)hi.x, v[5] += (int)hi.y, v[6] += (int)hi.z, v[7] += (int)hi.w;
                }
                const int *mu = reinterpret_cast<const int *>(ss) + cc * 8;
                const int lo = a.act == 1 ? q.zy : -128;
                unsigned packed[2] = {0u, 0u};
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    long long t = rr64((long long)(v[i] + mu[2 * BN + i]) * (long long)mu[i], mu[BN + i]);
                    if (a.res) t += rr64((long long)((int)(int8_t)(res[p][e][i >> 2] >> (8 * (i & 3))) - q.z_res) * (long long)q.m_res, q.sh_res);
                    t += q.zy;
                    const int c = (int)(t < lo ? lo : t > 127 ? 127 : t);
                    packed[i >> 2] |= (unsigned)(c & 0xFF) << (8 * (i & 3));
                }
                __builtin_amdgcn_raw_buffer_store_b64(ck_u32x2{packed[0], packed[1]}, ry, o, 0, 0);
            } else {
                float v[8] = {};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float4 lo = __builtin_bit_cast(float4, src[k * 32 * PROW]), hi = __builtin_bit_cast(float4, src[k * 32 * PROW + 1]);
                    v[0] += lo.x, v[1] += lo.y, v[2] += lo.z, v[3] += lo.w;
                    v[4] += hi.x, v[5] += hi.y, v[6] += hi.z, v[7] += hi.w;
                }
                float sc[8], sh[8];
                load8(reinterpret_cast<const float *>(ss) + cc * 8, sc), load8(reinterpret_cast<const float *>(ss) + BN + cc * 8, sh);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    v[i] = v[i] * sc[i] + sh[i];
                    if (a.res) v[i] += bf2f(i & 1 ? res[p][e][i >> 1] >> 16 : res[p][e][i >> 1] & 0xFFFFu);
                }
                u32x4_t w;
                with_activation(a.act, a.hsigmoid, [&](auto act) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) w[i] = pack_bf16x2(activate_as<decltype(act)::value>(v[2 * i]), activate_as<decltype(act)::value>(v[2 * i + 1]));
                });
                __builtin_amdgcn_raw_buffer_store_b128(w, ry, o, 0, 0);
            }
        }
    }
}

// Positions of the frame that the worst tile of bm consecutive output pixels needs: a tile that runs over as many row ends as
// possible, and over as many image ends.
static long ksplit_positions(const ConvArgs &a, int bm) {
    const long wp = a.W + 2, pq = (long)a.P * a.Q, n = std::min<long>(bm, (long)a.B * pq);
    const long rows = (n - 1 + a.Q - 1) / a.Q, images = std::min<long>((n - 1 + pq - 1) / pq, a.B - 1);
    return n - 1 + 2 * rows + 2 * wp * images + 2 * (wp + 1) + 1;
}

template <int FT, int PT, bool I8>
static hipError_t launch_ksplit_tile(const ConvArgs &a, const QuantArgs &q, hipStream_t s) {
    constexpr int BN = 32 * FT, BM = 32 * PT, CC = 8, CPC = I8 ? 16 : 8;
    KsplitGeom g;
    g.M = a.B * a.P * a.Q;
    g.tiles_f = (a.K + BN - 1) / BN, g.tiles_m = (g.M + BM - 1) / BM;
    g.hp = a.H + 2, g.wp = a.W + 2;
    g.ps = (int)ksplit_positions(a, BM) | 1;
    g.nchunks = ((a.C + CPC - 1) / CPC + CC - 1) / CC;
    g.part = std::max(2 * CC * g.ps, 4 * 32 * (BN / 4 + 1));
    g.dq = make_fastdiv(a.Q), g.dp = make_fastdiv(a.P), g.dwp = make_fastdiv(g.wp), g.dhp = make_fastdiv(g.hp);
    const size_t lds = ((size_t)g.part + 3 * (BN / 4)) * 16;  // (less than 64 KiB)
    const int per_xcd = (int)(((long)g.tiles_m * g.tiles_f + 7) / 8);
    hipLaunchKernelGGL((conv_ksplit_kernel<I8, FT, PT>), dim3(per_xcd * 8), dim3(256), lds, s, a, g, q);
    return hipGetLastError();
}

// From 96 channels on, int8 from 120 (eight cells, a whole chunk): below, the last chunk is half empty or more, and the gain over the
// other kernels goes.  By the rule below over 48 square layers of each width (7 x 7 to 56 x 56, 1 to 96 images, warm), us without
// and with this kernel, and how many layers get slower by 3 % and more: bf16 80 channels 544 / 534, 88 570 / 553, 1 (24 x 28 x 28
// 11.6 / 12.2), 96 577 / 554, 0, 104 737 / 710, 0 (16 x 28 x 28 11.4 / 9.7), 128 799 / 737, 0; int8 96 533 / 528, 1, 104 and 112
// 595 / 591, 5 (12 x 28 x 28 9.2 / 11.1), 120 630 / 614, 1, 128 640 / 620, 1.  Inside queries 28 x 28 x 104 of 2 to 24 images takes
// 79.3 / 69.6 in all, at the extremes 5.9 / 6.4 (2 images) and 17.1 / 12.2 (24).
template <bool I8>
static bool ksplit_covers(const ConvArgs &a) {
    const int es = I8 ? 1 : 2;
    if (a.in_f32 || a.out_f32 || (a.C & 7) || a.C < (I8 ? 120 : 96) || (a.K & 7) || a.K < 8) return false;
    if (a.R != 3 || a.pad != 1 || a.stride != 1 || a.Rmax != 3) return false;
    const long M = (long)a.B * a.P * a.Q, lim = (1l << 31) - 4096;
    return M * a.K * es < lim && (long)a.B * a.H * a.W * a.C * es < lim && 9l * a.CG * a.Kpad * 16 < (1l << 30) &&
           (long)a.B * (a.H + 2) * (a.W + 2) < lim && (M + 31) / 32 * ((a.K + 31) / 32) < (1l << 22);
}

// What a tile shape takes, in us: fits to 132 layers of each type (batch 1 to 61, 7 x 7 to 28 x 28, 104 to 720 channels; 4 to 13 %
// rms), fixed + per step and round of 256 workgroups, a quarter more where there are several rounds.
struct KsplitShape {
    int ft, pt;
    double fixed[2], step[2];  // bf16, int8
};
constexpr KsplitShape KSPLIT_SHAPES[] = {{1, 1, {4.5, 4.8}, {0.054, 0.062}},
                                         {1, 2, {4.9, 5.7}, {0.066, 0.079}},
                                         {2, 2, {4.9, 6.1}, {0.101, 0.110}},
                                         {3, 2, {6.1, 7.4}, {0.142, 0.164}},
                                         {2, 4, {6.2, 8.0}, {0.154, 0.170}}};

template <bool I8>
static int ksplit_shape(const ConvArgs &a, double *us) {
    const long M = (long)a.B * a.P * a.Q;
    const int cpc = I8 ? 16 : 8, steps = ((a.C + cpc - 1) / cpc + 7) / 8 * 9;
    int best = -1;
    for (int i = 0; i < (int)(sizeof(KSPLIT_SHAPES) / sizeof(KSPLIT_SHAPES[0])); ++i) {
        const KsplitShape &k = KSPLIT_SHAPES[i];
        if (ksplit_positions(a, 32 * k.pt) > KSPLIT_POSITIONS) continue;
        const long wgs = ((M + 32 * k.pt - 1) / (32 * k.pt)) * ((a.K + 32 * k.ft - 1) / (32 * k.ft)), rounds = (wgs + 255) / 256;
        const double t = k.fixed[I8] + k.step[I8] * steps * rounds * (rounds > 1 ? 1.25 : 1.0);
        if (best < 0 || t < *us) best = i, *us = t;
    }
    return best;
}

// Against conv_small_kernel by that fit and one of its own times (3.4 us + its 16 x 16 tiles x steps / 8500, int8 2.9 + / 5600; 1.6
// times the work where pixels lie a multiple of 256 bytes apart, which crowds few cache channels): 3 x 14 x 14 x 208 6.5 us here
// and 6.2 there, x 256 6.5 and 10.9; 1 x 7 x 7 x 720 11.0 and 7.7.  Against the patch kernel: short reductions (two chunks) on
// many pixels stay there (61 x 28 x 28 x 128 20.4 us here at best, 19.0 there; int8 x 256 channels the same).  Against the
// tile kernel always.  Over the 264 layers: 2816 us, the better of all kernels each time 2773, before this kernel 3658.
template <bool I8>
static hipError_t launch_ksplit(const ConvArgs &a, const QuantArgs &q, hipStream_t s, bool patch) {
    if (!ksplit_covers<I8>(a)) return hipErrorNotSupported;
    double us = 0.0;
    const int shape = ksplit_shape<I8>(a, &us);
    if (shape < 0) return hipErrorNotSupported;
    const long M = (long)a.B * a.P * a.Q;
    const int cpc = I8 ? 16 : 8, cells = (a.C + cpc - 1) / cpc;
    const double work = (double)((M + 15) / 16) * ((a.K + 15) / 16) * ((9 * cells + 3) / 4);
    if (us > (I8 ? 2.9 : 3.4) + work / (I8 ? 5600.0 : 8500.0) * (a.C * (I8 ? 1 : 2) % 256 == 0 ? 1.6 : 1.0)) return hipErrorNotSupported;
    if (patch && cells <= 16 && M > 24000) return hipErrorNotSupported;
    switch (shape) {
        case 0: return launch_ksplit_tile<1, 1, I8>(a, q, s);
        case 1: return launch_ksplit_tile<1, 2, I8>(a, q, s);
        case 2: return launch_ksplit_tile<2, 2, I8>(a, q, s);
        case 3: return launch_ksplit_tile<3, 2, I8>(a, q, s);
        default: return launch_ksplit_tile<2, 4, I8>(a, q, s);
    }
}

hipError_t launch_conv_ksplit(const ConvArgs &a, hipStream_t s, bool patch) { return launch_ksplit<false>(a, QuantArgs{}, s, patch); }
hipError_t launch_conv_ksplit_i8(const ConvArgs &a, const QuantArgs &q, hipStream_t s, bool patch) { return launch_ksplit<true>(a, q, s, patch); }

}  // namespace sushi
