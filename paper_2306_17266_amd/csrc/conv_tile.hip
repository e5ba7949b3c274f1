// Dense 1x1 and 3x3 convolution with few output tiles (late stages of a batch, middle stages of a small one) on the
// matrix cores: an implicit GEMM whose reduction is split over wave groups INSIDE a workgroup.
//
// A workgroup of KS groups of four waves computes 64 filters x 64 consecutive output pixels.  The reduction is
// one flat sequence of 16-byte cells, k = tap * (cells per tap) + cell, whatever the channel count: no padding to a
// chunk per tap.  A step is eight cells; group g multiplies steps g * per .. (g + 1) * per - 1 in LDS buffers of its own
// (two, [cell][row] planes of odd length: neighbouring lanes store the eight cells of one pixel and read 32 rows of one
// cell, both free of bank conflicts), wave (wf, wm) of a group owning 32 filters x 32 pixels.  The loads of the next
// two steps are in flight in registers, one barrier per step.  The KS partial tiles then meet in LDS as they were
// accumulated (32 bits), are added in the order of the groups, and every thread finishes pieces of eight filters of one
// pixel: 16-byte residual loads and stores, contiguous along the channels.
//
// Bound: the serial steps of a workgroup (load latency over two steps, the barrier) and LDS operand reads (a 32 x 32 wave
// tile reads two bytes per clock of what the matrix core could use one of), so the chip has to be filled with
// workgroups and each workgroup's chain be short: hence 64 x 64 tiles and the split.
#include "kernels.h"
#include "device_common.h"

#include <algorithm>
#include <type_traits>

namespace sushi {

typedef __attribute__((ext_vector_type(16))) float ct_f32x16;
typedef __attribute__((ext_vector_type(16))) int ct_i32x16;
typedef __attribute__((ext_vector_type(4))) int ct_i32x4;
typedef __attribute__((ext_vector_type(4))) unsigned ct_u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned ct_u32x2;
constexpr int CT_OOB = 0x7FFFFFF0;

struct TileGeom {
    int tiles_f, tiles_m;
    TileOrder order;
    int M;       // B * P * Q
    int kcells;  // cells of the reduction: taps * cells per tap
    int per;     // steps (of eight cells) per wave group
    int part;    // cell offset of the scale / shift (int8: multiplier, shift, bias) copies in LDS
    int gates;   // cell offset of the gates of the tile's images in LDS
    FastDiv dq, dp, dcell;  // division by Q, P, cells per tap
};

// GATED (bf16, 1x1): every operand cell is multiplied by its image's gates (float32) on its way into LDS and rounded to bf16
// again, which is what a pass over the map would have stored.
template <int KS, int R, bool I8, bool GATED>
__global__ __launch_bounds__(256 * KS, 4) void conv_tile_kernel(ConvArgs a, TileGeom g, QuantArgs q) {
    constexpr int ES = I8 ? 1 : 2, CPC = 16 / ES;  // bytes per element, channels per cell
    constexpr int BN = 64, BM = 64, SA = BN + 1, SB = BM + 1, NT = 256 * KS;
    constexpr int D = 2;  // (with four steps in flight int8 spills and bf16 gains nothing)
    constexpr int BUF = 8 * (SA + SB);  // cells of one LDS buffer: eight weight planes, eight activation planes
    constexpr int NB = 2;               // activation cells a thread stages per step (and two weight cells)
    constexpr int PROW = BN / 4 + 1;    // 16-byte cells per pixel row of a partial tile
    extern __shared__ uint4 ct_lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int grp = __builtin_amdgcn_readfirstlane(tid >> 8), wave = __builtin_amdgcn_readfirstlane((tid >> 6) & 3);
    const int gt = tid & 255;
    const int wf = wave >> 1, wm = wave & 1, l32 = lane & 31, kh = lane >> 5;
    const int ntiles = g.tiles_f * g.tiles_m, per_xcd = (ntiles + 7) >> 3;
    const int tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (tile >= ntiles) return;
    int tf, tm;
    tile_place(tile, g.order, &tf, &tm);
    const int f0 = tf * BN, m0 = tm * BM;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<void *>(a.x), 0, (int)((long)a.B * a.H * a.W * a.C * ES), 0x00020000);
    const __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w), 0, (int)((long)R * R * a.CG * a.Kpad * 16), 0x00020000);

    // what this thread stages: cell bk of pixels (gt >> 3) + 32 i (byte offset of the pixel's window, one bit per tap
    // inside the image), weight cells wave and wave + 4 of filter f0 + lane
    const int bk = gt & 7;
    unsigned boff[NB], bmask[NB], goff[GATED ? NB : 1];
    const int n0 = GATED ? fdiv(fdiv(m0, g.dq), g.dp) : 0;  // first image of the tile
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int m = m0 + (gt >> 3) + 32 * i;
        const bool live = m < g.M;
        const int t = fdiv(live ? m : 0, g.dq), qq = (live ? m : 0) - t * a.Q;
        const int n = fdiv(t, g.dp), pp = t - n * a.P;
        const int h0 = pp * a.stride - a.pad, w0 = qq * a.stride - a.pad;
        boff[i] = (unsigned)(((n * a.H + h0) * a.W + w0) * a.C * ES);
        if (GATED) goff[GATED ? i : 0] = (unsigned)g.gates + (unsigned)((live ? n - n0 : 0) * (a.C >> 2));
        bmask[i] = 0;
        if (R == 1) {
            bmask[i] = live ? 1u : 0u;
        } else {
#pragma unroll
            for (int tap = 0; tap < R * R; ++tap) {
                const int h = h0 + tap / R, w = w0 + tap % R;
                if (live && h >= 0 && h < a.H && w >= 0 && w < a.W) bmask[i] |= 1u << tap;
            }
        }
    }
    const unsigned woff = (unsigned)(f0 + lane) * 16u;
    const bool wlive = f0 + lane < a.Kpad;
    const int k0 = grp * g.per * 8;  // first cell of this group
    ct_u32x4 ra[D][2], rb[D][NB];
    unsigned rin[D];  // int8: bits 0 .. NB - 1: the cell of pixel i holds image; bit 8: a cell of the reduction; bit 9: its upper half is beyond C
    auto load_step = [&](int s, ct_u32x4 *qa, ct_u32x4 *qb, unsigned &in) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int k = k0 + s * 8 + wave + 4 * i;
            const int tap = R == 1 ? 0 : fdiv(k, g.dcell);
            const int cg = k - tap * g.dcell.d;
            const unsigned off = (unsigned)(tap * a.CG + cg) * (unsigned)a.Kpad * 16u;
            qa[i] = __builtin_amdgcn_raw_buffer_load_b128(rw, offset_if(wlive & (k < g.kcells), woff + off), 0, 0);
        }
        const int k = k0 + s * 8 + bk;
        const unsigned live = k < g.kcells ? 1u : 0u;
        const int tap = R == 1 ? 0 : fdiv(k, g.dcell);
        const int cg = k - tap * g.dcell.d;
        const int dr = R == 1 ? 0 : (tap * 11) >> 5, ds = tap - dr * R;  // (tap / 3 for tap < 9)
        const unsigned off = ((unsigned)(dr * a.W + ds) * (unsigned)a.C + (unsigned)cg * CPC) * ES;
        in = live << 8 | (I8 && cg * CPC + 8 >= a.C ? 512u : 0u);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const unsigned ok = bmask[i] >> (tap & 31) & live;
            qb[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, offset_if(ok, boff[i] + off), 0, 0);
            if (I8) in |= ok << i;
        }
    };
    // int8: a cell of the frame holds the code of the real value 0 (the input's zero point) in its active channels, the
    // upper half of a cell that straddles the SubNet's channel count zeros
    const unsigned zfill = (unsigned)(q.zx & 0xFF) * 0x01010101u;
    uint4 *const base = ct_lds + grp * 2 * BUF;
    auto store_step = [&](int s, const ct_u32x4 *qa, const ct_u32x4 *qb, unsigned in) {
        uint4 *dst = base + (s & 1) * BUF;
#pragma unroll
        for (int i = 0; i < 2; ++i) dst[(wave + 4 * i) * SA + lane] = __builtin_bit_cast(uint4, qa[i]);
        dst += 8 * SA + bk * SB + (gt >> 3);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            ct_u32x4 v = qb[i];
            if (GATED) {  // (cells past the last: zeros, times the gates of the last)
                const uint4 *gc = ct_lds + goff[GATED ? i : 0] + 2 * min(k0 + s * 8 + bk, g.kcells - 1);
                v = gate_cell(v, __builtin_bit_cast(ct_u32x4, gc[0]), __builtin_bit_cast(ct_u32x4, gc[1]));
            }
            if (I8) {
                if ((in & 256u) && !(in >> i & 1u)) v = ct_u32x4{zfill, zfill, zfill, zfill};
                if (in & 512u) v[2] = 0u, v[3] = 0u;
            }
            dst[32 * i] = __builtin_bit_cast(uint4, v);
        }
    };

    // The tile's epilogue constants first, then the loads of the first D steps.  Every load below is issued on every
    // path, also past the last step (those return zeros and store them where nobody reads): a load under a branch
    // would make the wait for a step's cells a wait for ALL loads in flight.
    uint4 cst[I8 ? 4 : 2];
    {
        auto rsrc = [&](const void *p) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, p ? a.K * 4 : 0, 0x00020000); };
        const void *const src[4] = {I8 ? (const void *)q.qmult : (const void *)a.scale, I8 ? (const void *)q.qshift : (const void *)a.shift, q.qbias, q.wsum};
#pragma unroll
        for (int i = 0; i < (I8 ? 4 : 2); ++i)
            cst[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc(src[i]), (f0 + (tid & 15) * 4) * 4, 0, 0));
    }
#pragma unroll
    for (int d = 0; d < D; ++d) load_step(d, ra[d], rb[d], rin[d]);
    __builtin_amdgcn_sched_barrier(0);
    if (I8) {  // (the zero-point term goes to the bias: minus z_x times the sum of the active weights)
        cst[1] = make_uint4(max((int)cst[1].x, 1), max((int)cst[1].y, 1), max((int)cst[1].z, 1), max((int)cst[1].w, 1));  // (filters beyond K: any valid shift)
        cst[I8 ? 2 : 0].x -= q.zx * cst[I8 ? 3 : 0].x, cst[I8 ? 2 : 0].y -= q.zx * cst[I8 ? 3 : 0].y, cst[I8 ? 2 : 0].z -= q.zx * cst[I8 ? 3 : 0].z, cst[I8 ? 2 : 0].w -= q.zx * cst[I8 ? 3 : 0].w;
    } else if (!a.scale) {
        cst[0] = make_uint4(0x3F800000u, 0x3F800000u, 0x3F800000u, 0x3F800000u);
    }
    if (GATED) {
        const int last = min(m0 + BM, g.M) - 1, cells = (fdiv(fdiv(last, g.dq), g.dp) - n0 + 1) * (a.C >> 2);
        const uint4 *src = reinterpret_cast<const uint4 *>(q.gate + (long)n0 * a.C);
        for (int k = tid; k < cells; k += NT) ct_lds[g.gates + k] = src[k];
    }
    if (tid < BN / 4)
#pragma unroll
        for (int i = 0; i < (I8 ? 3 : 2); ++i) ct_lds[g.part + i * (BN / 4) + tid] = cst[i];

    typename std::conditional<I8, ct_i32x16, ct_f32x16>::type acc;
#pragma unroll
    for (int k = 0; k < 16; ++k) acc[k] = 0;

    if (GATED) __syncthreads();  // (the gates are there)
    store_step(0, ra[0], rb[0], rin[0]);
    __syncthreads();
    // one step: s is in LDS buffer s & 1, set d took it there and is free; the cells of step s + 1 are in set (d + 1) % D
    auto step = [&](int s, auto d_tag, auto load_tag) {
        constexpr int d = decltype(d_tag)::value, dn = (d + 1) % D;
        const uint4 *wb = base + (s & 1) * BUF, *pb = wb + 8 * SA;
        Frag fa[4], fb[4];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            fa[h].u = wb[(2 * h + kh) * SA + wf * 32 + l32];
            fb[h].u = pb[(2 * h + kh) * SB + wm * 32 + l32];
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(load_tag)::value) load_step(s + D, ra[d], rb[d], rin[d]);
        store_step(s + 1, ra[dn], rb[dn], rin[dn]);
#pragma unroll
        for (int h = 0; h < 4; ++h)
            if constexpr (I8)
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(ct_i32x4, fa[h].u), __builtin_bit_cast(ct_i32x4, fb[h].u), acc, 0, 0, 0);
            else
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[h].v, fb[h].v, acc, 0, 0, 0);
        __syncthreads();
    };
    using std::integral_constant;
    int s = 0;
    for (; s + D <= g.per; s += D) {
        step(s, integral_constant<int, 0>{}, std::true_type{});
        step(s + 1, integral_constant<int, 1>{}, std::true_type{});
    }
    if (s < g.per) step(s, integral_constant<int, 0>{}, std::false_type{});  // (in flight already)

    // ---- the partial tiles meet: [group][pixel][filter] (32-bit), over the staging buffers (the barrier above has released them)
    uint4 *const part = ct_lds;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        typedef typename std::conditional<I8, ct_i32x4, f32x4_t>::type v4;
        const v4 v = {acc[4 * jj], acc[4 * jj + 1], acc[4 * jj + 2], acc[4 * jj + 3]};
        part[(grp * BM + wm * 32 + l32) * PROW + wf * 8 + 2 * jj + kh] = __builtin_bit_cast(uint4, v);
    }
    constexpr int PIECES = BM * (BN / 8), EPT = (PIECES + NT - 1) / NT;
    const int cc = tid & 7, f = f0 + cc * 8;  // (the same eight filters in all of a thread's pieces)
    const int obytes = (int)((long)g.M * a.K * ES);
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.res ? a.res : a.y), 0, obytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(a.y, 0, obytes, 0x00020000);
    ct_u32x4 res[EPT];
    int ooff[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int idx = tid + NT * e, m = m0 + (idx >> 3);
        ooff[e] = idx < PIECES && m < g.M && f < a.K ? (m * a.K + f) * ES : CT_OOB;
        res[e] = ct_u32x4{0u, 0u, 0u, 0u};
        if (a.res) {
            if (I8) {
                const ct_u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rr, ooff[e], 0, 0);
                res[e][0] = v[0], res[e][1] = v[1];
            } else {
                res[e] = __builtin_amdgcn_raw_buffer_load_b128(rr, ooff[e], 0, 0);
            }
        }
    }
    __syncthreads();
    const uint4 *const ss = ct_lds + g.part;
    float sc[8], sh[8];
    if constexpr (!I8) load8(reinterpret_cast<const float *>(ss) + cc * 8, sc), load8(reinterpret_cast<const float *>(ss) + BN + cc * 8, sh);
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int idx = tid + NT * e;
        if (PIECES % NT != 0 && idx >= PIECES) break;
        const uint4 *src = part + (idx >> 3) * PROW + 2 * cc;
        if constexpr (I8) {
            int v[8] = {};
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                const uint4 lo = src[k * BM * PROW], hi = src[k * BM * PROW + 1];
                v[0] += (int)lo.x, v[1] += (int)lo.y, v[2] += (int)lo.z, v[3] += (int)lo.w;
                v[4] += (int)hi.x, v[5] += (int)hi.y, v[6] += (int)hi.z, v[7] += (int)hi.w;
            }
            const int *mu = reinterpret_cast<const int *>(ss) + cc * 8;
            const int lo = a.act == 1 ? q.zy : -128;
            unsigned packed[2] = {0u, 0u};
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                long long t = rr64((long long)(v[i] + mu[2 * BN + i]) * (long long)mu[i], mu[BN + i]);
                if (a.res) t += rr64((long long)((int)(int8_t)(res[e][i >> 2] >> (8 * (i & 3))) - q.z_res) * (long long)q.m_res, q.sh_res);
                t += q.zy;
                const int c = (int)(t < lo ? lo : t > 127 ? 127 : t);
                packed[i >> 2] |= (unsigned)(c & 0xFF) << (8 * (i & 3));
            }
            __builtin_amdgcn_raw_buffer_store_b64(ct_u32x2{packed[0], packed[1]}, ry, ooff[e], 0, 0);
        } else {
            float v[8] = {};
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                const float4 lo = __builtin_bit_cast(float4, src[k * BM * PROW]), hi = __builtin_bit_cast(float4, src[k * BM * PROW + 1]);
                v[0] += lo.x, v[1] += lo.y, v[2] += lo.z, v[3] += lo.w;
                v[4] += hi.x, v[5] += hi.y, v[6] += hi.z, v[7] += hi.w;
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                v[i] = v[i] * sc[i] + sh[i];
                if (a.res) v[i] += bf2f(i & 1 ? res[e][i >> 1] >> 16 : res[e][i >> 1] & 0xFFFFu);
            }
            ct_u32x4 o;
            with_activation(a.act, a.hsigmoid, [&](auto act) {
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = pack_bf16x2(activate_as<decltype(act)::value>(v[2 * i]), activate_as<decltype(act)::value>(v[2 * i + 1]));
            });
            __builtin_amdgcn_raw_buffer_store_b128(o, ry, ooff[e], 0, 0);
        }
    }
}

// Filters fast?  3x3 where the input is larger than the weights; 1x1 in bf16 where it is ten times as large (stride 2: and the reduction
// long); from about one tile per compute unit on.  In whole queries, pixels and filters fast, us: 16 x 56 x 56 x 176 3x3/2 25.3 and
// 22.1; 61 x 14 x 14, 256 -> 1024 23.7 and 20.0; 16 x 28 x 28, 512 -> 176 10.9 and 9.4; on the other side 16 x 14 x 14, 1024 -> 720
// 14.7 and 15.9; 16 x 56 x 56, 256 -> 512 /2 13.7 and 16.2; int8 16 x 28 x 28, 176 -> 512 11.8 and 13.9.
static bool tile_filters_fast(const ConvArgs &a, bool i8, long tiles) {
    const long M = (long)a.B * a.P * a.Q;
    if (tiles <= 192) return false;
    if (a.R == 3) return (long)a.B * a.H * a.W > 9l * a.K;
    return !i8 && M >= 10l * a.K && (a.stride == 1 || a.C >= 512);
}

// Cells of the gates that a tile of 64 pixels may need: as many images as it can touch.
static long tile_gate_cells(const ConvArgs &a) { return std::min((long)a.B, 62l / ((long)a.P * a.Q) + 2) * (a.C >> 2); }

template <int KS, int R, bool I8, bool GATED = false>
static hipError_t launch_tile(const ConvArgs &a, const QuantArgs &q, hipStream_t s) {
    constexpr int BM = 64, BUF = 8 * (65 + BM + 1), CPC = I8 ? 16 : 8;
    TileGeom g;
    g.M = a.B * a.P * a.Q;
    g.tiles_f = (a.K + 63) / 64, g.tiles_m = (g.M + BM - 1) / BM;
    g.order = tile_order(tile_filters_fast(a, I8, (long)g.tiles_f * g.tiles_m), g.tiles_f, g.tiles_m);
    const int cells = (a.C + CPC - 1) / CPC;
    g.kcells = R * R * cells;
    g.per = ((g.kcells + 7) / 8 + KS - 1) / KS;
    g.dq = make_fastdiv(a.Q), g.dp = make_fastdiv(a.P), g.dcell = make_fastdiv(cells);
    g.part = std::max(KS * 2 * BUF, KS * BM * 17);
    g.gates = g.part + (I8 ? 48 : 32);
    const size_t lds = ((size_t)g.gates + (GATED ? tile_gate_cells(a) : 0)) * 16;
    static_assert((size_t)KS * 2 * BUF * 16 + 768 <= 160 * 1024 && (size_t)KS * BM * 17 * 16 + 768 <= 160 * 1024, "LDS of a compute unit");
    auto kern = conv_tile_kernel<KS, R, I8, GATED>;
    static LdsLimit limit;
    const hipError_t e = limit.raise(kern);
    if (e != hipSuccess) return e;
    const int per_xcd = (g.tiles_m * g.tiles_f + 7) / 8;
    hipLaunchKernelGGL(kern, dim3(per_xcd * 8), dim3(256 * KS), lds, s, a, g, q);
    return hipGetLastError();
}

template <bool I8>
static bool tile_covers(const ConvArgs &a) {
    const int es = I8 ? 1 : 2;
    if (a.in_f32 || a.out_f32 || (a.C & 7) || a.C < 8 || (a.K & 7) || a.K < 8) return false;
    if (!(a.R == 1 || a.R == 3) || a.pad != (a.R - 1) / 2 || a.stride < 1 || a.stride > 2 || a.Rmax != a.R) return false;
    const long M = (long)a.B * a.P * a.Q, lim = (1l << 31) - 4096;
    return M * a.K * es < lim && (long)a.B * a.H * a.W * a.C * es < lim && (long)a.R * a.R * a.CG * a.Kpad * 16 < (1l << 30);
}

// Wave groups per workgroup: a reduction is split where the tiles leave compute units without enough waves and each
// group still has steps to run (every group costs a partial tile in LDS).  One, two, four groups, bf16, us:
// 16 x 7 x 7 x 720 3x3 (156 tiles, 102 steps) 39.6 / 27.3 / 23.6; 16 x 14 x 14 x 360 3x3 (294, 51) 27.7 / 25.8 / 29.1;
// 16 x 14 x 14, 1024 -> 360 (294, 16) 11.5 / 12.2 / 15.7; 28 x 28, 512 -> 176 (39, 8) 6.0 / 5.2 / 6.0.
static int tile_groups(const ConvArgs &a, bool i8, int *steps) {
    const int cpc = i8 ? 16 : 8;
    const long tiles = (((long)a.B * a.P * a.Q + 63) / 64) * ((a.K + 63) / 64);
    const int n = (a.R * a.R * ((a.C + cpc - 1) / cpc) + 7) / 8;
    *steps = n;
    return tiles <= 192 && n >= (i8 ? 16 : 64) ? 4 : (tiles <= 256 && n >= 4) || (tiles <= 512 && n >= (i8 ? 6 : 32)) ? 2 : 1;
}

template <bool I8>
static hipError_t launch_tile_ks(const ConvArgs &a, const QuantArgs &q, hipStream_t s) {
    int steps;
    const int ks = tile_groups(a, I8, &steps);
    if (!I8 && q.gate)
        return ks == 4   ? launch_tile<4, 1, false, true>(a, q, s)
               : ks == 2 ? launch_tile<2, 1, false, true>(a, q, s)
                         : launch_tile<1, 1, false, true>(a, q, s);
    if (a.R == 1)
        return ks == 4 ? launch_tile<4, 1, I8>(a, q, s) : ks == 2 ? launch_tile<2, 1, I8>(a, q, s) : launch_tile<1, 1, I8>(a, q, s);
    return ks == 4 ? launch_tile<4, 3, I8>(a, q, s) : ks == 2 ? launch_tile<2, 3, I8>(a, q, s) : launch_tile<1, 3, I8>(a, q, s);
}

// Few pixels: conv_small_kernel's 16 x 16 tiles spread a layer over the chip but re-read its operands per tile, so its time
// grows with tiles x steps; this kernel's grows with the serial steps of one workgroup.  Fits in us to 45 layer shapes from
// 1 x 7 x 7 to 32 x 7 x 7 and 1 x 112 x 112 (constants common to both left out): small = W / 6500 (bf16 1x1), W / 8500
// (bf16 3x3), W / 5000 (int8) with W = 16 x 16 tiles x steps of four cells; tile = 0.4 + steps per group x 0.23, 0.42, 0.75
// (int8 0.5, 0.75, 1.35) for one, two, four groups, and 1 for 3x3.  On both sides of the line (traces of whole queries): 2 x
// 28 x 28 x 176 3x3 10.4 us small, 11.4 tile; 3 x 28 x 28 13.3 and 11.8; 1 x 56 x 56, 208 -> 56 4.8 and 5.4, 208 -> 128
// 5.8 and 5.3.  Over 500 layers of both precisions the line costs 0.3 % over the better of the two.  Of up to 16 filters the
// tile kernel's 64 are mostly padding; those short reductions run here for any number of pixels (64 x 112 x 112, 16 -> 16 with
// residual: 22.5 us small, 36 tile; 128 -> 16: 35 and 43; 16 x 56 x 56, 96 -> 16: 4.2 and 6.0).
bool conv_small_is_faster(const ConvArgs &a, bool i8) {
    if (!i8 && a.R == 1 && a.K <= 16 && a.C <= 128) return true;
    const double M = (double)a.B * a.P * a.Q;
    const int cells = a.R * a.R * ((a.C + (i8 ? 15 : 7)) / (i8 ? 16 : 8));
    const double work = (double)(long)((M + 15) / 16) * ((a.K + 15) / 16) * ((cells + 3) / 4);
    int steps;
    const int ks = tile_groups(a, i8, &steps);
    const double per_step = ks == 1 ? (i8 ? 0.5 : 0.23) : ks == 2 ? (i8 ? 0.75 : 0.42) : (i8 ? 1.35 : 0.75);
    return work / (i8 ? 5000.0 : a.R == 1 ? 6500.0 : 8500.0) <= 0.4 + (steps + ks - 1) / ks * per_step + (a.R == 3 ? 1.0 : 0.0);
}

// Of the layers that the patch kernel covers as well (patch) these stay there:
//   3x3 with stride 1 and at least 128 of its tiles: one copy of the input serves nine taps (16 x 56 x 56 x 88: 15.6 us
//       there, 26.2 here; with 75 tiles, 16 x 14 x 14 x 360, 33.8 against 25.8);
//   3x3 with stride 2 where its tiles are 128 filters wide and fill whole rounds of the chip, one on each compute unit, to
//       0.85 and more (96 x 14 x 14 x 720, 222 tiles: 92 us there, 116 here; 61 x 28 x 28 x 360, 282 tiles, 92 against 76; in
//       tiles of 96 filters, 61 x 56 x 56 x 176, 748 tiles, 81 against 65);
//   bf16 1x1 of at most 128 channels, all prologue and epilogue, without a residual where its tiles pad fewer filters and there
//       are pixels for several rounds of the chip (64 x 112 x 112, 32 -> 72: 53 us there, 62 here; 16 x 56 x 56, 64 -> 96: 6.7
//       and 8.0; 16 x 28 x 28, 64 -> 96: 5.3 and 4.4), and those of very many pixels and more than one tile here (64 x 112 x
//       112, 64 -> 144: 129 and 145).  The rest ran there until the epilogue here took its activation branch once: 16 x 56 x
//       56, 64 -> 256 with residual 12.9 us here, 19.0 there, 64 x 14 x 14, 80 -> 256 6.8 and 7.6; 61 x 56 x 56, 64 -> 64
//       12.0 and 14.1;
//   1x1 of more channels without a residual where its tiles, two on each compute unit, fill rounds to 0.85, in bf16 those of at most 96
//       filters (96 x 14 x 14, 816 -> 288, 441 tiles: 24 us there, 29 here; 61 x 14 x 14, 816 -> 288, 282 tiles, 21 on both;
//       in tiles of 128, 96 x 14 x 14, 1024 -> 360, 40 against 37);
//   1x1 of many pixels where its tiles pad fewer filters (16 x 56 x 56, 256 -> 88: 11.3 us there, 16.1 here).
template <bool I8>
static bool tile_is_faster(const ConvArgs &a, bool patch) {
    if (!patch) return true;
    const long M = (long)a.B * a.P * a.Q;
    const int pf = conv_patch_tile_filters(a.K);
    const long tiles = ((M + 127) / 128) * ((a.K + pf - 1) / pf);
    auto full_rounds = [&](long per_round) { return tiles * 100 >= (tiles + per_round - 1) / per_round * per_round * 85; };
    if (a.R == 3) return a.stride == 1 ? tiles < 128 : pf != 128 || !full_rounds(256);
    if (a.stride != 1) return true;  // (not covered there)
    const bool pads_fewer = (a.K + 63) / 64 * 64 > (a.K + pf - 1) / pf * pf;
    if (!I8 && a.C <= 128) return a.res || M <= 32768 || !(pads_fewer || (M > 1l << 19 && a.K > 64));
    if (M <= 32768) return a.res || (!I8 && pf == 128) || !full_rounds(512);
    return !pads_fewer;
}

bool conv_tile_gated_covers(const ConvArgs &a) { return a.R == 1 && tile_covers<false>(a) && tile_gate_cells(a) * 16 <= 24 * 1024; }

hipError_t launch_conv_tile(const ConvArgs &a, hipStream_t s, bool patch, const float *gate) {
    if (!tile_covers<false>(a) || !tile_is_faster<false>(a, patch)) return hipErrorNotSupported;
    QuantArgs q{};
    q.gate = gate;
    return launch_tile_ks<false>(a, q, s);
}

hipError_t launch_conv_tile_i8(const ConvArgs &a, const QuantArgs &q, hipStream_t s, bool patch) {
    if (!tile_covers<true>(a) || !tile_is_faster<true>(a, patch)) return hipErrorNotSupported;
    return launch_tile_ks<true>(a, q, s);
}

}  // namespace sushi
