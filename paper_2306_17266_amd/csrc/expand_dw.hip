// The first two layers of an inverted-residual block in one launch (bf16): 1x1 expansion, then the depthwise k x k layer on the
// expanded map, which stays in LDS: the map of the block with the most channels is neither written nor read.  Optionally the
// sums of the output per image and channel (the pooling of a squeeze-excite block) come with it.
//
// A workgroup (8 waves) owns 32 expanded channels and runs through tiles of the output, one after the other:
//   expansion   the tile's input region (halo included) in quads of four neighbouring pixels of a row: the rows of a matrix
//               instruction are 16 pixels (operands straight from the channels-last map), the columns 16 channels, so a lane
//               ends with four neighbouring pixels of one channel and stores them, activated and rounded to bf16, as 8 bytes of
//               that channel's plane in LDS.  What a quad needs (offsets into the map and the plane, which of its pixels lie in
//               the image) comes from tables in LDS; pixels outside are computed from whatever is read there and masked to zeros.
//   depthwise   a matrix instruction multiplies, for ONE channel, the Toeplitz operand of two kernel rows (rows: a block of 2 x 8
//               outputs, 4 x 4 for stride 2; reduction: two input rows x 16 columns) with those rows of the plane (columns:
//               16 blocks, anywhere in the tile, of one or several images).  4 instructions of 16 clocks for 256 outputs of a 7x7
//               kernel (stride 2: 7); with channels along the rows and diagonal operands (dwconv_mfma.hip) it is 28.  The
//               Toeplitz operands stay in registers for all tiles.
//   output      through LDS, so that the 32 channels of a pixel are stored in one run.
// The expansion is computed again for the halo (1.7 times in all for 14 x 28 outputs of a 7x7 kernel); with 8 to 160 input
// channels that costs less than writing and reading the map.
//
// Both layers with a launch each and here: 64 x 56 x 56, 24 -> 144, 7x7 80 and 50 us (1.3 TB/s of what is left to move), 64 x
// 28 x 28, 40 -> 240, with the pooling 40 and 28; one image, 56 x 56, 24 -> 144, 8.3 us in two kernels and 8.5 here, but one
// launch of 3.7 us less.  Not bound by the matrix cores (by count 5 of the 50 us) nor by memory, but by the vector
// instructions that scale, activate and pack every expanded value, halo included, and by the phases' LDS traffic between
// barriers; at one image by the prologue (tables, Toeplitz operands, first loads: 4 us).
//
// Zero times infinity: an operand's zeros meet values of the same channel only, and sums that are not finite are computed
// again tap by tap.
#include "kernels.h"
#include "device_common.h"

#include <algorithm>
#include <type_traits>

namespace sushi {

constexpr int XDW_CPW = 4, XDW_CB = 8 * XDW_CPW;  // channels of a wave, of a workgroup
constexpr int XDW_OP = 2 * XDW_CB + 16;           // bytes of an output pixel in LDS
constexpr int XDW_OQ = 4 * XDW_OP + 16;           // bytes of four (an odd multiple of 16: lanes write every fourth pixel)

template <int ACT>
__device__ __forceinline__ float xdw_act(float v) {
    return ACT == 1 ? fmaxf(v, 0.0f) : v * fminf(fmaxf(v + 3.0f, 0.0f), 6.0f) * (1.0f / 6.0f);
}

template <int CTRL>
__device__ __forceinline__ float xdw_dpp(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

template <int R, int S, int KS, int ACT>
__global__ __launch_bounds__(512, 2) void expand_dw_kernel(ExpandDwArgs a, ExpandDwGeom g) {
    constexpr int HALF = (R - 1) / 2, CPW = XDW_CPW, CB = XDW_CB, NT = CB / 16, OP = XDW_OP, OQ = XDW_OQ;
    constexpr int BW = S == 1 ? 8 : 4, BH = S == 1 ? 2 : 4;   // outputs of a block
    constexpr int NF = S == 1 ? (R + 1) / 2 : (R + 7) / 2;    // Toeplitz operands of a channel: pairs of input rows of a block
    constexpr int D = KS <= 2 ? 4 : S == 2 && KS >= 4 ? 1 : 2;  // matrix tiles of the expansion in flight
    extern __shared__ uint4 xdw_lds[];
    char *const plane = reinterpret_cast<char *>(xdw_lds), *const aux = plane + g.out;
    uint2 *const quad = reinterpret_cast<uint2 *>(plane + g.tab);       // [quad] offset into the map, into a plane
    const int nqp = (g.nq + 3) & ~3;
    uint2 *const mask = quad + nqp;                                     // [2][quad] which of its pixels lie in the image
    uint4 *const block = reinterpret_cast<uint4 *>(mask + 2 * nqp);     // [16 blocks][lane] its operand, outputs, first of them, image
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // consecutive workgroup ids land on different XCDs: every XCD gets one range of jobs, so that the channel blocks of a tile
    // share its input and the lines of its output in one L2
    const int job = (int)(blockIdx.x & 7) * ((int)gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    const int worker = job / g.groups;
    if (worker >= g.workers) return;
    const int c0 = (job - worker * g.groups) * CB;
    const int cells = a.C >> 3;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.x), 0, (int)((long)a.B * a.H * a.W * a.C * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w1), 0, cells * a.Kpad1 * 16, 0x00020000);
    const int task_end = (int)((long)(worker + 1) * g.total / g.workers);
    int task = (int)((long)worker * g.total / g.workers);

    // ---- weights and constants of the channel block
    unsigned tap[8];  // thread (kernel row, channel): the row's taps (row R: zeros)
    const int trow = tid / CB, tch = tid % CB;
#pragma unroll
    for (int k = 0; k < 8; ++k)
        tap[k] = k < R && trow < R ? static_cast<const uint16_t *>(a.w2)[dw_tap_index(trow - HALF, k - HALF) * a.Kpad2 + min(c0 + tch, a.Kpad2 - 1)] : 0u;
    u32x4_t we[NT][KS];
    float sc1[NT], sh1[NT], sc2[CPW], sh2[CPW];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int ch = c0 + t * 16 + l16, cc = min(ch, a.K - 1);
#pragma unroll
        for (int k = 0; k < KS; ++k)
            we[t][k] = __builtin_amdgcn_raw_buffer_load_b128(
                rw, offset_if((k * 4 + kg < cells) & (ch < a.Kpad1), ((unsigned)(k * 4 + kg) * (unsigned)a.Kpad1 + (unsigned)ch) * 16u), 0, 0);
        sc1[t] = a.scale1[cc], sh1[t] = a.shift1[cc];
    }
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
        const int cc = min(c0 + wave * CPW + c, a.K - 1);
        sc2[c] = a.scale2[cc], sh2[c] = a.shift2[cc];
    }
    __builtin_amdgcn_sched_barrier(0);
    // ---- zeros: the planes (what lies outside the image in every tile stays so)
    for (int k = tid; k < CB * g.pp / 16; k += 512) xdw_lds[k] = make_uint4(0, 0, 0, 0);

    // ---- tiles and the tables
    int n0 = 0, oy0 = 0, ox0 = 0, tile = 0;  // first image of a tile, its first output, its number in the image
    unsigned base = 0;                       // byte offset of its region (may lie before the map)
    auto locate = [&](int t) {
        const int grp = fdiv(t, g.dper);
        tile = t - grp * g.dper.d, n0 = grp * g.im;
        const int y = fdiv(tile, g.dtx);
        oy0 = y * g.by * BH, ox0 = (tile - y * g.tx) * g.bx * BW;
        base = (unsigned)(((n0 * a.H + oy0 * S - HALF) * a.W + ox0 * S - HALF) * a.C * 2);
    };
    // masks of the current tile's quads; two words of two bf16 values
    auto masks = [&](int set) {
        for (int q = tid; q < nqp; q += 512) {
            const int i = fdiv(q, g.dqw), col = (q - i * g.qw) * 4, row = i - fdiv(i, g.drows) * g.rows + g.r0;
            const int h = oy0 * S - HALF + row, w = ox0 * S - HALF + col;
            const bool in = q < g.nq && h >= 0 && h < a.H;
            unsigned m[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) m[k] = in && w + k >= 0 && w + k < a.W ? 0xFFFFu : 0u;
            mask[set * nqp + q] = make_uint2(m[0] | m[1] << 16, m[2] | m[3] << 16);
        }
    };
    locate(task);
    // operands of matrix tile mt: pixel l16 & 3 of quad 4 mt + l16 / 4, cells 4 k + kg
    const unsigned lane_off = (unsigned)((l16 & 3) * a.C * 2 + kg * 16), tail = (KS - 1) * 4 + kg < cells ? 0u : PAST_END;
    u32x4_t px[D][KS];
    auto load = [&](unsigned off, u32x4_t *dst) {
        off += base + lane_off;
#pragma unroll
        for (int k = 0; k < KS; ++k) dst[k] = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)((k == KS - 1 ? off | tail : off) + k * 64u), 0, 0);
    };
    auto quad_offset = [&](int q) {
        const int i = fdiv(q, g.dqw), col = (q - i * g.qw) * 4, img = fdiv(i, g.drows), row = i - img * g.rows + g.r0;
        return (unsigned)(((img * a.H + row) * a.W + col) * a.C * 2);
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load(quad_offset(min((wave + 8 * d) * 4 + (l16 >> 2), g.nq - 1)), px[d]);
    __builtin_amdgcn_sched_barrier(0);
    for (int q = tid; q < nqp; q += 512) {
        const int i = fdiv(q, g.dqw), col = (q - i * g.qw) * 4, img = fdiv(i, g.drows), row = i - img * g.rows + g.r0;
        quad[q] = q < g.nq ? make_uint2((unsigned)(((img * a.H + row) * a.W + col) * a.C * 2), (unsigned)((img * g.rh + row) * g.rp + col * 2))
                           : make_uint2(PAST_END, (unsigned)g.pp - 16u);  // (the last 16 bytes of a plane are nobody's)
    }
    masks(0);
    if (wave < g.ng) {
        const int col = wave * 16 + l16, img = g.im == 1 ? 0 : col / g.ns, b = col - img * g.ns;
        const int yb = fdiv(b, g.dbx), xb = b - yb * g.bx;
        const bool there = yb < g.by && img < g.im;
        const int y = there ? yb * BH + (S == 1 ? kg >> 1 : kg) : 0, x = there ? xb * BW + (S == 1 ? (kg & 1) * 4 : 0) : 0;  // (first of four outputs)
        const int quads = (g.im * g.dth.d * g.dtw.d) >> 2, oq = there ? ((img * g.dth.d + y) * g.dtw.d + x) >> 2 : quads;  // (past the last: nobody's)
        block[wave * 64 + lane] = make_uint4((unsigned)((there ? (img * g.rh + yb * BH * S) * g.rp + xb * 16 : 0) + (kg >> 1) * g.rp + (kg & 1) * 16),
                                             (unsigned)(oq * OQ), (unsigned)(y << 16 | x), there ? (unsigned)img : ~0u);
    }
    // The taps, [channel][kernel row]: eight zeros, the row's taps, zeros up to 24 values; and the same one value further on, so
    // that eight values from any position on start on a word of one of the two.  A row of zeros behind the last.
    if (trow <= R) {
        uint4 *const dst = reinterpret_cast<uint4 *>(aux) + (tch * (R + 1) + trow) * 6;
        dst[0] = dst[2] = dst[5] = make_uint4(0, 0, 0, 0);
        dst[1] = make_uint4(tap[0] | tap[1] << 16, tap[2] | tap[3] << 16, tap[4] | tap[5] << 16, tap[6]);
        dst[3] = make_uint4(0, 0, 0, tap[0] << 16);
        dst[4] = make_uint4(tap[1] | tap[2] << 16, tap[3] | tap[4] << 16, tap[5] | tap[6] << 16, 0);
    }
    __syncthreads();
    Frag toep[CPW][NF];
    {
        // row l16 of the operand: output (dy, ox) of a block; reduction value 8 kg + j: input row kg / 2, column 8 (kg % 2) + j
        const int dy = l16 / BW, ox = l16 % BW, from = 8 + (kg & 1) * 8 - ox * S;
        const char *src = aux + wave * CPW * (R + 1) * 96 + (from & 1) * 48 + (from & ~1) * 2;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const int r = 2 * f + (kg >> 1) - dy * S, row = r >= 0 && r < R ? r : R;
#pragma unroll
            for (int c = 0; c < CPW; ++c) {
                const uint32_t *p = reinterpret_cast<const uint32_t *>(src + (c * (R + 1) + row) * 96);
                toep[c][f].u = make_uint4(p[0], p[1], p[2], p[3]);
            }
        }
    }
    const int mtiles = nqp >> 2;
    for (int turn = 0; task < task_end; ++task, turn ^= 1) {
        // ---- expansion
        const uint2 *const live = mask + (g.dper.d == 1 ? 0 : turn * nqp);
        // (table entries are read one matrix tile ahead)
        auto entry = [&](int mt, uint2 &m, unsigned &own, unsigned &next) {
            const int q = min(mt * 4 + kg, nqp - 1);
            m = live[q], own = quad[q].y, next = quad[min((mt + 8 * D) * 4 + (l16 >> 2), nqp - 1)].x;
        };
        uint2 m_ahead;
        unsigned own_ahead, next_ahead;
        entry(wave, m_ahead, own_ahead, next_ahead);
        for (int mt = wave; mt < mtiles; mt += 8 * D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const uint2 m = m_ahead;
                const unsigned own = own_ahead, next = next_ahead;
                entry(mt + 8 * (d + 1), m_ahead, own_ahead, next_ahead);
                __builtin_amdgcn_sched_barrier(0);
                if (mt + 8 * d < mtiles) {
                    char *const dst = plane + own + l16 * g.pp;
                    f32x4_t acc[NT];
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int k = 0; k < KS; ++k)
                            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, px[d][k]), __builtin_bit_cast(bf16x8_t, we[t][k]),
                                                                             acc[t], 0, 0, 0);
                    }
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        float v[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = xdw_act<ACT>(acc[t][i] * sc1[t] + sh1[t]);
                        *reinterpret_cast<uint2 *>(dst + t * 16 * g.pp) = make_uint2(pack_bf16x2(v[0], v[1]) & m.x, pack_bf16x2(v[2], v[3]) & m.y);
                    }
                }
                load(next, px[d]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();
        const int on0 = n0, ooy = oy0, oox = ox0, otile = tile;
        if (task + 1 < task_end) {
            locate(task + 1);
            if (g.dper.d > 1) masks(turn ^ 1);
        }
#pragma unroll
        for (int d = 0; d < D; ++d) load(quad[min((wave + 8 * d) * 4 + (l16 >> 2), nqp - 1)].x, px[d]);
        __builtin_amdgcn_sched_barrier(0);

        // ---- depthwise, 16 blocks at a time
        float sum[CPW];
#pragma unroll
        for (int c = 0; c < CPW; ++c) sum[c] = 0.f;
#pragma unroll 1
        for (int grp = 0; grp < g.ng; ++grp) {
            const uint4 mine = block[grp * 64 + lane];
            const char *const src = plane + wave * CPW * g.pp + mine.x;
            f32x4_t acc[CPW];
            Frag in[2][CPW];
#pragma unroll
            for (int c = 0; c < CPW; ++c) acc[c] = f32x4_t{0.f, 0.f, 0.f, 0.f}, in[0][c].u = *reinterpret_cast<const uint4 *>(src + c * g.pp);
#pragma unroll
            for (int f = 0; f < NF; ++f) {
#pragma unroll
                for (int c = 0; c < CPW; ++c)
                    if (f + 1 < NF) in[(f + 1) & 1][c].u = *reinterpret_cast<const uint4 *>(src + c * g.pp + 2 * (f + 1) * g.rp);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int c = 0; c < CPW; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(toep[c][f].v, in[f & 1][c].v, acc[c], 0, 0, 0);
            }
            float all = 0.f;
#pragma unroll
            for (int c = 0; c < CPW; ++c) all += acc[c][0] + acc[c][1] + acc[c][2] + acc[c][3];
            const int img = (int)mine.w, y = (int)(mine.z >> 16), x = (int)(mine.z & 0xFFFFu);
            const bool there = img >= 0;
            if (!(all * 0.f == 0.f)) {  // (not finite, or a finite sum of large values that is not: tap by tap is right for both)
#pragma unroll 1
                for (int k = 0; k < CPW * 4; ++k) {
                    const int c = k >> 2, i = k & 3, ch = min(c0 + wave * CPW + c, a.Kpad2 - 1);
                    float s = 0.f;
#pragma unroll 1
                    for (int t = 0; t < R * R; ++t) {
                        const int dr = t / R, ds = t % R;
                        const uint16_t v = *reinterpret_cast<const uint16_t *>(plane + (wave * CPW + c) * g.pp + ((there ? img : 0) * g.rh + y * S + dr) * g.rp + ((x + i) * S + ds) * 2);
                        s = fmaf(bf2f(static_cast<const uint16_t *>(a.w2)[(long)dw_tap_index(dr - HALF, ds - HALF) * a.Kpad2 + ch]), bf2f(v), s);
                    }
#pragma unroll
                    for (int cc = 0; cc < CPW; ++cc)
#pragma unroll
                        for (int ii = 0; ii < 4; ++ii)
                            if (cc == c && ii == i) acc[cc][ii] = s;
                }
            }
            unsigned o[4][CPW / 2];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int c = 0; c < CPW; c += 2)
                    o[i][c / 2] = pack_bf16x2(xdw_act<ACT>(acc[c][i] * sc2[c] + sh2[c]), xdw_act<ACT>(acc[c + 1][i] * sc2[c + 1] + sh2[c + 1]));
            char *const dst = aux + mine.y + wave * CPW * 2;
#pragma unroll
            for (int i = 0; i < 4; ++i) *reinterpret_cast<uint2 *>(dst + i * OP) = make_uint2(o[i][0], o[i][1]);
            if (a.pool) {
                const int lim = there && ooy + y < a.P ? a.Q - oox - x : 0;  // how many of the four lie in the map
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int c = 0; c < CPW; c += 2) {
                        const unsigned v = i < lim ? o[i][c / 2] : 0u;
                        sum[c] += bf2f(v & 0xFFFFu), sum[c + 1] += bf2f(v >> 16);
                    }
                if (g.im > 1 || grp + 1 == g.ng) {  // over the lanes of an image; lane kg ends with channel kg
                    const bool k1 = kg & 1, k2 = kg & 2;
                    const float s0 = (k1 ? sum[1] : sum[0]) + __shfl_xor(k1 ? sum[0] : sum[1], 16), s2 = (k1 ? sum[3] : sum[2]) + __shfl_xor(k1 ? sum[2] : sum[3], 16);
                    float t = (k2 ? s2 : s0) + __shfl_xor(k2 ? s0 : s2, 32);
                    if (g.ns > 1) t += xdw_dpp<0xB1>(t);   // lane ^ 1
                    if (g.ns > 2) t += xdw_dpp<0x4E>(t);   // lane ^ 2
                    if (g.ns > 4) t += xdw_dpp<0x141>(t);  // the other half of eight
                    if (g.ns > 8) t += xdw_dpp<0x140>(t);  // the other half of sixteen
                    const int n = on0 + img, ch = c0 + wave * CPW + kg;
                    if ((l16 & (min(g.ns, 16) - 1)) == 0 && there && n < a.B && ch < a.K) a.pool[((long)n * g.parts + (g.im > 1 ? 0 : otile)) * a.K + ch] = t;
#pragma unroll
                    for (int c = 0; c < CPW; ++c) sum[c] = 0.f;
                }
            }
        }
        __syncthreads();
        // ---- the tile's pixels, 32 channels each
        const int pieces = g.im * g.dth.d * g.dtw.d * (CB / 8);
        const int f = c0 + (tid % (CB / 8)) * 8;
        for (int from = tid; from < pieces; from += 1024) {
            uint4 v[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int p = min(from + 512 * e, pieces - 1) / (CB / 8);
                v[e] = *reinterpret_cast<const uint4 *>(aux + (p >> 2) * OQ + (p & 3) * OP + (f - c0) * 2);
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int p = (from + 512 * e) / (CB / 8), i = fdiv(p, g.dtw), x = p - i * g.dtw.d, img = fdiv(i, g.dth), y = i - img * g.dth.d;
                const int n = on0 + img;
                if (from + 512 * e < pieces && n < a.B && ooy + y < a.P && oox + x < a.Q && f < a.K)
                    *reinterpret_cast<uint4 *>(static_cast<uint16_t *>(a.y) + (((long)n * a.P + ooy + y) * a.Q + oox + x) * a.K + f) = v[e];
            }
        }
    }
}

static size_t xdw_lds_bytes(const ExpandDwGeom &g) { return (size_t)g.tab + ((g.nq + 3) & ~3) * 24 + g.ng * 1024; }

// The tile: as few turns of the busiest workgroup as possible, weighted by what a turn costs (clocks, about: 1200 fixed, 300 per
// round of eight matrix tiles of the expansion, 1500 per 16 blocks).  Several images share a tile where one is at most 16 blocks.
ExpandDwGeom expand_dw_geom(const ExpandDwArgs &a) {
    const int S = a.stride, R = a.R, HALF = (R - 1) / 2, BW = S == 1 ? 8 : 4, BH = S == 1 ? 2 : 4;
    const int xb = (a.Q + BW - 1) / BW, yb = (a.P + BH - 1) / BH;
    ExpandDwGeom best{};
    double least = 1e30;
    // (A query that meets a SubNet for the first time pays for this search, for each of its blocks: what is of no use ends early.)
    for (int bx = 1; bx <= std::min(xb, 8); ++bx) {
        const int tx = (xb + bx - 1) / bx;
        if (tx > 1 && (xb + tx - 1) / tx != bx) continue;  // (even tiles only)
        for (int by = 1; by <= std::min(yb, 16) && bx * by <= 32; ++by) {
            const int ty = (yb + by - 1) / by, nb = bx * by;
            if (ty > 1 && (yb + ty - 1) / ty != by) continue;
            for (int im = 1; im <= 8; im *= 2) {
                if (im > 1 && (tx * ty > 1 || nb > 16 || im > a.B)) break;
                ExpandDwGeom g{};
                g.bx = bx, g.by = by, g.im = im;
                g.tx = tx, g.ty = ty;
                g.ns = 1;
                while (g.ns < nb) g.ns *= 2;
                g.ng = im == 1 ? (nb + 15) / 16 : (im * g.ns + 15) / 16;
                if (g.ng > 2) continue;
                const int th = std::min(by * BH, a.P), tw = std::min(bx * BW, a.Q);
                const int nr = (th - 1) * S + R, nc = (tw - 1) * S + R;
                g.rp = bx * 16 + 16, g.rh = by * BH * S + R + (S == 1 ? -1 : 0);
                // with one tile along an axis only the image itself is computed: what lies outside is zeros in every tile
                g.r0 = g.ty == 1 ? HALF : 0;
                g.rows = g.ty == 1 ? std::min(nr - HALF, a.H) : nr;
                g.qw = ((g.tx == 1 ? std::min(nc, HALF + a.W) : nc) + 3) / 4;
                g.nq = im * g.rows * g.qw;
                g.pp = (im * g.rh * g.rp + 127) / 128 * 128 + 16;
                const int nqp = (g.nq + 3) & ~3;
                g.out = XDW_CB * g.pp;
                g.tab = g.out + std::max(XDW_CB * (R + 1) * 96, (im * by * BH * bx * BW / 4 + 1) * XDW_OQ);
                if (xdw_lds_bytes(g) > 160 * 1024) continue;
                g.groups = (a.K + XDW_CB - 1) / XDW_CB;
                g.total = (a.B + im - 1) / im * g.tx * g.ty;
                g.workers = std::min(g.total, std::max(1, 256 / g.groups));
                const double turns = (double)((g.total + g.workers - 1) / g.workers);
                const int parts = g.tx * g.ty;  // (the gates' kernel has sixteen loads in flight)
                const double cost = turns * (1200 + 300 * ((nqp / 4 + 7) / 8) + 1500 * g.ng) + (a.pool && parts > 16 ? 150.0 * (parts - 16) : 0.0);
                if (cost < least) least = cost, best = g;
            }
        }
    }
    ExpandDwGeom &g = best;
    g.dqw = make_fastdiv(g.qw), g.drows = make_fastdiv(g.rows), g.dper = make_fastdiv(g.tx * g.ty), g.dtx = make_fastdiv(g.tx);
    g.dbx = make_fastdiv(g.bx), g.dtw = make_fastdiv(g.bx * BW), g.dth = make_fastdiv(g.by * BH);
    if (g.im == 1) g.ns = 1 << 20;  // (all columns are the one image's)
    g.parts = g.tx * g.ty;
    return g;
}

template <int R, int S, int KS, int ACT>
static hipError_t launch_xdw(const ExpandDwArgs &a, const ExpandDwGeom &g, hipStream_t s) {
    static LdsLimit limit;
    const hipError_t e = limit.raise(expand_dw_kernel<R, S, KS, ACT>);
    if (e != hipSuccess) return e;
    const size_t lds = xdw_lds_bytes(g);
    const unsigned wgs = (unsigned)(((long)g.workers * g.groups + 7) / 8 * 8);
    hipLaunchKernelGGL((expand_dw_kernel<R, S, KS, ACT>), dim3(wgs), dim3(512), lds, s, a, g);
    return hipGetLastError();
}

template <int R, int S, int ACT>
static hipError_t launch_xdw_ks(const ExpandDwArgs &a, const ExpandDwGeom &g, hipStream_t s) {
    switch ((a.C + 31) / 32) {
        case 1: return launch_xdw<R, S, 1, ACT>(a, g, s);
        case 2: return launch_xdw<R, S, 2, ACT>(a, g, s);
        case 3: return launch_xdw<R, S, 3, ACT>(a, g, s);
        case 4: return launch_xdw<R, S, 4, ACT>(a, g, s);
        case 5: return launch_xdw<R, S, 5, ACT>(a, g, s);
        default: return hipErrorInvalidValue;
    }
}

template <int R, int S>
static hipError_t launch_xdw_act(const ExpandDwArgs &a, const ExpandDwGeom &g, hipStream_t s) {
    return a.act == 1 ? launch_xdw_ks<R, S, 1>(a, g, s) : launch_xdw_ks<R, S, 2>(a, g, s);
}

// From an expansion of 2 on: below, the map that is kept from memory is no larger than input and output, and the halo's products
// are paid for all the same.  160 channels are five reduction steps, whose operands a wave still holds in registers.  The
// families' activations (ReLU, hard swish) and kernel sizes only; offsets within 31 bits.
bool expand_dw_covers(const ExpandDwArgs &a) {
    const long lim = (1l << 31) - 256;
    if ((a.C & 7) || a.C < 8 || a.C > 160 || (a.K & 7) || a.K < 8 || a.K < 2 * a.C || a.act < 1 || a.act > 2) return false;
    if (!(a.R == 3 || a.R == 5 || a.R == 7) || a.stride < 1 || a.stride > 2 || !a.scale1 || !a.scale2) return false;
    return (long)a.B * a.H * a.W * a.C * 2 < lim && (long)(a.C >> 3) * a.Kpad1 * 16 < lim && (long)a.B * a.P * a.Q < (1l << 30);
}

hipError_t launch_expand_dw(const ExpandDwArgs &a, const ExpandDwGeom &g, hipStream_t s) {
    if (!expand_dw_covers(a)) return hipErrorInvalidValue;
    switch (a.R * 4 + a.stride) {
        case 3 * 4 + 1: return launch_xdw_act<3, 1>(a, g, s);
        case 3 * 4 + 2: return launch_xdw_act<3, 2>(a, g, s);
        case 5 * 4 + 1: return launch_xdw_act<5, 1>(a, g, s);
        case 5 * 4 + 2: return launch_xdw_act<5, 2>(a, g, s);
        case 7 * 4 + 1: return launch_xdw_act<7, 1>(a, g, s);
        default: return launch_xdw_act<7, 2>(a, g, s);
    }
}

}  // namespace sushi
