// Depthwise k x k convolution on the matrix cores (bf16, activations [B][H][W][C], float32 accumulation).
//
// A depthwise layer has no sum over channels, so one v_mfma_f32_16x16x32_bf16 is used as 16 channels x 16 pixels x TWO
// taps: rows are the channels of a group of 16, columns 16 neighbouring output pixels of a row, and the 32 reduction
// values are (tap, channel).  The weight operand is diagonal per tap (row f holds its weight at channel f,
// zeros elsewhere): 15 of 16 products are zeros, yet an instruction still does 512 useful multiply-adds in 16 clocks, twice
// what the vector ALUs do in that time, and the input needs no unpacking: the 16-byte cells of channels-last memory ARE
// the operand (lane (pixel, kg) holds tap kg / 2 and channels 8 (kg % 2) .. + 7).  The two taps are neighbours of one
// tap row, an odd row's last tap is paired with nothing (its cells are requested past the end of the buffer and arrive
// as zeros, as do all cells outside the image).
//
// A wave keeps the diagonal operands of all taps of its channel group in registers (28 for 7x7) and computes strips of
// T output rows x 16 columns.  An input row's cells are loaded once (PD rows ahead, in registers), pass through a row
// of LDS that belongs to the wave (its LDS instructions execute in order: no barrier), and come back as the row's
// (R + 1) / 2 operands, which are multiplied into every output row of the strip that uses them; the whole strip is
// straight-line code.  The four waves of a workgroup take neighbouring channel groups, so that together they read and
// write whole cache lines.
//
// Bound by the first loads on small maps; on large ones by the matrix cores to about a half (64 x 56 x 56 x 144, 7x7:
// 50 us, of them 24 matrix instructions).
//
// Zero times infinity is not zero: an infinity or NaN in one channel makes the sums of its whole group NaN at the outputs
// that use it.  Sums that are not finite are therefore computed again channel by channel on the vector ALUs, so channels
// stay apart; finite sums cannot have met such a value.
#include "kernels.h"
#include "device_common.h"

#include <algorithm>

namespace sushi {

typedef __attribute__((ext_vector_type(4))) unsigned dm_u32x4;
constexpr int DM_OOB = 0x7FFFFFF0;

struct DwTasks {
    int groups;          // channel groups of 16
    int strips;          // strips of T output rows in a column tile
    int ctiles;          // column tiles of 16
    int total, workers;  // strips of a channel group over all images; waves that share them
};

template <int R, int S, int T, int PD>
__global__ __launch_bounds__(256, 2) void dw_mfma_kernel(ConvArgs a, DwTasks t) {
    constexpr int HALF = (R - 1) / 2, NP = (R + 1) / 2, NH = (T - 1) * S + R;  // NH input rows per strip
    constexpr int NCELL = 2 * (15 * S + R), NL = (NCELL + 63) / 64;  // cells of an input row; loads per lane
    __shared__ uint4 rows_lds[4][NCELL + 1];  // (the last one stays zero: the pair of an odd row's last tap)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // consecutive workgroup ids land on different XCDs: give every XCD one range of jobs, so that the channel groups and
    // the strips that share cache lines meet in its L2
    const int job = ((int)(blockIdx.x & 7) * ((int)gridDim.x >> 3) + (int)(blockIdx.x >> 3)) * 4 + wave;
    const int l16 = lane & 15, kg = lane >> 4, tap2 = kg >> 1;
    const int worker = __builtin_amdgcn_readfirstlane(job / t.groups);
    if (worker >= t.workers) return;
    const int c0 = __builtin_amdgcn_readfirstlane(job % t.groups) * 16;
    const uint16_t *w = static_cast<const uint16_t *>(a.w);
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.x), 0, (int)((long)a.B * a.H * a.W * a.C * 2), 0x00020000);
    uint4 *const row = rows_lds[wave];
    if (lane == 0) row[NCELL] = make_uint4(0, 0, 0, 0);

    // diagonal operands: this lane's one non-zero weight of a tap pair sits at channel l16, if the lane's half has it
    Frag fw[R][NP];
    {
        const bool mine = (l16 >> 3) == (kg & 1);
        const int word = (l16 & 7) >> 1, shift = (l16 & 1) * 16;
        const int cw = min(c0 + l16, a.Kpad - 1);
#pragma unroll
        for (int dr = 0; dr < R; ++dr)
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int t0 = dw_tap_index(dr - HALF, 2 * p - HALF);
                const int t1 = 2 * p + 1 < R ? dw_tap_index(dr - HALF, 2 * p + 1 - HALF) : t0;
                const unsigned raw = w[(tap2 ? t1 : t0) * a.Kpad + cw];
                const unsigned v = mine && 2 * p + tap2 < R ? raw << shift : 0u;
                fw[dr][p].u = make_uint4(word == 0 ? v : 0u, word == 1 ? v : 0u, word == 2 ? v : 0u, word == 3 ? v : 0u);
            }
    }
    const int fs = min(c0 + kg * 4, a.K - 4);
    const float4 sc = *reinterpret_cast<const float4 *>(a.scale + fs), sh = *reinterpret_cast<const float4 *>(a.shift + fs);
    const int row_bytes = a.W * a.C * 2;
    int ridx[NP];  // where this lane reads its operand of tap pair p
#pragma unroll
    for (int p = 0; p < NP; ++p) ridx[p] = 2 * p + tap2 < R ? (l16 * S + 2 * p + tap2) * 2 + (kg & 1) : NCELL;

    const int task_end = (int)((long)(worker + 1) * t.total / t.workers);
    for (int task = (int)((long)worker * t.total / t.workers); task < task_end; ++task) {
        const int st = task % t.strips, rest = task / t.strips;
        const int ct = rest % t.ctiles, n = rest / t.ctiles;
        const int p0 = st * T, q = ct * 16 + l16, h0 = p0 * S - HALF;
        int coff[NL];  // this lane's cells of an input row: byte offset in image n, or -1
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            const int cell = lane + 64 * k, x = ct * 16 * S - HALF + (cell >> 1), cc = c0 + (cell & 1) * 8;
            coff[k] = cell < NCELL && x >= 0 && x < a.W && cc < a.C ? ((n * a.H * a.W + x) * a.C + cc) * 2 : -1;
        }
        auto load_row = [&](int i, dm_u32x4 *dst) {
            const int h = h0 + i;
            const bool ok = h >= 0 && h < a.H;
            const int add = h * row_bytes;
#pragma unroll
            for (int k = 0; k < NL; ++k)
                dst[k] = __builtin_amdgcn_raw_buffer_load_b128(rx, ok && coff[k] >= 0 ? coff[k] + add : DM_OOB, 0, 0);
        };
        auto hand_over = [&](const dm_u32x4 *src, Frag *dst) {
#pragma unroll
            for (int k = 0; k < NL; ++k)
                if (lane + 64 * k < NCELL) row[lane + 64 * k] = __builtin_bit_cast(uint4, src[k]);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int p = 0; p < NP; ++p) dst[p].u = row[ridx[p]];
            __builtin_amdgcn_wave_barrier();
        };
        dm_u32x4 g[PD][NL];  // input rows on their way: row i in set i % PD
        Frag b[2][NP];       // operands of rows i and i + 1
#pragma unroll
        for (int k = 0; k < PD; ++k) load_row(k, g[k]);
        hand_over(g[0], b[0]);
        f32x4_t acc[T];
#pragma unroll
        for (int j = 0; j < T; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < NH; ++i) {
            if (i + 1 < NH) hand_over(g[(i + 1) % PD], b[(i + 1) & 1]);
            if (i + PD < NH) load_row(i + PD, g[i % PD]);
            __builtin_amdgcn_sched_barrier(0);  // (the loads stay ahead of their use)
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int j = 0; j < T; ++j) {
                    const int dr = i - j * S;
                    if (dr >= 0 && dr < R)
                        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[dr][p].v, b[i & 1][p].v, acc[j], 0, 0, 0);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        const int f = c0 + kg * 4;
        const bool mine = q < a.Q && f < a.K;
        auto finish = [&](int p, float s0, float s1, float s2, float s3) {
            float v0 = s0 * sc.x + sh.x, v1 = s1 * sc.y + sh.y, v2 = s2 * sc.z + sh.z, v3 = s3 * sc.w + sh.w;
            with_activation(a.act, 0, [&](auto act) {
                constexpr int ACT = decltype(act)::value;
                v0 = activate_as<ACT>(v0), v1 = activate_as<ACT>(v1), v2 = activate_as<ACT>(v2), v3 = activate_as<ACT>(v3);
            });
            *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(a.y) + (((long)n * a.P + p) * a.Q + q) * a.K + f) =
                make_uint2(pack_bf16x2(v0, v1), pack_bf16x2(v2, v3));
        };
        float bad = 0.f;  // NaN if one of the lane's sums is not finite
#pragma unroll
        for (int j = 0; j < T; ++j)
            if (mine && p0 + j < a.P) {
#pragma unroll
                for (int i = 0; i < 4; ++i) bad = fmaf(acc[j][i], 0.f, bad);
                finish(p0 + j, acc[j][0], acc[j][1], acc[j][2], acc[j][3]);
            }
        // (channel by channel, cells outside the image as zeros)
#pragma unroll 1
        for (int p = bad == bad ? a.P : p0; p < min(p0 + T, a.P); ++p) {
            float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int k = 0; k < R * R; ++k) {
                const int dr = k / R - HALF, ds = k % R - HALF, h = p * S + dr, x = q * S + ds;
                const uint2 wv = *reinterpret_cast<const uint2 *>(w + dw_tap_index(dr, ds) * a.Kpad + f);
                uint2 xv = make_uint2(0u, 0u);
                if (h >= 0 && h < a.H && x >= 0 && x < a.W)
                    xv = *reinterpret_cast<const uint2 *>(static_cast<const uint16_t *>(a.x) + (((long)n * a.H + h) * a.W + x) * a.C + f);
                s[0] = fmaf(bf2f(wv.x & 0xFFFFu), bf2f(xv.x & 0xFFFFu), s[0]), s[1] = fmaf(bf2f(wv.x >> 16), bf2f(xv.x >> 16), s[1]);
                s[2] = fmaf(bf2f(wv.y & 0xFFFFu), bf2f(xv.y & 0xFFFFu), s[2]), s[3] = fmaf(bf2f(wv.y >> 16), bf2f(xv.y >> 16), s[3]);
            }
            finish(p, s[0], s[1], s[2], s[3]);
        }
    }
}

template <int R, int S, int T, int PD>
static hipError_t launch_dw(const ConvArgs &a, hipStream_t s) {
    DwTasks t;
    t.groups = (a.K + 15) / 16;
    t.ctiles = (a.Q + 15) / 16;
    t.strips = (a.P + T - 1) / T;
    t.total = a.B * t.ctiles * t.strips;
    // 2048 waves fit the chip at this register count; the waves of a channel group share its strips
    t.workers = std::min(t.total, std::max(1, 2048 / t.groups));
    hipLaunchKernelGGL((dw_mfma_kernel<R, S, T, PD>), dim3((unsigned)(((long)t.workers * t.groups + 31) / 32 * 8)), dim3(256), 0, s, a, t);
    return hipGetLastError();
}

// Which layers: where one-row strips fill the chip at most once, every kernel size: a small layer is bound by its
// serial load rounds, and the row-strip kernel of dwconv.hip has R of them (7x7 at 14 x 14 x 336, one image: 13.5 us,
// here 4.8; 3x3: 5.2, here 3.8).  On larger maps 3x3 stays there (memory-bound, and the wider loads of that kernel win:
// 21 us against 23 at 64 x 56 x 56 x 96), 5x5 and 7x7 come here (64 x 56 x 56 x 144 7x7: 78 us there, 50 here; 64 x 48 x
// 48 x 144 5x5: 38 and 28), except where less than 0.7 of the strips is map and the rest, counted in whole strips, comes
// to a half (5x5) or 1.65 times (7x7) of what runs at once: that padding costs what the matrix cores gain (us there and
// here: 5x5 48 x 10 x 10 x 480, 0.86 times, 11.3 and 13.0, with 16 images 0.29, 9.0 and 8.2; 7x7 96 x 14 x 14 x 672 / 2, 2.4
// times, 17.5 and 20.4, with 48 images 1.2, 14.2 and 11.8).
template <int R, int S, int T, int PD>
static hipError_t pick_strip(const ConvArgs &a, hipStream_t s) {
    const long ctiles = (a.Q + 15) / 16, columns = a.B * ctiles * ((a.K + 15) / 16);
    if (columns * a.P <= 2048) return launch_dw<R, S, 1, R>(a, s);
    const long strips = (a.P + T - 1) / T;
    const double map = (double)a.Q * a.P / (double)(ctiles * 16 * strips * T);
    if (R == 3 || (map < 0.7 && columns * strips * (1.0 - map) > (R == 5 ? 0.5 : 1.65) * 2048)) return hipErrorNotSupported;
    // T rows per strip re-read fewer input rows, one row per strip spreads a layer over more waves: the fewer input rows
    // in sequence, a strip's first loads counted as eight
    auto cost = [&](int rows) { return (columns * ((a.P + rows - 1) / rows) + 2047) / 2048 * ((rows - 1) * S + R + 8); };
    return cost(T) < cost(1) ? launch_dw<R, S, T, PD>(a, s) : launch_dw<R, S, 1, R>(a, s);
}

// Returns hipErrorNotSupported (nothing launched) for layers the kernel does not cover or that the row-strip kernel
// runs faster.
hipError_t launch_dwconv_mfma(const ConvArgs &a, hipStream_t s) {
    if ((a.K & 7) != 0 || a.C != a.K || a.pad != (a.R - 1) / 2 || !a.scale) return hipErrorNotSupported;
    if ((long)a.B * a.H * a.W * a.C * 2 >= (1l << 31) - 256) return hipErrorNotSupported;
    if ((long)a.B * ((a.Q + 15) / 16) * a.P >= (1l << 30)) return hipErrorNotSupported;
    switch (a.R * 4 + a.stride) {
        case 3 * 4 + 1: return pick_strip<3, 1, 1, 3>(a, s);
        case 3 * 4 + 2: return pick_strip<3, 2, 1, 3>(a, s);
        case 5 * 4 + 1: return pick_strip<5, 1, 8, 5>(a, s);
        case 5 * 4 + 2: return pick_strip<5, 2, 4, 4>(a, s);
        case 7 * 4 + 1: return pick_strip<7, 1, 7, 4>(a, s);
        case 7 * 4 + 2: return pick_strip<7, 2, 4, 3>(a, s);
        default: return hipErrorNotSupported;
    }
}

}  // namespace sushi
