// Dense convolution and fully connected layers with few pixels (one image, per-image vectors), bf16, int8 and all of the
// float32 mode, on the matrix cores: latency decides, so a layer is spread over as many waves as it has work for.
//
// A workgroup computes 16 filters x 16 pixels; its WK = blockDim.x / 64 waves (chosen by the host) share the reduction.
// The reduction is one flat sequence of 16-byte cells, k = tap * (cells per tap) + cell; a step is four cells, one matrix
// instruction (16x16x32_bf16, 16x16x64_i8; four 16x16x4_f32), and wave w takes steps w, w + WK, ...  Operands come straight
// from memory in operand order, U steps in flight in registers: a step's registers are requested again as soon as it is
// multiplied.  Every load is issued on every path, past the end of the buffer where there is nothing to load (zeros arrive):
// a load under a branch would make the wait for one step a wait for all of them.  The partial sums are added in the order
// of the waves through LDS; the epilogue's constants and the residual are requested behind the first U steps.
//
// Bound by the number of serial load rounds and, with many tiles, by the activation gather (a wave load touches 16 pixels'
// cache lines) and the index arithmetic of a step.  Consecutive tiles run on one XCD and share the weight tile in its L2.
#include "kernels.h"
#include "device_common.h"

#include <algorithm>
#include <type_traits>

namespace sushi {

typedef __attribute__((ext_vector_type(4))) unsigned cs_u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned cs_u32x2;
typedef __attribute__((ext_vector_type(4))) int cs_i32x4;

struct SmallGeom {
    int tiles_f, tiles_m;
    int M;        // B * P * Q
    int kcells;   // cells of the reduction: taps * cells per tap
    int nsteps;   // steps of four cells
    FastDiv dq, dp, dcell, dr;  // division by Q, P, cells per tap, taps per row
};

// IN32: the input is a float32 vector per image (H = W = 1): every value is split into two bf16 terms, x = hi + lo with
// hi = bf16(x) and lo = bf16(x - hi), and both are multiplied with the same weight operand, so the product carries about
// 16 bits of the input's mantissa instead of 8.
// ST_F32: the float32 mode; a cell is half a stored group of eight channels, four v_mfma_f32_16x16x4_f32 per step (float32
// products and sums; which channel a lane holds does not matter as long as both operands agree).
// ST_GATED: bf16, 1x1; every operand cell is multiplied by its image's gates (float32) and rounded to bf16 again, which is what a
// pass over the map would have stored.
enum SmallType { ST_BF16, ST_IN32, ST_I8, ST_F32, ST_GATED };

template <int U, SmallType TYPE>
__global__ __launch_bounds__(TYPE == ST_F32 ? 512 : 256) void conv_small_kernel(ConvArgs a, SmallGeom g, QuantArgs q) {
    constexpr bool IN32 = TYPE == ST_IN32, I8 = TYPE == ST_I8, F32 = TYPE == ST_F32, GATED = TYPE == ST_GATED;
    extern __shared__ float cs_red[];  // [WK][4][64]
    const int WK = blockDim.x >> 6, lane = threadIdx.x & 63;
    const int wk = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    const int ntiles = g.tiles_f * g.tiles_m, per_xcd = (ntiles + 7) >> 3;
    const int tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (tile >= ntiles) return;
    const int tf = tile / g.tiles_m, f0 = tf * 16, m0 = (tile - tf * g.tiles_m) * 16, m = m0 + l16;  // (m: this lane's pixel)
    constexpr int CPC = I8 ? 16 : F32 ? 4 : 8, ES = IN32 ? 4 : 16 / CPC;  // channels per cell, bytes per element
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<void *>(a.x), 0, (int)((long)a.B * a.H * a.W * a.C * ES), 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<void *>(a.w), 0, (int)((long)a.R * a.R * a.CG * a.Kpad * (F32 ? 32 : 16)), 0x00020000);

    const bool live = m < g.M;
    const int pq = fdiv(live ? m : 0, g.dq), qq = (live ? m : 0) - pq * a.Q;
    const int n = fdiv(pq, g.dp), pp = pq - n * a.P;
    const int h0 = pp * a.stride - a.pad, w0 = qq * a.stride - a.pad;
    const unsigned boff = (unsigned)(((n * a.H + h0) * a.W + w0) * a.C * ES);
    const unsigned woff = (unsigned)(f0 + l16) * (F32 ? 32 : 16);  // (filters are padded to 16)
    const __amdgpu_buffer_rsrc_t rg =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(q.gate), 0, GATED ? a.B * a.C * 4 : 0, 0x00020000);
    const unsigned goff = (unsigned)(n * a.C) * 4u;
    cs_u32x4 rb[U], rb2[IN32 ? U : 1], ra[U], rg0[GATED ? U : 1], rg1[GATED ? U : 1];
    unsigned in[U];  // int8: bit 0: the cell holds image; bit 8: a cell of the reduction; bit 9: its upper half is beyond C
    auto load_step = [&](int step, int u) {
        const int k = step * 4 + kg;
        const int tap = fdiv(k, g.dcell), cg = k - tap * g.dcell.d;
        const int dr = fdiv(tap, g.dr), ds = tap - dr * a.R;
        const unsigned off = ((unsigned)(dr * a.W + ds) * (unsigned)a.C + (unsigned)cg * CPC) * ES;
        const unsigned wcell = F32 ? (unsigned)(tap * a.CG + (cg >> 1)) * (unsigned)a.Kpad * 32 + (cg & 1) * 16
                                   : (unsigned)(tap * a.CG + cg) * (unsigned)a.Kpad * 16;
        const bool kv = k < g.kcells;
        const bool ok = kv & live & ((unsigned)(h0 + dr) < (unsigned)a.H) & ((unsigned)(w0 + ds) < (unsigned)a.W);
        ra[u] = __builtin_amdgcn_raw_buffer_load_b128(rw, offset_if(kv, woff + wcell), 0, 0);
        rb[u] = __builtin_amdgcn_raw_buffer_load_b128(rx, offset_if(ok, boff + off), 0, 0);
        if (IN32) rb2[IN32 ? u : 0] = __builtin_amdgcn_raw_buffer_load_b128(rx, offset_if(ok, boff + off + 16), 0, 0);
        if (GATED) {
            rg0[GATED ? u : 0] = __builtin_amdgcn_raw_buffer_load_b128(rg, offset_if(ok, goff + (unsigned)cg * 32u), 0, 0);
            rg1[GATED ? u : 0] = __builtin_amdgcn_raw_buffer_load_b128(rg, offset_if(ok, goff + (unsigned)cg * 32u + 16u), 0, 0);
        }
        in[u] = (ok ? 1u : 0u) | (kv ? 256u : 0u) | (cg * CPC + 8 >= a.C ? 512u : 0u);
    };
#pragma unroll
    for (int u = 0; u < U; ++u) load_step(wk + u * WK, u);
    // what the epilogue needs, requested by every wave (nothing arrives at those that do not finish the tile), behind the
    // operands: constants of the lane's four filters, four values of the residual
    const int fb = f0 + kg * 4;
    const bool last = wk == 0;
    cs_u32x4 cst[I8 ? 4 : 2];
    {
        const void *const src[4] = {I8 ? (const void *)q.qmult : (const void *)a.scale, I8 ? (const void *)q.qshift : (const void *)a.shift, q.qbias, q.wsum};
#pragma unroll
        for (int i = 0; i < (I8 ? 4 : 2); ++i)
            cst[i] = __builtin_amdgcn_raw_buffer_load_b128(
                __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(src[i]), 0, src[i] ? a.K * 4 : 0, 0x00020000), offset_if(last, (unsigned)fb * 4), 0, 0);
    }
    const bool vec = (a.K & 3) == 0;
    constexpr int OS = F32 ? 4 : I8 ? 1 : 2;  // bytes per element of the residual
    cs_u32x4 res = {0u, 0u, 0u, 0u};
    {
        const int rows = min(16, g.M - m0);  // (the tile's own: a residual may be larger than a buffer can be)
        const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char *>(static_cast<const char *>(a.res)) + (a.res ? (long)m0 * a.K * OS : 0), 0, a.res && vec ? rows * a.K * OS : 0, 0x00020000);
        const int o = offset_if(last & (fb < a.K), (unsigned)((l16 * a.K + fb) * OS));
        if constexpr (F32) {
            res = __builtin_amdgcn_raw_buffer_load_b128(rr, o, 0, 0);
        } else if constexpr (I8) {
            res[0] = __builtin_amdgcn_raw_buffer_load_b32(rr, o, 0, 0);
        } else {
            const cs_u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rr, o, 0, 0);
            res[0] = v[0], res[1] = v[1];
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    typedef typename std::conditional<I8, cs_i32x4, f32x4_t>::type acc_t;
    acc_t acc = acc_t{0, 0, 0, 0};
    const unsigned zfill = (unsigned)(q.zx & 0xFF) * 0x01010101u;
    auto multiply = [&](int u) {
        if constexpr (I8) {
            // a cell of the frame holds the code of the real value 0 (the input's zero point) in its active channels,
            // the upper half of a cell that straddles the SubNet's channel count zeros
            cs_u32x4 b = rb[u];
            if ((in[u] & 256u) && !(in[u] & 1u)) b = cs_u32x4{zfill, zfill, zfill, zfill};
            if (in[u] & 512u) b[2] = 0u, b[3] = 0u;
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(cs_i32x4, ra[u]), __builtin_bit_cast(cs_i32x4, b), acc, 0, 0, 0);
        } else if constexpr (F32) {
            const f32x4_t w = __builtin_bit_cast(f32x4_t, ra[u]), x = __builtin_bit_cast(f32x4_t, rb[u]);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i], x[i], acc, 0, 0, 0);
        } else if constexpr (IN32) {
            const bf16x8_t w = __builtin_bit_cast(bf16x8_t, ra[u]);
            Frag hi, lo;
            split_f32x8(__builtin_bit_cast(uint4, rb[u]), __builtin_bit_cast(uint4, rb2[u]), &hi.u, &lo.u);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, hi.v, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, lo.v, acc, 0, 0, 0);
        } else {
            const cs_u32x4 b = GATED ? gate_cell(rb[u], rg0[GATED ? u : 0], rg1[GATED ? u : 0]) : rb[u];
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, ra[u]), __builtin_bit_cast(bf16x8_t, b), acc, 0, 0, 0);
        }
    };
    // rounds of U steps; the steps of the last round have no successor
    int step = wk;
    for (; step + U * WK < g.nsteps; step += U * WK) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            multiply(u);
            load_step(step + (U + u) * WK, u);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) multiply(u);  // (steps past the end multiply zeros)

    if (WK > 1) {
        reinterpret_cast<acc_t *>(cs_red)[wk * 64 + lane] = acc;
        __syncthreads();
        if (wk != 0) return;
        acc = acc_t{0, 0, 0, 0};
        for (int k = 0; k < WK; ++k) acc += reinterpret_cast<const acc_t *>(cs_red)[k * 64 + lane];
    }
    if (fb >= a.K || !live) return;
    const long o = (long)m * a.K + fb;
    if constexpr (I8) {  // (K is a multiple of 4)
        const int lo = a.act == 1 ? q.zy : -128;
        unsigned packed = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // (the zero-point term goes to the bias: minus z_x times the sum of the active weights)
            const int bias = (int)cst[I8 ? 2 : 0][i] - q.zx * (int)cst[I8 ? 3 : 0][i];
            long long t64 = rr64((long long)(acc[i] + bias) * (long long)(int)cst[0][i], (int)cst[1][i]);
            if (a.res) t64 += rr64((long long)((int)(int8_t)(res[0] >> (8 * i)) - q.z_res) * (long long)q.m_res, q.sh_res);
            t64 += q.zy;
            const int c = (int)(t64 < lo ? lo : t64 > 127 ? 127 : t64);
            packed |= (unsigned)(c & 0xFF) << (8 * i);
        }
        *reinterpret_cast<unsigned *>(static_cast<int8_t *>(a.y) + o) = packed;
    } else {
        const f32x4_t sc = a.scale ? __builtin_bit_cast(f32x4_t, cst[0]) : f32x4_t{1.f, 1.f, 1.f, 1.f}, sh = __builtin_bit_cast(f32x4_t, cst[1]);
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = acc[i] * sc[i] + sh[i];
        if (a.res) {
            if (!vec) {
                for (int i = 0; i < min(4, a.K - fb); ++i) v[i] += F32 ? static_cast<const float *>(a.res)[o + i] : bf2f(static_cast<const uint16_t *>(a.res)[o + i]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] += F32 ? __uint_as_float(res[i]) : bf2f(i & 1 ? res[i >> 1] >> 16 : res[i >> 1] & 0xFFFFu);
            }
        }
        with_activation(a.act, a.hsigmoid, [&](auto act) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = activate_as<decltype(act)::value>(v[i]);
        });
        if (F32 || a.out_f32) {
            float *yp = static_cast<float *>(a.y) + o;
            if (vec)
                *reinterpret_cast<float4 *>(yp) = make_float4(v[0], v[1], v[2], v[3]);
            else
                for (int i = 0; i < min(4, a.K - fb); ++i) yp[i] = v[i];
        } else {
            uint16_t *yp = static_cast<uint16_t *>(a.y) + o;
            if (vec)
                *reinterpret_cast<uint2 *>(yp) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
            else
                for (int i = 0; i < min(4, a.K - fb); ++i) yp[i] = (uint16_t)f2bf(v[i]);
        }
    }
}

template <SmallType TYPE>
static hipError_t launch_small(const ConvArgs &a, const QuantArgs &q, hipStream_t s) {
    constexpr int U = 4, CPC = TYPE == ST_I8 ? 16 : TYPE == ST_F32 ? 4 : 8;  // (two steps in flight cost up to 1 us)
    SmallGeom g;
    g.M = a.B * a.P * a.Q;
    g.tiles_f = (a.K + 15) / 16, g.tiles_m = (g.M + 15) / 16;
    const int cells = (a.C + CPC - 1) / CPC;
    g.kcells = a.R * a.R * cells, g.nsteps = (g.kcells + 3) / 4;
    g.dq = make_fastdiv(a.Q), g.dp = make_fastdiv(a.P), g.dcell = make_fastdiv(cells), g.dr = make_fastdiv(a.R);
    // Waves per tile, each with at least one round of U steps: four.  More shorten the chain of rounds, but take the places of
    // other tiles and have a longer sum through LDS.  4, 8, 16 waves, us: 7 x 7 x 720 3x3, 180 tiles of 203 steps, 9.2, 9.6, 10.4;
    // 3 x 7 x 7 x 720, 450 tiles, 12.6, 12.6, 13.2; 16 x 7 x 7 x 264, 833 tiles of 75 steps, 9.6, 10.4, 12.1; over 330 layers of
    // both precisions 3167, 3224, 3324.  Float32, four times the matrix instructions per step: eight up to 1024 tiles.
    int wk = std::max(1, std::min((g.nsteps + U - 1) / U, TYPE == ST_F32 && (long)g.tiles_m * g.tiles_f <= 1024 ? 8 : 4));
    const int per_xcd = (int)(((long)g.tiles_m * g.tiles_f + 7) / 8);
    while (wk > 1 && (long)per_xcd * 8 * 64 * wk >= 1l << 32) --wk;  // (a launch has fewer than 2^32 threads)
    const size_t lds = wk > 1 ? (size_t)wk * 1024 : 0;
    hipLaunchKernelGGL((conv_small_kernel<U, TYPE>), dim3(per_xcd * 8), dim3(64 * wk), lds, s, a, g, q);
    return hipGetLastError();
}

static bool small_fits(const ConvArgs &a, long es) {
    const long lim = (1l << 31) - 256;
    return a.C >= 8 && (a.C & 7) == 0 && (long)a.B * a.P * a.Q < lim && (long)a.B * a.H * a.W * a.C * es < lim &&
           (long)a.R * a.R * a.CG * a.Kpad * (es == 4 && !a.in_f32 ? 32 : 16) < lim && ((a.K + 15) / 16) * (((long)a.B * a.P * a.Q + 15) / 16) < (1l << 26) - 8;
}

bool conv_small_covers(const ConvArgs &a) { return !a.in_f32 && small_fits(a, 2); }

hipError_t launch_conv_small(const ConvArgs &a, hipStream_t s, const float *gate) {
    if (!a.in_f32) {
        if (!small_fits(a, 2)) return hipErrorNotSupported;
        if (gate) {
            QuantArgs q{};
            q.gate = gate;
            return launch_small<ST_GATED>(a, q, s);
        }
        return launch_small<ST_BF16>(a, QuantArgs{}, s);
    }
    // float32 vectors: rows in pieces below 2 GiB
    if (a.H * a.W != 1 || a.res || !a.out_f32) return hipErrorInvalidValue;
    const long rows = ((1l << 31) - 4096) / ((long)a.C * 4);
    ConvArgs part = a;
    for (long n = 0; n < a.B; n += rows) {
        part.B = (int)std::min(rows, a.B - n);
        part.x = static_cast<const float *>(a.x) + n * a.C;
        part.y = static_cast<float *>(a.y) + n * a.K;
        if (!small_fits(part, 4)) return hipErrorInvalidValue;
        const hipError_t e = launch_small<ST_IN32>(part, QuantArgs{}, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_conv_small_f32(const ConvArgs &a, hipStream_t s) {
    if (!small_fits(a, 4)) return hipErrorNotSupported;
    return launch_small<ST_F32>(a, QuantArgs{}, s);
}

hipError_t launch_conv_small_i8(const ConvArgs &a, const QuantArgs &q, hipStream_t s) {
    if (!small_fits(a, 1) || (a.K & 3)) return hipErrorInvalidValue;
    return launch_small<ST_I8>(a, q, s);
}

}  // namespace sushi
