// Device kernels of the SubNet forward pass and their launchers (gfx950).
//
// Layouts
//   activations   [B][H][W][C]  channels fastest, C = active channels of the SubNet (compact)
//   dense weights [tap][channel group of 8][filter (padded to 16)][8 channels]
//                 so the slice (K' filters, C' channels) of a SubNet is, for every tap and channel
//                 group below C'/8, the contiguous prefix of K' * 8 elements; a 16-filter x 32-channel
//                 matrix-core operand is four 256-byte runs
//   depthwise     [tap in ring order][channel]: the 9 taps of the centre 3x3 first, then the 16 of
//                 the 5x5 ring, then the 24 of the 7x7 ring, so a centred k x k crop is the prefix
//                 of k*k taps
//   scale/shift   float32 prefixes of length K'
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

namespace sushi {

// Raises a kernel's limit of dynamic LDS to all a compute unit has, once per device (the limit belongs to a kernel on one
// device); what fails is tried again by the next launch.  One static object per kernel; any number of threads.
class LdsLimit {
    std::atomic<uint64_t> raised_{0};  // bit d: done on device d

public:
    template <typename Kernel>
    hipError_t raise(Kernel kernel) {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;  // (beyond 64 devices: by every launch)
        if (raised_.load(std::memory_order_acquire) & bit) return hipSuccess;
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e == hipSuccess)
            raised_.fetch_or(bit, std::memory_order_release);
        else
            (void)hipGetLastError();  // (reported here; the next launch must not find it)
        return e;
    }
};

// Division of a non-negative int below 2^31 by a fixed divisor d: n / d = mulhi(n, mul) >> shr for d > 1
// (mul = ceil(2^(31 + ceil(log2 d)) / d) fits 32 bits), n itself for d = 1 (mul = shr = 0, one = all bits; no branch).  The
// host prepares (mul, shr, one).
struct FastDiv {
    unsigned mul, shr, one;
    int d;
};

__host__ inline FastDiv make_fastdiv(int d) {
    FastDiv f{0u, 0u, d > 1 ? 0u : ~0u, d};
    if (d > 1) {
        int lg = 0;
        while ((1ll << lg) < d) ++lg;
        const int p = 31 + lg;
        f.mul = (unsigned)(((1ull << p) + (unsigned long long)d - 1) / (unsigned long long)d);
        f.shr = (unsigned)(p - 32);
    }
    return f;
}

// Order of a dense layer's tiles: consecutive tiles run on one XCD (one of eight equal ranges each).  With pixels fast an XCD reads
// the whole input and an eighth of the weights, with filters fast an eighth of the input and all weights.
struct TileOrder {
    int filters_fast;
    FastDiv fast;  // division by the tiles along the fast axis
};

struct ConvArgs {
    const void *x;       // input activations
    void *y;             // output activations
    const void *res;     // optional residual, same shape as y
    const void *w;       // packed weights of the layer
    const float *scale;  // may be null (= 1)
    const float *shift;  // shift or bias
    int B, H, W, C;      // input
    int P, Q, K;         // output
    int R, stride, pad;  // taps per side of the active kernel
    int Rmax;            // taps per side of the stored kernel (depthwise crops)
    int Kpad, CG;        // packed layout: padded filters, stored channel groups
    int act;             // sushi_act; applied after the residual add
    int hsigmoid;        // replace act by min(max(v+3,0),6)/6
    int out_f32;         // store float32 regardless of the activation type
    int in_f32;          // bf16 mode: the input is a float32 vector per image (pooled features, squeeze-excite and
                         // head vectors); the kernels split it into two bf16 terms (value = hi + lo) on the fly
};

// 1x1 expansion and the depthwise layer behind it (expand_dw.hip).
struct ExpandDwArgs {
    const void *x;          // [B][H][W][C]
    void *y;                // [B][P][Q][K]
    const void *w1, *w2;    // packed dense and depthwise weights
    const float *scale1, *shift1, *scale2, *shift2;
    float *pool;            // [B][ExpandDwGeom::parts][K] partial sums of the output over an image, or null
    int B, H, W, C, K, P, Q;
    int R, stride;          // of the depthwise layer
    int Kpad1, Kpad2, act;  // (the same activation behind both)
};

// How a layer pair is cut into tiles; depends on the shapes alone.
struct ExpandDwGeom {
    int tx, ty;           // tiles of an image along x and y
    int bx, by, im;       // blocks of a tile along x and y, images of a tile (several only where an image is one tile)
    int ns, ng;           // matrix columns set aside for an image; groups of 16 columns
    int rp, rh, pp;       // plane: bytes of a row, rows of an image, bytes in all
    int r0, rows, qw;     // first row of an image's region that may lie in the image, how many; quads of a row
    int nq;               // quads of a tile
    int total, workers;   // tiles over all images; workgroups that share them (times channel blocks)
    int groups;           // channel blocks
    int parts;            // of ExpandDwArgs::pool
    int out, tab;         // LDS offsets of the outputs (first: the taps) and of the tables
    FastDiv dqw, drows, dper, dtx, dbx, dtw, dth;  // division by qw, rows, tx * ty, tx, bx, outputs of a tile's row, of its column
};

// The two fully connected layers of a squeeze-excite block (squeeze_excite.hip).
struct SeGateArgs {
    const float *pooled;  // [B][parts][C]: their sum over the parts, times inv, is the block's input
    const void *w1, *w2;  // packed bf16 weights [cell of 8 inputs][filter (padded)][8]
    const float *b1, *b2;
    float *gate;  // [B][C]
    int B, C, red, Kpad1, Kpad2, parts;
    float inv;
};

// What an int8 layer needs beyond ConvArgs / PoolArgs (int8.hip), and the gates of a bf16 layer.  An int8 layer's weights are
// [tap][channel group of 16][filter (padded to 16)][16] and ConvArgs::CG counts the stored groups of 16.
struct QuantArgs {
    const int32_t *qmult;   // per filter: requantisation multiplier (classifier: bit pattern of a float32 factor)
    const int32_t *qshift;  // per filter: rounding right shift
    const int32_t *qbias;   // per filter: added to the accumulator
    const int32_t *wsum;    // per filter: sum of the active slice's weights over taps and channels (zero-point term)
    int zx, zy;             // zero points of the input and the output tensor (pooling: zx of the pooled map)
    int m_res, sh_res, z_res;  // residual: multiplier, shift, zero point
    int pool_hw;            // classifier: pixels the pooling before it summed over
    const float *gate;      // (bf16, 1x1: [B][C] multipliers of the input, value * gate rounded to bf16; null: none)
};

struct PoolArgs {
    const void *x;
    void *y;
    const float *gate;  // OP_GATE: [B][C] multipliers
    int B, H, W, C, P, Q;
    int out_f32;        // OP_GAP in bf16 mode: store the averages as float32
};

inline TileOrder tile_order(bool filters_fast, int tiles_f, int tiles_m) {
    return TileOrder{filters_fast ? 1 : 0, make_fastdiv(filters_fast ? tiles_f : tiles_m)};
}

// Kernel families, for per-kernel accounting.
enum KernelClass {
    KC_CONV_DIRECT = 0,   // conv_direct_kernel
    KC_CONV_MFMA = 1,     // conv_mfma_kernel
    KC_CONV_SMALL = 2,    // conv_small_kernel
    KC_DW_ROWS = 3,       // dwconv_rows_kernel
    KC_MAXPOOL = 4,
    KC_GAP = 5,
    KC_GATE = 6,
    KC_STREAM = 7,  // sushi_stream_kernel (one launch per query)
    KC_TEAM = 8,    // sushi_team_kernel (persistent; one launch serves many queries)
    KC_CONV_PATCH = 9,  // conv_patch_kernel (large pixel counts; the input patch of a tile staged in LDS)
    KC_CONV_I8_DIRECT = 10,  // conv_i8_direct_kernel (int8: the input layer)
    KC_I8_OTHER = 11,   // int8 mode: max-pool, pooled sums, classifier
    KC_STEM = 12,       // stem_mfma_kernel (bf16: the 3-channel input layer)
    KC_CONV_TILE = 13,  // conv_tile_kernel (64-filter tiles, the reduction split over wave groups)
    KC_DW_MFMA = 14,    // dw_mfma_kernel (depthwise on the matrix cores)
    KC_DW = 15,         // dwconv_kernel (depthwise: float32, and tensors of 2 GiB and more)
    KC_SE_GATE = 16,    // se_gate_kernel (both fully connected layers of a squeeze-excite block)
    KC_EXPAND_DW = 17,  // expand_dw_kernel (1x1 expansion and depthwise layer)
    KC_CONV_KSPLIT = 18,  // conv_ksplit_kernel (3x3, the reduction split over the waves of a workgroup)
    KC_COUNT = 19
};
const char *kernel_class_name(int kc);

// Every launcher returns hipSuccess or the launch error.  bf16 = activations and weights are bf16.
// Launchers that choose between kernels report the family they picked in *kc.
// patch_min_pixels: dense 1x1 / 3x3 layers with at least that many output pixels (B * P * Q) go to the patch
// kernel (conv_patch.hip) where it covers the shape; 0 = never; PATCH_AUTO: from 3136 pixels on where it is the fastest.
constexpr long PATCH_AUTO = -1;
inline bool patch_from(long min_pixels, long pixels, bool long_reduction) {
    const long n = min_pixels == PATCH_AUTO ? 3136 : min_pixels;
    return n > 0 && pixels >= n && (pixels >= 4 * n || long_reduction);
}
// finite_w: the layer's weights are all finite; if not, float32 layers and the input layer run in the kernel that skips
// taps outside the image (in the others zero meets the tap's weight, and zero times infinity is NaN).
hipError_t launch_conv(const ConvArgs &a, bool bf16, hipStream_t s, int *kc, long patch_min_pixels, bool finite_w);  // dense conv and FC
hipError_t launch_gated_conv(const ConvArgs &a, const float *gate, hipStream_t s, int *kc);  // (gated_conv_covers)

// Dense 1x1 (stride 1) and 3x3 (stride 1 or 2) convolution, bf16, C and K multiples of 8, tensors below 2 GiB: the
// patch kernel (conv_patch.hip).  Returns hipErrorNotSupported (nothing launched) for any other case.
hipError_t launch_conv_patch(const ConvArgs &a, hipStream_t s);
int conv_patch_tile_filters(int K);  // filters of one of its tiles for a layer of K filters

// Dense 1x1 and 3x3 convolution (stride 1 or 2), C and K multiples of 8, tensors below 2 GiB: the tile kernel
// (conv_tile.hip).  patch: the patch kernel would take the layer otherwise.  Returns hipErrorNotSupported (nothing
// launched) for any other case and where another kernel is the faster one.
hipError_t launch_conv_tile(const ConvArgs &a, hipStream_t s, bool patch, const float *gate = nullptr);
bool conv_tile_gated_covers(const ConvArgs &a);
hipError_t launch_conv_tile_i8(const ConvArgs &a, const QuantArgs &q, hipStream_t s, bool patch);

// 3x3 with stride 1 and long reductions, which the waves of a workgroup split (conv_ksplit.hip); patch as above.  Returns
// hipErrorNotSupported (nothing launched) for any other case and where another kernel is the faster one.
hipError_t launch_conv_ksplit(const ConvArgs &a, hipStream_t s, bool patch);
hipError_t launch_conv_ksplit_i8(const ConvArgs &a, const QuantArgs &q, hipStream_t s, bool patch);

// Dense convolution of few pixels and fully connected layers, C a multiple of 8 (conv_small.hip).  bf16 and float32:
// return hipErrorNotSupported (nothing launched) for tensors of 2 GiB and more.
hipError_t launch_conv_small(const ConvArgs &a, hipStream_t s, const float *gate = nullptr);
bool conv_small_covers(const ConvArgs &a);  // (bf16)
hipError_t launch_conv_small_f32(const ConvArgs &a, hipStream_t s);  // the float32 mode
hipError_t launch_conv_small_i8(const ConvArgs &a, const QuantArgs &q, hipStream_t s);
bool conv_small_is_faster(const ConvArgs &a, bool i8);  // than the tile kernel (conv_tile.hip)

// Squeeze-excite in two launches behind the pooling: the gates (squeeze_excite.hip), then the 1x1 layer behind the block with
// its gates (conv_small.hip, conv_tile.hip).  The covers functions say whether a layer can go that way.
bool se_gate_covers(const SeGateArgs &a);
hipError_t launch_se_gate(const SeGateArgs &a, hipStream_t s);
bool gated_conv_covers(const ConvArgs &a);

// An inverted-residual block's expansion and depthwise layer in one launch (expand_dw.hip).
bool expand_dw_covers(const ExpandDwArgs &a);
ExpandDwGeom expand_dw_geom(const ExpandDwArgs &a);
hipError_t launch_expand_dw(const ExpandDwArgs &a, const ExpandDwGeom &g, hipStream_t s);

// 3x3 convolution of a 3-channel bf16 image (stem.hip).  Returns hipErrorNotSupported (nothing launched) for any
// other case.
hipError_t launch_stem(const ConvArgs &a, hipStream_t s);
hipError_t launch_dwconv(const ConvArgs &a, bool bf16, hipStream_t s, int *kc);
hipError_t launch_maxpool(const PoolArgs &a, bool bf16, hipStream_t s);   // 3x3 stride 2 pad 1
hipError_t launch_gap(const PoolArgs &a, bool bf16, hipStream_t s);       // [B][H][W][C] -> [B][C]
hipError_t launch_gate(const PoolArgs &a, bool bf16, hipStream_t s);      // y = x * gate[b][c]

// Depthwise k x k, k in {3, 5, 7}, stride 1 or 2, bf16, tensors below 2 GiB: the row-strip kernel (dwconv.hip).
// Returns hipErrorNotSupported (nothing launched) for any other case.
hipError_t launch_dwconv_rows(const ConvArgs &a, hipStream_t s);

// The same on the matrix cores, kernels 5x5 and 7x7 and small 3x3 layers (dwconv_mfma.hip).  Returns
// hipErrorNotSupported (nothing launched) for any other case.
hipError_t launch_dwconv_mfma(const ConvArgs &a, hipStream_t s);

// int8 mode (int8.hip): dense conv 1x1 / 3x3 on the int8 matrix cores (3 input channels: vector ALUs) with integer
// requantisation, 3x3/2 max-pool on codes, exact int32 pooled sums, int64 classifier with float32 logits.
hipError_t launch_conv_i8(const ConvArgs &a, const QuantArgs &q, hipStream_t s, int *kc, long patch_min_pixels);
hipError_t launch_conv_patch_i8(const ConvArgs &a, const QuantArgs &q, hipStream_t s);  // conv_patch.hip
hipError_t launch_fc_i8(const ConvArgs &a, const QuantArgs &q, hipStream_t s);
hipError_t launch_maxpool_i8(const PoolArgs &a, hipStream_t s);
hipError_t launch_gap_i8(const PoolArgs &a, const QuantArgs &q, hipStream_t s);

// Streams `bytes` of `buf` through the caches (reads every 16-byte word once; `sink` receives one word that
// depends on all of them, so the reads cannot be dropped).  A measurement aid: see SUSHI_OPT_COLD_SWEEP_MIB.
hipError_t launch_cold_sweep(const void *buf, size_t bytes, void *sink, hipStream_t s);

// The library's static scratch buffer on the current device: STATIC_SCRATCH_BYTES of device memory that
// belong to the loaded code object (no allocation), for sushi_infer_static.  The address is looked up once
// per device, with that device current.
constexpr size_t STATIC_SCRATCH_BYTES = 16u << 20;
hipError_t static_scratch(int device, void **ptr);

// Ring order of depthwise taps: tap t of a 7x7 kernel sits at row/col offset (dr, ds) from the centre.
void dw_tap_offsets(int t, int *dr, int *ds);
hipError_t upload_tap_table();

}  // namespace sushi
