"""The per-layer kernels at the edges of their tiles, through small SuperNets built for it, against the CPU oracle.

Where a kernel has no float32 or int8 variant the comparison is exact (small integers, see test_input_layer_exact); that
the nets reach the kernels they are meant for is checked in test_host_launches.py.

bf16 tolerance: every stored feature map is rounded to bf16 on both sides (relative error 2^-9 at most per value, at
random), and a rounding that falls the other way moves a value by 2^-8; averaged over a map and summed over the channels
of a classifier that stays below 2^-8 = 3.9e-3 of the logits for nets of a few layers."""
import dataclasses

import numpy as np
import pytest
import torch

from tests.common import make_problem, oracle_logits_bf16_stores, rel_l2
from workloads import arch as A
from workloads import tensors as T

pytestmark = pytest.mark.gpu

BF16_TOL = 2.0 ** -8


def _check(arch, cfg, batch, seed, tol, bf16=True):
    import paper_2306_17266_amd as S
    from oracle import subnet_eval as E
    blob, wts = make_problem(arch, seed, bf16)
    ctx = S.Sushi(0)
    ctx.sushi_load_supernet(arch, blob, S.BF16 if bf16 else S.FP32)
    x = T.make_input(seed, 0, batch, cfg.resolution, arch.in_channels, bf16)
    xd = torch.from_numpy(x).cuda()
    xd = xd.to(torch.bfloat16) if bf16 else xd
    logits = torch.full((batch, arch.n_classes), float("nan"), device="cuda", dtype=torch.float32)
    ctx.sushi_infer(cfg, xd.contiguous(), logits)
    torch.cuda.synchronize()
    ctx.close()
    want = oracle_logits_bf16_stores(arch, wts, cfg, x) if bf16 else E.forward(
        arch, wts, cfg, np.ascontiguousarray(x.transpose(0, 3, 1, 2)))
    for n in range(batch):
        assert rel_l2(logits[n].cpu().numpy(), want[n]) <= tol, n


def _chain(widths, res, classes=64, channels=3):
    """A Tiny-family net: 3x3 layers (stride 1) of the given widths, pooling, classifier."""
    n = len(widths)
    return dataclasses.replace(A.tiny_arch(), n_classes=classes, in_channels=channels, stage_base_out=list(widths),
                               stage_stride=[1] * n, stage_max_depth=[1] * n, stage_act=[A.ACT_RELU] * n,
                               stage_se=[0] * n, depth_drop_choices=[0], width_choices=[1.0], res_choices=[res])


# odd sizes: patch rows that start on odd elements, tensors of an odd number of elements (the general kernel), columns
# outside on either side; 15 x 15 = one pixel short of a tile; widths of half a filter tile, a ragged one, several groups
@pytest.mark.parametrize("res,width,batch", [(8, 8, 1), (9, 24, 2), (9, 16, 1), (15, 32, 4), (33, 40, 2), (31, 72, 3), (12, 16, 6), (224, 16, 4)])
def test_input_layer(res, width, batch):
    arch = _chain([width, 16], res)
    _check(arch, A.max_cfg(arch), batch, 41, BF16_TOL)


# A weight of minus infinity and an input above 0: minus infinity, ReLU'd to 0, wherever its tap lies inside the image, and
# outside it the tap is no part of the sum.  The oracle gets a large finite weight instead.  Input layer and float32 layers.
@pytest.mark.parametrize("bf16,layer", [(True, 0), (False, 0), (False, 1)])
def test_infinite_weight_outside_the_image(bf16, layer):
    import paper_2306_17266_amd as S
    from oracle import subnet_eval as E
    arch = _chain([8, 16], 8)
    cfg = A.max_cfg(arch)
    table = S.sushi_describe_supernet(arch)

    def tensors(weight):
        tens = T.make_weights([(s, k) for _, s, k in table], 59, bf16)
        for (name, _, _), t in zip(table, tens):
            if name == "conv%d.w" % layer:
                t[:4, 0, 0, 0] = weight
            elif name == "conv0.shift":
                t[:] = 20.0 if layer == 1 else t  # (its output is above 0 everywhere)
        return tens

    x = np.abs(T.make_input(59, 0, 2, 8, 3, bf16)) + np.float32(0.25)
    x = T.round_to_bf16(x) if bf16 else x
    wts = E.name_weights(arch, tensors(-1e30))
    want = oracle_logits_bf16_stores(arch, wts, cfg, x) if bf16 else E.forward(arch, wts, cfg, np.ascontiguousarray(x.transpose(0, 3, 1, 2)))
    ctx = S.Sushi(0)
    ctx.sushi_load_supernet(arch, T.flatten(tensors(-np.inf)), S.BF16 if bf16 else S.FP32)
    xd = torch.from_numpy(x).cuda()
    logits = torch.full((2, arch.n_classes), float("nan"), device="cuda", dtype=torch.float32)
    ctx.sushi_infer(cfg, xd.to(torch.bfloat16) if bf16 else xd, logits)
    torch.cuda.synchronize()
    ctx.close()
    assert rel_l2(logits.cpu().numpy(), want) <= (BF16_TOL if bf16 else 1e-5)


def _mobile(expand, kernel, strides, act, res, out=16):
    """An inverted-residual net of one block per stage: stage widths `out`, one kernel size, no squeeze-excite."""
    n = len(strides)
    return dataclasses.replace(A.small_mbv3_arch(), stage_base_out=[out] * n, stage_stride=list(strides), stage_max_depth=[1] * n,
                               stage_act=[act] * n, stage_se=[0] * n, depth_drop_choices=[0], expand_choices=[float(expand)],
                               kernel_choices=[kernel], res_choices=[res], stem_out=out)


# channel counts of half a group of 16 (24), 40 and 144; maps narrower than a column tile, one column past it (34 -> 17), odd
# ones; one-row strips (one image) and long strips with a ragged last one (the large batches); both strides
@pytest.mark.parametrize("kernel", [3, 5, 7])
@pytest.mark.parametrize("expand,strides,res,batch,out", [(3, (1, 2), 8, 1, 8), (1, (2, 1), 34, 1, 40), (3, (1, 2), 30, 2, 48),
                                                          (3, (1, 2), 46, 24, 48)])
def test_depthwise(kernel, expand, strides, res, batch, out):
    arch = _mobile(expand, kernel, strides, A.ACT_HSWISH if kernel == 5 else A.ACT_RELU, res, out)
    _check(arch, A.max_cfg(arch), batch, 43, 2 * BF16_TOL)  # (twice the layers of the other nets)


# A channel whose expanded values overflow to infinity and whose depthwise weights are all negative: minus infinity, which
# ReLU makes 0.  The other channels must be what they are with that channel's map at 0.
@pytest.mark.parametrize("kernel", [3, 5, 7])
@pytest.mark.parametrize("strides,res,batch", [((1, 2), 8, 1), ((2, 1), 46, 24)])
def test_depthwise_keeps_channels_apart(kernel, strides, res, batch):
    import paper_2306_17266_amd as S
    arch = _mobile(1, kernel, strides, A.ACT_RELU, res, 40)
    cfg = A.max_cfg(arch)
    table = S.sushi_describe_supernet(arch)
    got = []
    for scale in (3e38, 0.0):
        tens = T.make_weights([(s, k) for _, s, k in table], 53, True)
        for (name, _, _), t in zip(table, tens):
            for block in ("s0b0.", "s1b0."):
                if name == block + "expand.scale":
                    t[[5, 38]] = scale
                elif name in (block + "expand.shift", block + "dw.shift"):
                    t[[5, 38]] = 0.0
                elif name == block + "dw.w":
                    t[[5, 38]] = -np.abs(t[[5, 38]]) - 0.01
        ctx = S.Sushi(0)
        ctx.sushi_load_supernet(arch, T.flatten(tens), S.BF16)
        x = torch.from_numpy(T.make_input(53, 0, batch, cfg.resolution, arch.in_channels, True)).cuda().to(torch.bfloat16)
        logits = torch.full((batch, arch.n_classes), float("nan"), device="cuda", dtype=torch.float32)
        ctx.sushi_infer(cfg, x, logits)
        torch.cuda.synchronize()
        ctx.close()
        got.append(logits.cpu().numpy())
    for n in range(batch):
        assert rel_l2(got[0][n], got[1][n]) <= 2 * BF16_TOL, n


def _bottleneck(widths, strides, res, expand, classes=64):
    """A bottleneck net of two blocks per stage (projection, then a residual from the block's input)."""
    n = len(widths)
    return dataclasses.replace(A.small_resnet_arch(), n_classes=classes, stage_base_out=list(widths), stage_stride=list(strides),
                               stage_max_depth=[2] * n, stage_act=[A.ACT_RELU] * n, stage_se=[0] * n, depth_drop_choices=[0],
                               width_choices=[1.0], expand_choices=[expand], res_choices=[res])


# The input layer and the depthwise kernels output by output.  Images and weights are small integers, scales 1 and shifts
# integers, every other layer copies its channels: all products, sums (below 256 per output, or even and below 512: the
# bf16 stores too) are exact whatever their order, and the logits are the channels' averages.  An average times its pixel count is an integer
# below 2^15, the head's two-term split of it carries 16 bits: rounded to the nearest it is the channel's exact sum.

def _exact(arch, weights, x):
    """weights(name, shape): integer tensors.  The logits of the library and of the oracle."""
    import paper_2306_17266_amd as S
    from oracle import subnet_eval as E
    cfg = A.max_cfg(arch)
    table = S.sushi_describe_supernet(arch)
    tens = [np.ascontiguousarray(weights(name, s), dtype=np.float32) for name, s, _ in table]
    want = E.forward(arch, E.name_weights(arch, tens), cfg, np.ascontiguousarray(x.transpose(0, 3, 1, 2)))
    ctx = S.Sushi(0)
    ctx.sushi_load_supernet(arch, T.flatten(tens), S.BF16)
    logits = torch.full(want.shape, float("nan"), device="cuda", dtype=torch.float32)
    ctx.sushi_infer(cfg, torch.from_numpy(x).cuda().to(torch.bfloat16), logits)
    torch.cuda.synchronize()
    ctx.close()
    return logits.cpu().numpy().astype(np.float64), np.asarray(want, dtype=np.float64)


def _copy(shape):
    """1x1 (or centre of a larger kernel): output channel k is input channel k modulo their count."""
    w = np.zeros(shape)
    for k in range(shape[0]):
        w[(k, k % shape[1]) + tuple(r // 2 for r in shape[2:])] = 1.0
    return w


# (resolution, stride, width, batch): patch rows from odd elements and columns outside on either side, tensors of an odd
# number of elements (the general kernel), 15 x 15 = one pixel short of a tile, widths of half a filter tile, a ragged one and
# several; from 131072 outputs on four pixel tiles per wave (134540 and 132940 end with a ragged one)
INPUT_LAYERS = [(8, 1, 8, 1), (9, 1, 24, 2), (9, 1, 16, 1), (15, 1, 32, 4), (33, 1, 40, 2), (31, 1, 72, 4), (31, 1, 16, 140), (33, 1, 40, 128),
                (8, 2, 8, 1), (9, 2, 24, 2), (9, 2, 16, 1), (30, 2, 32, 4), (33, 2, 40, 2), (31, 2, 72, 4), (12, 2, 16, 6), (33, 2, 16, 460), (33, 2, 40, 460)]


def input_layer_net(res, stride, width):
    """The input layer alone (stride 1), or before layers that copy its channels."""
    return _chain([width], res, width) if stride == 1 else dataclasses.replace(depthwise_net(3, 1, 4, width), res_choices=[res])


@pytest.mark.parametrize("res,stride,width,batch", INPUT_LAYERS)
def test_input_layer_exact(res, stride, width, batch):
    arch = input_layer_net(res, stride, width)
    rng = np.random.default_rng(61)
    x = rng.integers(-1, 3, (batch, res, res, 3)).astype(np.float32)

    def weights(name, shape):
        if name == "conv0.w":
            return rng.integers(-1, 2, shape)
        if name == "stem.w":
            return 3 * rng.integers(-1, 2, shape)  # (h-swish leaves 0 and multiples of 3 as they are, ReLU'd)
        if name.endswith(".scale"):
            return np.ones(shape)
        if name == "head.shift":
            return np.full(shape, 4.0)  # (h-swish again)
        return np.zeros(shape) if name == "first.pw.w" or not name.endswith(".w") else _copy(shape)

    got, want = _exact(arch, weights, x)
    pixels, shift = ((res - 1) // stride + 1) ** 2, 4.0 * (stride == 2)
    np.testing.assert_array_equal(np.rint((got - shift) * pixels), np.rint((want - shift) * pixels))


# (map, channels, batch): maps narrower than a column tile, of one, one past it and three; channel counts of half a group of 16,
# 24, 40 and more; one-row strips (few images) and strips of several rows with a ragged last one; the row kernel (3x3, and narrow
# maps of many images)
DEPTHWISE = [(4, 8, 1), (15, 24, 2), (17, 40, 1), (33, 24, 1), (23, 144, 24), (16, 144, 24), (33, 40, 24), (5, 320, 220), (9, 144, 200)]


def depthwise_net(kernel, stride, size, channels):
    """Input layer (copies, two pixels to one), a block of the depthwise layer alone on a size x size map, head (copies)."""
    return dataclasses.replace(_mobile(1, kernel, (stride,), A.ACT_RELU, 2 * size, channels), head_mid=channels, head_feat=channels,
                               n_classes=channels)


@pytest.mark.parametrize("kernel", [3, 5, 7])
@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("size,channels,batch", DEPTHWISE)
def test_depthwise_exact(kernel, stride, size, channels, batch):
    arch = depthwise_net(kernel, stride, size, channels)
    rng = np.random.default_rng(67)
    # 0 or at least 3: h-swish leaves those as they are
    x = rng.choice(np.array([0.0, 0.0, 0.0, 3.0], np.float32), (batch, 2 * size, 2 * size, 3)).astype(np.float32)

    def weights(name, shape):
        if name.endswith(".scale"):
            return np.ones(shape)
        if name == "s0b0.dw.w":
            return rng.integers(-1, 2, shape)
        if name == "head.shift":
            return np.full(shape, 4.0)  # (h-swish again)
        return np.zeros(shape) if name == "first.pw.w" or not name.endswith(".w") else _copy(shape)

    got, want = _exact(arch, weights, x)
    pixels = ((size - 1) // stride + 1) ** 2
    np.testing.assert_array_equal(np.rint((got - 4.0) * pixels), np.rint((want - 4.0) * pixels))


def _check_dense(arch, batch, int8):
    if int8:
        from tests.test_gpu_int8 import _check as check_int8
        check_int8(arch, [A.max_cfg(arch)], 47, batch)
    else:
        _check(arch, A.max_cfg(arch), batch, 47, 2 * BF16_TOL)  # (up to fourteen layers)


# Ragged pixels and filters; one, two and four wave groups; 1x1 and 3x3, both strides, with and without a residual; int8:
# channel counts that are no multiple of a cell of 16, reductions of one step and of 33 (the last net: a 1x1 in four groups)
TILED = [(_bottleneck([136, 1040], [1, 2], 112, 0.2), 9), (_bottleneck([136, 1040], [1, 2], 60, 0.6), 9), (_chain([8, 264, 40], 29), 6),
         (_bottleneck([520, 264], [1, 2], 112, 0.2), 9), (_bottleneck([680], [2], 112, 0.2), 57), (_bottleneck([2056], [1], 60, 0.1), 7),
         (_bottleneck([200, 328], [1, 2], 112, 0.2), 9), (_chain([8, 88, 88], 29), 6)]


@pytest.mark.parametrize("arch,batch", TILED)
@pytest.mark.parametrize("int8", [False, True])
def test_tiled_layers(arch, batch, int8):
    _check_dense(arch, batch, int8)


# reductions of less than a step, of less than a round, of several rounds with a ragged last one and of 194 steps; one to four
# waves (float32: eight); pixel tiles of one to 16 pixels, both strides, residuals; a classifier whose class count is no multiple of 4; int8: cells
# that straddle the channel count; the last five: several hundred to a thousand tiles
FEW_PIXELS = [(_chain([8, 24, 200], 9, 10), 1), (_chain([40, 688, 24], 11, 37), 1),
              (_bottleneck([208, 328], [1, 2], 60, 0.35), 1), (_bottleneck([72, 136], [1, 2], 44, 0.2), 3),
              (_chain([24, 200, 72], 15), 6), (_chain([24, 488, 72], 15), 6), (_chain([8, 264, 40], 59), 1),
              (_bottleneck([264, 520], [1, 2], 60, 0.35), 5), (_bottleneck([1640], [1], 28, 0.2), 12)]


@pytest.mark.parametrize("arch,batch", FEW_PIXELS)
@pytest.mark.parametrize("dtype", ["bf16", "int8", "fp32"])
def test_few_pixels(arch, batch, dtype):
    if dtype == "fp32":
        # float32 sums of up to 6192 products against float64: 2^-24 per addition, at random 2^-24 sqrt(6192) = 4.7e-6
        _check(arch, A.max_cfg(arch), batch, 47, 1e-5, False)
    else:
        _check_dense(arch, batch, dtype == "int8")


# The patch kernel of the int8 mode on every layer it covers: tiles of 64, 96 and 128 filters, 1x1 with and without a residual,
# 3x3 with both strides, ragged pixels and channel counts that are no multiple of a cell
@pytest.mark.parametrize("arch,batch", [(_chain([24, 72, 200, 40], 29), 2), (_bottleneck([88, 264], [1, 2], 60, 0.35), 3)])
def test_int8_patch_kernel(arch, batch):
    import paper_2306_17266_amd as S
    from oracle import int8_eval as Q
    from tests.test_gpu_int8 import _problem, _run
    from workloads import quant
    cfg = A.max_cfg(arch)
    ctx, qm = _problem(arch, 71)
    ctx.sushi_set_option(S.OPT_PATCH_CONV_MIN_PIXELS, 1)
    xq = quant.quantize_input(T.make_input(71, 0, batch, cfg.resolution, arch.in_channels, False))
    got = _run(ctx, cfg, xq, arch.n_classes)
    ctx.close()
    np.testing.assert_array_equal(got, Q.forward_int8(arch, qm, cfg, np.ascontiguousarray(xq.transpose(0, 3, 1, 2))))


# The patch kernel with its filter tiles next to each other (1x1, 16384 pixels and more) and pixel tiles next to each other (fewer),
# ragged in both, against the other kernels bit for bit: images and weights are small integers, few weights per filter, so that all
# sums stay below 2^24 and are exact whatever their order.
@pytest.mark.parametrize("arch,batch", [(_bottleneck([136, 264], [1, 1], 112, 0.75), 21), (_bottleneck([136, 264], [1, 1], 112, 0.75), 20),
                                        (_bottleneck([72, 200], [1, 2], 108, 1.0), 129)])
def test_patch_kernel_tile_order(arch, batch):
    import paper_2306_17266_amd as S
    rng = np.random.default_rng(103)
    tens = []
    for name, shape, kind in S.sushi_describe_supernet(arch):
        t = np.ones(shape) if kind in (T.KIND_SCALE, T.KIND_SCALE_RES) else rng.integers(-1, 2, shape)
        if kind == T.KIND_CONV:
            t = np.zeros(shape)
            for k, row in enumerate(t.reshape(shape[0], -1)):
                row[rng.choice(row.size, 4, False)] = rng.choice([-1.0, 1.0], 4)
        tens.append(np.ascontiguousarray(t, dtype=np.float32))
    x = torch.from_numpy(rng.integers(0, 3, (batch, arch.res_choices[0], arch.res_choices[0], 3)).astype(np.float32)).cuda().to(torch.bfloat16)
    got = []
    for pixels in (1, 0):  # the patch kernel wherever it covers a layer, and nowhere
        ctx = S.Sushi(0)
        ctx.sushi_load_supernet(arch, T.flatten(tens), S.BF16)
        ctx.sushi_set_option(S.OPT_PATCH_CONV_MIN_PIXELS, pixels)
        ctx.sushi_set_option(S.OPT_KERNEL_TIMING, 1)
        y = torch.full((batch, arch.n_classes), float("nan"), device="cuda", dtype=torch.float32)
        ctx.sushi_infer(A.max_cfg(arch), x, y)
        torch.cuda.synchronize()
        assert ("conv_patch_kernel" in [k["name"] for k in ctx.sushi_get_kernel_stats() if k["launches"]]) == (pixels == 1)
        ctx.close()
        got.append(y.cpu().numpy())
    assert len(np.unique(got[0])) > got[0].size // 4
    np.testing.assert_array_equal(got[0], got[1])


# Maps of 2 GiB and more go to the kernels with 64-bit addresses.  An image's logits do not depend on the batch: four
# images, repeated, against the same four alone.
@pytest.mark.parametrize("kernel,dtype,batch,arch", [
    ("conv_mfma_kernel", "bf16", 260, _chain([64, 64, 136, 24], 256)),
    ("conv_direct_kernel", "fp32", 132, _chain([64, 40], 256)),
    ("dwconv_kernel", "bf16", 260, _mobile(1, 5, (2,), A.ACT_HSWISH, 512, 64))])
def test_maps_of_two_gib(kernel, dtype, batch, arch):
    import paper_2306_17266_amd as S
    cfg = A.max_cfg(arch)
    bf16 = dtype == "bf16"
    blob, _ = make_problem(arch, 73, bf16)
    ctx = S.Sushi(0)
    ctx.sushi_load_supernet(arch, blob, S.BF16 if bf16 else S.FP32)
    x = torch.from_numpy(T.make_input(73, 0, 4, cfg.resolution, arch.in_channels, bf16)).cuda()
    x = x.to(torch.bfloat16) if bf16 else x
    want = torch.full((4, arch.n_classes), float("nan"), device="cuda", dtype=torch.float32)
    ctx.sushi_infer(cfg, x, want)
    logits = torch.full((batch, arch.n_classes), float("nan"), device="cuda", dtype=torch.float32)
    ctx.sushi_set_option(S.OPT_KERNEL_TIMING, 1)
    ctx.sushi_infer(cfg, x.repeat(batch // 4, 1, 1, 1), logits)
    torch.cuda.synchronize()
    assert kernel in [k["name"] for k in ctx.sushi_get_kernel_stats() if k["launches"]]
    ctx.close()
    want = want.cpu().numpy()
    for n, got in enumerate(logits.cpu().numpy()):
        assert rel_l2(got, want[n % 4]) <= (2 * BF16_TOL if bf16 else 1e-5), n


# An input that starts one element into its buffer: aligned to its element type and no more.  Three and eight input channels (the
# latter read in whole cells), few and many pixels.
@pytest.mark.parametrize("dtype", ["bf16", "fp32", "int8"])
@pytest.mark.parametrize("channels,res,batch", [(3, 9, 2), (8, 9, 1), (8, 30, 8)])
def test_unaligned_input(dtype, channels, res, batch):
    import paper_2306_17266_amd as S
    arch = _chain([24, 40], res, channels=channels)
    cfg = A.max_cfg(arch)
    torch_type = {"bf16": torch.bfloat16, "fp32": torch.float32, "int8": torch.int8}[dtype]
    if dtype == "int8":
        from tests.test_gpu_int8 import _problem
        ctx, _ = _problem(arch, 79)
    else:
        ctx = S.Sushi(0)
        ctx.sushi_load_supernet(arch, make_problem(arch, 79, dtype == "bf16")[0], S.BF16 if dtype == "bf16" else S.FP32)
    x = torch.from_numpy(T.make_input(79, 0, batch, res, channels, dtype == "bf16")).cuda()
    x = torch.round(x * 32).clamp(-128, 127).to(torch_type) if dtype == "int8" else x.to(torch_type)
    shifted = torch.empty(x.numel() + 8, device="cuda", dtype=torch_type)[1:1 + x.numel()].view(x.shape)
    shifted.copy_(x)
    out = []
    for t in (x, shifted):
        out.append(torch.full((batch, arch.n_classes), float("nan"), device="cuda", dtype=torch.float32))
        ctx.sushi_infer(cfg, t, out[-1])
    torch.cuda.synchronize()
    ctx.close()
    # (the bf16 input layer has another kernel for odd addresses)
    assert rel_l2(out[1].cpu().numpy(), out[0].cpu().numpy()) <= (BF16_TOL if dtype == "bf16" and channels == 3 else 0.0)
