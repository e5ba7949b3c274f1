"""The per-layer kernels at the edges of their tiles, through small SuperNets built for it, against the CPU oracle.

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


def _chain(widths, strides, res, classes=64, channels=3):
    """A Tiny-family net: 3x3 layers of the given widths and strides, pooling, classifier."""
    n = len(widths)
    return dataclasses.replace(A.tiny_arch(), n_classes=classes, in_channels=channels, stage_base_out=list(widths),
                               stage_stride=list(strides), stage_max_depth=[1] * n, stage_act=[A.ACT_RELU] * n,
                               stage_se=[0] * n, depth_drop_choices=[0], width_choices=[1.0], res_choices=[res])


# odd sizes: patch rows that start on odd elements, tensors of an odd number of elements (the general kernel), columns
# outside on either side; 15 x 15 = one pixel short of a tile; widths of half a filter tile, a ragged one, several groups
@pytest.mark.parametrize("res,stride,width,batch", [(8, 1, 8, 1), (9, 1, 24, 2), (9, 2, 16, 1), (15, 1, 32, 4), (33, 2, 40, 2), (31, 2, 72, 3),
                                                     (12, 2, 16, 6), (224, 1, 16, 4)])
def test_input_layer(res, stride, width, batch):
    arch = _chain([width, 16], [stride, 2], res)
    _check(arch, A.max_cfg(arch), batch, 41, BF16_TOL)


# A weight of minus infinity and an input above 0: minus infinity, ReLU'd to 0, wherever its tap lies inside the image, and
# outside it the tap is no part of the sum.  The oracle gets a large finite weight instead.  Input layer and float32 layers.
@pytest.mark.parametrize("bf16,layer", [(True, 0), (False, 0), (False, 1)])
def test_infinite_weight_outside_the_image(bf16, layer):
    import paper_2306_17266_amd as S
    from oracle import subnet_eval as E
    arch = _chain([8, 16], [1, 1], 8)
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


# 60, 44 and 45 tiles of 64 x 64 with ragged pixels and filters; reductions of one step, of an odd number of steps and of 69
# (split over one, two and four wave groups), not a multiple of a step; 1x1 and 3x3, both strides, with and without a residual;
# int8: channel counts that are no multiple of a cell of 16, 128 tiles and more
@pytest.mark.parametrize("arch,batch", [(_chain([24, 200, 72], [1, 1, 2], 15), 6), (_chain([24, 488, 72], [1, 1, 1], 15), 6),
                                        (_chain([8, 264, 40], [2, 1, 1], 59), 1), (_bottleneck([264, 520], [1, 2], 60, 0.35), 5),
                                        (_bottleneck([200, 328], [1, 2], 112, 0.2), 9)])
@pytest.mark.parametrize("int8", [False, True])
def test_tiled_layers(arch, batch, int8):
    if int8:
        from tests.test_gpu_int8 import _check as check_int8
        check_int8(arch, [A.max_cfg(arch)], 47, batch)
    else:
        _check(arch, A.max_cfg(arch), batch, 47, 2 * BF16_TOL)  # (up to fourteen layers)


# reductions of less than a step, of less than a round, of several rounds with a ragged last one and of 194 steps (16 waves);
# pixel tiles of one to 16 pixels, both strides, residuals; a classifier whose class count is no multiple of 4; int8: cells
# that straddle the channel count
@pytest.mark.parametrize("arch,batch", [(_chain([8, 24, 200], [1, 2, 1], 9, 10), 1), (_chain([40, 688, 24], [2, 1, 1], 11, 37), 1),
                                        (_bottleneck([208, 328], [1, 2], 60, 0.35), 1), (_bottleneck([72, 136], [1, 2], 44, 0.2), 3)])
@pytest.mark.parametrize("dtype", ["bf16", "int8", "fp32"])
def test_few_pixels(arch, batch, dtype):
    if dtype == "fp32":
        # float32 sums of up to 6192 products against float64: 2^-24 per addition, at random 2^-24 sqrt(6192) = 4.7e-6
        _check(arch, A.max_cfg(arch), batch, 47, 1e-5, False)
    else:
        test_tiled_layers(arch, batch, dtype == "int8")
