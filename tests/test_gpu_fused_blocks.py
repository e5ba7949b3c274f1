"""Launches that run several layers of an inverted-residual block against the same layers one by one (the route of a context
whose patch threshold is set) and against the CPU oracle, at the edges of their tiles.

Tolerance: 2^-8 of the logits' norm per net of a few layers, as in test_gpu_layer_kernels.py (a bf16 store that falls the other
way); both routes round the same values at the same places, so it bounds their difference too."""
import dataclasses

import numpy as np
import pytest
import torch

from tests.common import make_problem, oracle_logits_bf16_stores, rel_l2
from workloads import arch as A
from workloads import tensors as T

pytestmark = pytest.mark.gpu

TOL = 2 * 2.0 ** -8  # (up to sixteen layers)


def block_net(expand, kernel, strides, act, res, out, se=1):
    """An inverted-residual net of one block per stage, all of one width."""
    n = len(strides)
    return dataclasses.replace(A.small_mbv3_arch(), stage_base_out=[out] * n, stage_stride=list(strides), stage_max_depth=[1] * n,
                               stage_act=[act] * n, stage_se=[se] * n, depth_drop_choices=[0], expand_choices=[float(expand)],
                               kernel_choices=[kernel], res_choices=[res], stem_out=out)


def _logits(arch, blob, x, fused):
    import paper_2306_17266_amd as S
    ctx = S.Sushi(0)
    ctx.sushi_load_supernet(arch, blob, S.BF16)
    if not fused:
        ctx.sushi_set_option(S.OPT_PATCH_CONV_MIN_PIXELS, 0)
    y = torch.full((x.shape[0], arch.n_classes), float("nan"), device="cuda", dtype=torch.float32)
    ctx.sushi_set_option(S.OPT_KERNEL_TIMING, 1)
    ctx.sushi_infer(A.max_cfg(arch), x, y)
    torch.cuda.synchronize()
    ran = {k["name"] for k in ctx.sushi_get_kernel_stats() if k["launches"]}
    ctx.close()
    return y.cpu().numpy(), ran


def _check(arch, batch, kernels, seed=83):
    blob, wts = make_problem(arch, seed, True)
    res = max(arch.res_choices)
    x_np = T.make_input(seed, 0, batch, res, arch.in_channels, True)
    x = torch.from_numpy(x_np).cuda().to(torch.bfloat16).contiguous()
    got, ran = _logits(arch, blob, x, True)
    single, ran_single = _logits(arch, blob, x, False)
    assert kernels <= ran and not kernels & ran_single, (ran, ran_single)
    few = x_np[:4]
    want = oracle_logits_bf16_stores(arch, wts, A.max_cfg(arch), few)
    for n in range(batch):
        assert rel_l2(got[n], single[n]) <= TOL, n
        assert n >= len(few) or rel_l2(got[n], want[n]) <= TOL, n


# (expand, width, resolution, batch): hidden vectors of less than a filter tile, of one and of several with a ragged last one;
# 8 gates and more than a chunk's; inputs that end inside a reduction step (24, 72, 144); maps of one pixel and of more than a
# tile of the 1x1 layer; one image per workgroup, eight and a ragged last group; a gated 1x1 layer of more workgroups (1176) than
# the chip holds at once (1024), so that some start after others have stored
@pytest.mark.parametrize("expand,width,res,batch", [(1, 8, 8, 1), (3, 24, 14, 3), (6, 24, 34, 2), (6, 120, 8, 5), (1, 136, 8, 300), (3, 72, 8, 130),
                                                    (6, 160, 12, 64), (6, 24, 62, 9), (6, 40, 56, 96)])
def test_squeeze_excite(expand, width, res, batch):
    _check(block_net(expand, 3, (2, 2) if res == 8 else (1, 2), A.ACT_HSWISH, res, width), batch, {"se_gate_kernel"})


# Expansion and depthwise layer in one launch: every kernel size and stride; input channels of one to five reduction steps, ending
# inside one (8, 24, 40, 72, 120, 160); expanded channels that end inside a block of 32 (24, 72, 120, 240); maps smaller than the
# kernel, of one tile, one pixel past it and of several, odd ones; one image and many tiles per workgroup; with the pooling's sums
@pytest.mark.parametrize("kernel", [3, 5, 7])
@pytest.mark.parametrize("expand,width,strides,res,batch,se", [
    (3, 8, (1, 2), 8, 1, 0), (3, 24, (1, 2), 28, 2, 0), (6, 40, (2, 1), 66, 1, 1), (3, 72, (1, 2), 34, 3, 1), (2, 120, (1, 2), 30, 1, 0), (6, 160, (1, 2), 14, 2, 1),
    (3, 24, (2, 1), 112, 3, 1), (6, 8, (2, 2), 8, 70, 1), (4, 24, (1, 2), 62, 30, 0)])
def test_expand_depthwise(kernel, expand, width, strides, res, batch, se):
    _check(block_net(expand, kernel, strides, A.ACT_HSWISH if kernel == 5 else A.ACT_RELU, res, width, se), batch, {"expand_dw_kernel"})


# Expanded values that overflow to infinity at a few pixels of two channels, depthwise weights all negative there: minus infinity,
# which ReLU makes 0, at the outputs that use them, and what the single layers give elsewhere
@pytest.mark.parametrize("kernel", [3, 5, 7])
@pytest.mark.parametrize("strides,res", [((1, 2), 20), ((2, 1), 70)])
def test_expand_depthwise_infinite_values(kernel, strides, res):
    import paper_2306_17266_amd as S
    arch = block_net(3, kernel, strides, A.ACT_RELU, res, 16, 0)
    table = S.sushi_describe_supernet(arch)
    tens = T.make_weights([(s, k) for _, s, k in table], 89, True)
    for (name, _, _), t in zip(table, tens):
        if name == "s0b0.expand.scale":
            t[[5, 38]] = 3e38
        elif name == "s0b0.expand.shift":
            t[[5, 38]] = -3e38
        elif name == "s0b0.dw.shift":
            t[[5, 38]] = 0.0
        elif name == "s0b0.dw.w":
            t[[5, 38]] = -np.abs(t[[5, 38]]) - 0.01
    x = torch.from_numpy(T.make_input(89, 0, 2, res, arch.in_channels, True)).cuda().to(torch.bfloat16)
    got, _ = _logits(arch, T.flatten(tens), x, True)
    want, _ = _logits(arch, T.flatten(tens), x, False)
    assert np.isfinite(want).all()
    for n in range(2):
        assert rel_l2(got[n], want[n]) <= TOL, n
