"""Launches that run several layers of an inverted-residual block against the same layers one by one (the route of a context
whose patch threshold is set) and against the CPU oracle, at the edges of their tiles.

Tolerance against the oracle: 2^-8 of the logits' norm per net of a few layers, as in test_gpu_layer_kernels.py (a bf16 store that
falls the other way); both routes round the same values at the same places, so it bounds their difference too.  The tests named
"exact" have nets whose sums do not depend on their order and hold both routes to the same bits."""
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


# Both routes bit for bit.  Images of 0 and 3 (h-swish leaves those), a first block that adds nothing, weights of -1, 0 and 1, few
# of them per filter where sums would grow: up to the last depthwise layer all sums are integers, or with h-swish multiples of
# 2^-9 below 2^9, exact in any order, so both routes round the same values to bf16.  A squeeze-excite block is the last one, with
# ReLU: its pooling adds integers to less than 2^16 (with h-swish it would add bf16 values down to 2^-16 to sums of 2^15, which
# float32 does not hold).  Its two layers and its projection have one weight per filter (four over averages that are exact, of
# 2^n pixels): what is no integer is not added up.

def _exact_net(expand, kernel, strides, act, res, width, se):
    net = block_net(expand, kernel, strides, act, res, width, se)
    return dataclasses.replace(net, stage_base_out=[int(expand * width)]) if se else net


def _sparse(rng, shape, per_row):
    w = np.zeros(shape, np.float32)
    for k, row in enumerate(w.reshape(shape[0], -1)):
        n = row.size
        row[(k + np.arange(per_row) * max(1, n // per_row)) % n] = rng.choice([-1.0, 1.0], per_row)
    return w


def _exact_tensors(arch, se_terms, special=()):
    """special: channels of the first block whose expanded values are infinite where the input's channel 0 is 3 and 0 elsewhere,
    and whose depthwise weights are all negative."""
    import paper_2306_17266_amd as S
    rng = np.random.default_rng(97)
    out = []
    for name, shape, kind in S.sushi_describe_supernet(arch):
        layer = name.rsplit(".", 1)[0]
        last = layer.split("b0.")[-1]
        if kind in (T.KIND_SCALE, T.KIND_SCALE_RES):
            t = np.ones(shape)
        elif not name.endswith(".w"):
            t = np.zeros(shape) if layer in ("stem", "first.dw", "first.pw") else rng.integers(-1, 2, shape)
        elif layer in ("stem", "head"):
            t = np.zeros(shape)
            for k in range(shape[0]):
                t[(k, k % shape[1]) + tuple(r // 2 for r in shape[2:])] = 1.0
        elif layer in ("first.dw", "first.pw"):
            t = np.zeros(shape)
        elif last == "expand":
            t = _sparse(rng, shape, min(8, shape[1]))
        elif last == "dw":
            t = rng.integers(-1, 2, shape)
        elif last == "se1":
            t = _sparse(rng, shape, se_terms)
        elif last == "se2":
            t = _sparse(rng, shape, 1) * 0.25
        elif last == "project":
            t = np.eye(shape[0]).reshape(shape) if shape[0] == shape[1] else _sparse(rng, shape, 4)
        else:
            t = rng.standard_normal(shape) * (2.0 / shape[1]) ** 0.5
        t = np.ascontiguousarray(t, dtype=np.float32)
        if special and name.startswith("s0b0."):
            if name.endswith("expand.w"):
                t[special] = 0.0
                t[special, 0] = 1.0
            elif name.endswith("expand.scale"):
                t[special] = 3e38
            elif name.endswith("expand.shift"):
                t[special] = -3e38  # 3 x 3e38 - 3e38 is beyond the largest float32
            elif name.endswith("dw.w"):
                t[special] = -1.0
            elif name.endswith("dw.shift"):
                t[special] = 0.0
        out.append(T.round_to_bf16(t) if name.endswith(".w") else t)
    return out


def _check_exact(arch, batch, kernels, se_terms=1, special=()):
    res = max(arch.res_choices)
    x = np.random.default_rng(101).choice(np.array([0.0, 0.0, 3.0], np.float32), (batch, res, res, 3))
    assert len(np.unique(x[0, ::2, ::2, 0])) == 2
    blob = T.flatten(_exact_tensors(arch, se_terms, special))
    xd = torch.from_numpy(x).cuda().to(torch.bfloat16).contiguous()
    got, ran = _logits(arch, blob, xd, True)
    single, ran_single = _logits(arch, blob, xd, False)
    assert kernels <= ran and not kernels & ran_single, (ran, ran_single)
    assert np.isfinite(single).all() and len(np.unique(single)) > single.size // 2
    np.testing.assert_array_equal(got, single)


# as for test_expand_depthwise, maps past a tile by one output and by one halo among them
@pytest.mark.parametrize("kernel", [3, 5, 7])
@pytest.mark.parametrize("act", [A.ACT_RELU, A.ACT_HSWISH])
@pytest.mark.parametrize("expand,width,stride,res,batch", [
    (3, 8, 1, 8, 1), (3, 24, 1, 28, 2), (6, 40, 2, 66, 1), (3, 72, 1, 34, 3), (2, 120, 2, 30, 1), (6, 160, 1, 14, 2), (3, 24, 2, 112, 3), (6, 8, 2, 8, 70),
    (4, 24, 1, 62, 30), (6, 24, 1, 112, 5), (6, 24, 2, 118, 4)])
def test_expand_depthwise_exact(kernel, act, expand, width, stride, res, batch):
    _check_exact(_exact_net(expand, kernel, (stride,), act, res, width, 0), batch, {"expand_dw_kernel"})


# two blocks: the second one's input is the first one's output, any integers
@pytest.mark.parametrize("kernel", [3, 5, 7])
@pytest.mark.parametrize("strides", [(1, 2), (2, 1)])
def test_expand_depthwise_exact_two_blocks(kernel, strides):
    _check_exact(_exact_net(3, kernel, strides, A.ACT_RELU, 60, 40, 0), 3, {"expand_dw_kernel"})


# with the pooling's sums, the gates and the gated projection: maps of 2^n pixels (four terms per hidden value) and others; one
# image and several per workgroup, and more workgroups of the gated layer than run at once
@pytest.mark.parametrize("kernel", [3, 5, 7])
@pytest.mark.parametrize("expand,width,stride,res,batch", [(6, 24, 1, 64, 3), (6, 40, 2, 64, 9), (3, 72, 2, 16, 130), (4, 160, 1, 16, 2), (6, 24, 1, 58, 3), (3, 24, 2, 30, 5), (6, 40, 1, 56, 96)])
def test_squeeze_excite_exact(kernel, expand, width, stride, res, batch):
    size = res // 2 // stride
    _check_exact(_exact_net(expand, kernel, (stride,), A.ACT_RELU, res, width, 1), batch, {"expand_dw_kernel", "se_gate_kernel"}, 4 if size & (size - 1) == 0 else 1)


# Expanded values of two channels that are infinite at a third of the pixels, depthwise weights all negative there: minus infinity,
# which ReLU makes 0, at the outputs that use them, and what the single layers give elsewhere
@pytest.mark.parametrize("kernel", [3, 5, 7])
@pytest.mark.parametrize("strides,res", [((1, 2), 20), ((2, 1), 70)])
def test_expand_depthwise_infinite_values(kernel, strides, res):
    _check_exact(_exact_net(3, kernel, strides, A.ACT_RELU, res, 16, 0), 2, {"expand_dw_kernel"}, special=[5, 38])
