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
# tile of the 1x1 layer; one image per workgroup, eight and a ragged last group
@pytest.mark.parametrize("expand,width,res,batch", [(1, 8, 8, 1), (3, 24, 14, 3), (6, 24, 34, 2), (6, 120, 8, 5), (1, 136, 8, 300), (3, 72, 8, 130),
                                                    (6, 160, 12, 64), (6, 24, 62, 9)])
def test_squeeze_excite(expand, width, res, batch):
    _check(block_net(expand, 3, (2, 2) if res == 8 else (1, 2), A.ACT_HSWISH, res, width), batch, {"se_gate_kernel"})
