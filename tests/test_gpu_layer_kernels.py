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
