"""Timing cases of the library's serving path: what a program that serves SubNet queries calls, over the range of
SuperNets, batch sizes, resolutions, precisions and stream kinds that this repository configures, tests and benchmarks.

Two kinds of case:

  query   one sushi_infer of one SubNet on one input batch through the default execution mode (one launch per layer on
          the caller's stream): a lone request, or a batch that a front end has gathered.  bf16, int8 (the bottleneck
          family) and float32 (the Tiny family).
  stream  a session of many queries through the persistent kernel (execution mode 3): every query has its own input
          and its own logits; the scheduler accounts each query and re-chooses the cached SubGraph every Q queries, or
          (policy "levels") also picks the SubNet for the query's latency target.  The session starts with an empty
          cache and ends when all logits are there and the persistent kernel has left the GPU.

A SubNet is named by "min", "max" or the seed of a uniform draw over the SuperNet's elastic choices.
"""
import ctypes
import math
import os

import numpy as np
import torch

import paper_2306_17266_amd as S
from paper_2306_17266_amd import sushiabs
from workloads import arch as A
from workloads import quant, streams
from workloads import tensors as T
from workloads.rng import Stream

ARCHS = {"tiny": A.tiny_arch, "resnet": A.resnet_arch, "mbv3": A.mbv3_arch}
ELEM_BYTES = {"fp32": 4, "bf16": 2, "int8": 1}


def _query(name, family, dtype, batch, resolution, subnet):
    return {"name": name, "kind": "query", "family": family, "dtype": dtype, "batch": batch, "resolution": resolution,
            "subnet": subnet}


def _stream(name, family, policy, batch, queries, teams, q, budget_mib, seed):
    return {"name": name, "kind": "stream", "family": family, "dtype": "bf16", "policy": policy, "batch": batch,
            "queries": queries, "teams_per_xcd": teams, "q": q, "budget_mib": budget_mib, "stream_seed": seed}


def listed():
    return [
        # the smallest call: one image through the Tiny SuperNet in float32
        _query("tiny_fp32_b1", "tiny", "fp32", 1, 32, "max"),
        # a lone request of an interactive service, both families, SubNets of medium size
        _query("resnet_b1", "resnet", "bf16", 1, 224, 5),
        _query("mbv3_b1", "mbv3", "bf16", 1, 224, 3),
        # a few requests gathered into an odd batch at a reduced resolution
        _query("mbv3_b5_r160", "mbv3", "bf16", 5, 160, 7),
        # ordinary batches, the largest SubNet
        _query("resnet_b16", "resnet", "bf16", 16, 224, "max"),
        # offline scoring: large batches (odd: the last batch of a data set is rarely full)
        _query("resnet_b61", "resnet", "bf16", 61, 224, 2),
        _query("mbv3_b64", "mbv3", "bf16", 64, 224, "max"),
        # the paper's own precision, a lone request and a batch
        _query("resnet_int8_b1", "resnet", "int8", 1, 224, 5),
        _query("resnet_int8_b16", "resnet", "int8", 16, 224, "max"),
        # query streams at batch 1: sticky SubNets (bottleneck family), Zipf popularity with a resolution per query
        # (inverted-residual family)
        _stream("resnet_sticky_stream", "resnet", "sticky", 1, 1000, 16, 8, 16, 2),
        _stream("mbv3_regimes_stream", "mbv3", "regimes", 1, 1000, 16, 10, 32, 5),
        # batch-16 queries with a latency target each: Algorithm 1 picks the SubNet
        _stream("resnet_b16_levels_stream", "resnet", "levels", 16, 120, 1, 8, 64, 4),
    ]


def draw(rng):
    def log_int(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))

    subnet = rng.choice(["min", "max"] + [rng.randrange(1000) for _ in range(6)])
    kind = rng.choice(["tiny", "resnet", "resnet", "mbv3", "mbv3", "int8", "sticky", "regimes", "levels"])
    if kind == "tiny":
        case = _query("", "tiny", "fp32", log_int(1, 64), 32, subnet)
    elif kind == "resnet":
        case = _query("", "resnet", "bf16", log_int(1, 61), 224, subnet)
    elif kind == "mbv3":
        case = _query("", "mbv3", "bf16", log_int(1, 96), rng.choice([160, 192, 224]), subnet)
    elif kind == "int8":
        case = _query("", "resnet", "int8", log_int(1, 48), 224, subnet)
    elif kind == "sticky":
        case = _stream("", "resnet", "sticky", 1, log_int(250, 1000), rng.choice([8, 16]), rng.choice([4, 8, 16]),
                       rng.choice([8, 16]), rng.randrange(1000))
    elif kind == "regimes":
        case = _stream("", "mbv3", "regimes", 1, log_int(250, 1500), rng.choice([8, 16]), 10, rng.choice([4, 32]),
                       rng.randrange(1000))
    else:
        case = _stream("", "resnet", "levels", 16, log_int(30, 110), 1, 8, 64, rng.randrange(1000))
    del case["name"]
    return case


# ---------------------------------------------------------------- what a case consists of

def _subnet(arch, which, resolution):
    if which == "min":
        return A.min_cfg(arch, resolution)
    if which == "max":
        return A.max_cfg(arch, resolution)
    return streams.uniform_cfg(arch, Stream(int(which)), resolution)


def _stream_subnets(case, arch):
    """The SubNet of every query, or the pool that the scheduler chooses from."""
    n, seed = case["queries"], case["stream_seed"]
    if case["policy"] == "sticky":
        return streams.stream_sticky(arch, n, seed, 0.8, 224)
    if case["policy"] == "regimes":
        pool = streams.subnet_pool(arch, 32, 3, 224)
        picks = streams.stream_zipf(32, n, seed, 1.2, regime=500, resolutions=[160, 192, 224])
        return [streams.with_resolution(pool[i], r) for i, r in picks]
    return streams.subnet_pool(arch, 16, 4, 224)


class _Session:
    """What a stream's program keeps: the SubNets with their boxes and vectors, the candidate SubGraphs, the
    scheduler's inputs.  choose(ctx, t) is the scheduler's part of query t."""

    def __init__(self, case, arch):
        self.by_target = case["policy"] == "levels"
        self.budget = case["budget_mib"] << 20
        self.serving = _stream_subnets(case, arch)
        boxes = {}
        for c in self.serving:
            if c.key() not in boxes:
                boxes[c.key()] = S.sushi_subnet_layers(arch, c)
        self.boxes = boxes
        vec = {k: np.array([v for (kk, cc, _) in b for v in (kk, cc)], dtype=np.int32) for k, b in boxes.items()}
        self.candidates = streams.candidate_subgraphs(list(boxes.values()), self.budget, 2, 40)
        gvecs = [[v for (k, c, _) in b for v in (k, c)] for b in self.candidates]
        self.q = case["q"]
        if self.by_target:
            sizes = [streams.box_bytes(boxes[c.key()], 2) for c in self.serving]
            acc = [0.0] * len(self.serving)
            for rank, i in enumerate(sorted(range(len(sizes)), key=lambda i: sizes[i])):
                acc[i] = float(np.float32(0.70 + 0.01 * rank))
            path = sushiabs.table_path("resnet_bs16_levels", self.budget, case["teams_per_xcd"])
            table = sushiabs.load_table(path, len(self.serving), len(self.candidates))["table"]
            targets = sushiabs.latency_levels(table, 5)
            self.targets = [targets[i] for i in streams.stream_levels(5, case["queries"], case["stream_seed"])]
            self.sched = ([vec[c.key()] for c in self.serving], acc, gvecs, table)
        else:
            self.vecs = [vec[c.key()] for c in self.serving]
            n = len(gvecs[0])
            self.sched = ([[0] * n], [0.0], gvecs, [[1.0] * (len(gvecs) + 1)])

    def start(self, ctx):
        ctx.sushi_sched_init(*self.sched, self.q, S.STRICT_LATENCY)

    def served(self, case):
        """The SubNets of the whole session in order (host only)."""
        if not self.by_target:
            return list(self.serving)
        ctx = S.Sushi(-1)
        self.start(ctx)
        out = [self.serving[ctx.sushi_sched_step(0.0, lat)[0]] for lat in self.targets]
        ctx.close()
        return out


def _weight_blob(arch, gen):
    """float32 blob of a SuperNet's tensors: the distributions of workloads.tensors, drawn on the GPU."""
    table = S.sushi_describe_supernet(arch)
    sizes = [int(np.prod(s)) for _, s, _ in table]
    blob = torch.randn(sum(sizes), generator=gen, device="cuda", dtype=torch.float32)
    uni = torch.rand(max(sizes), generator=gen, device="cuda", dtype=torch.float32)
    at = 0
    for (_, shape, kind), n in zip(table, sizes):
        part = blob[at:at + n]
        if kind in (T.KIND_CONV, T.KIND_FC):
            part.mul_(math.sqrt(2.0 / float(np.prod(shape[1:]))))
        elif kind == T.KIND_DWCONV:
            part.mul_(math.sqrt(2.0 / (shape[-1] * shape[-2])))
        elif kind == T.KIND_SCALE:
            part.copy_(0.8 + 0.4 * uni[:n])
        elif kind == T.KIND_SCALE_RES:
            part.copy_(0.25 + 0.25 * uni[:n])
        else:
            part.mul_(0.05)
        at += n
    return table, sizes, blob


def _fixed_point(m):
    """float64 tensor of positive factors -> int32 multipliers in [2^30, 2^31) and right shifts."""
    frac, exp = torch.frexp(m)
    mult = torch.round(frac * 2.0 ** 31)
    over = mult >= 2.0 ** 31
    mult = torch.where(over, mult / 2, mult)
    return mult.to(torch.int32), (31 - exp - over.to(torch.int32)).to(torch.int32)


def _int8_model(arch, table, sizes, blob):
    """int8 weights and parameter words of the recipe in workloads.quant, computed on the GPU."""
    role = {"in": (quant.S_IN, 0), "relu": (quant.S_RELU, quant.Z_RELU), "lin": (quant.S_LIN, 0)}
    roles = quant.layer_roles(arch)
    part, at = {}, 0
    for (name, shape, _), n in zip(table, sizes):
        part[name] = blob[at:at + n].view(shape).double()
        at += n
    weights, words = [], []
    for name, shape, kind in table:
        if kind not in (T.KIND_CONV, T.KIND_FC):
            continue
        base = name[:-2]
        w = part[name].reshape(shape[0], -1)
        s_w = w.abs().amax(dim=1).clamp_min(1e-12) / 127.0
        weights.append(torch.round(w / s_w[:, None]).clamp_(-127, 127).to(torch.int8).reshape(-1))
        in_role, out_role, res_role = roles[base]
        s_x, z_x = role[in_role]
        scalars = torch.zeros(quant.Q_SCALARS, dtype=torch.int32, device=blob.device)
        scalars[0] = z_x
        if kind == T.KIND_CONV:
            s_y, z_y = role[out_role]
            g = part[base + ".scale"] * s_x * s_w
            mult, shift = _fixed_point(g / s_y)
            bias = torch.round(part[base + ".shift"] / g).to(torch.int32)
            scalars[1] = z_y
            if res_role is not None:
                s_r, z_r = role[res_role]
                scalars[2], scalars[3] = quant.fixed_point(s_r / s_y)
                scalars[4] = z_r
        else:
            factor = (s_x * s_w).float()
            mult, shift = factor.view(torch.int32), torch.zeros_like(factor, dtype=torch.int32)
            bias = torch.round(part[base + ".b"] / factor.double()).to(torch.int32)
        words += [mult, shift, bias, scalars]
    return torch.cat(weights).cpu().numpy(), torch.cat(words).cpu().numpy()


def _input(gen, dtype, shape):
    x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
    if dtype == "int8":
        return torch.round(x / quant.S_IN).clamp_(-128, 127).to(torch.int8)
    return x.to(torch.bfloat16) if dtype == "bf16" else x


def _context(arch, dtype, gen):
    table, sizes, blob = _weight_blob(arch, gen)
    ctx = S.Sushi(0)
    if dtype == "int8":
        ctx.sushi_load_supernet_int8(arch, *_int8_model(arch, table, sizes, blob))
    else:
        ctx.sushi_load_supernet(arch, blob.cpu().numpy(), S.BF16 if dtype == "bf16" else S.FP32)
    return ctx


def prepare(case, seed):
    arch = ARCHS[case["family"]]()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    ctx = _context(arch, case["dtype"], gen)
    state = {"kind": case["kind"], "ctx": ctx}
    batch = case["batch"]
    if case["kind"] == "query":
        state["cfg"] = _subnet(arch, case["subnet"], case["resolution"])
        state["x"] = _input(gen, case["dtype"], (batch, case["resolution"], case["resolution"], arch.in_channels))
        state["logits"] = torch.zeros(batch, arch.n_classes, device="cuda", dtype=torch.float32)
        torch.cuda.synchronize()
        return state
    ctx.sushi_set_option(S.OPT_EXEC_MODE, 3)
    ctx.sushi_set_option(S.OPT_TEAMS_PER_XCD, case["teams_per_xcd"])
    ses = _Session(case, arch)
    n = case["queries"]
    res = [224] * n if ses.by_target else [c.resolution for c in ses.serving]
    state["x"] = [_input(gen, case["dtype"], (batch, r, r, arch.in_channels)) for r in res]
    state["logits"] = torch.zeros(n, batch, arch.n_classes, device="cuda", dtype=torch.float32)
    # everything a query passes to the library, marshalled once
    cfgs = {}
    for c in ses.serving:
        if c.key() not in cfgs:
            cfgs[c.key()] = ctx.marshal_cfg(c)
    state.update(ses=ses, batch=batch, cfgs=[cfgs[c.key()] for c in ses.serving],
                 graphs=[ctx.marshal_subgraph(b) for b in ses.candidates],
                 x_ptr=[ctypes.c_void_p(x.data_ptr()) for x in state["x"]],
                 y_ptr=[ctypes.c_void_p(y.data_ptr()) for y in state["logits"]])
    if not ses.by_target:
        state["vecs"] = [ctx.marshal_vec(v) for v in ses.vecs]
    torch.cuda.synchronize()
    return state


def run(state):
    ctx = state["ctx"]
    if state["kind"] == "query":
        ctx.sushi_infer(state["cfg"], state["x"], state["logits"])
        return state["logits"]
    ses, batch, cfgs, graphs = state["ses"], state["batch"], state["cfgs"], state["graphs"]
    x_ptr, y_ptr = state["x_ptr"], state["y_ptr"]
    ses.start(ctx)
    ctx.sushi_set_subgraph_cache(None, 0)
    cached = -1
    for t in range(len(x_ptr)):
        if ses.by_target:
            i, j = ctx.sushi_sched_step(0.0, ses.targets[t])
            ctx.infer_marshalled(cfgs[i], x_ptr[t], batch, y_ptr[t])
        else:
            ctx.infer_marshalled(cfgs[t], x_ptr[t], batch, y_ptr[t])
            j = ctx.sched_record_marshalled(state["vecs"][t])
        if j >= 0 and j != cached:
            ctx.set_subgraph_cache_marshalled(graphs[j], ses.budget)
            cached = j
    ctx.sushi_quiesce()
    return state["logits"]


def _flops(arch, cfg):
    """Multiply-adds of one image, times two, from the library's own op list."""
    total = 0.0
    for op in S.sushi_team_plan(arch, cfg, 1, 2):
        out = op["P"] * op["Q"] * op["K"]
        if op["kind"] in (0, 4):
            total += 2.0 * out * op["C"] * op["R"] * op["R"]
        elif op["kind"] == 1:
            total += 2.0 * out * op["R"] * op["R"]
    return total


def work(case):
    """Each input image read once, the weights that the SubNets use read once, the logits written once."""
    arch = ARCHS[case["family"]]()
    es, batch = ELEM_BYTES[case["dtype"]], case["batch"]
    if case["kind"] == "query":
        served = [_subnet(arch, case["subnet"], case["resolution"])]
    else:
        served = _Session(case, arch).served(case)
    count = {}
    for c in served:
        count.setdefault(c.key(), [c, 0])[1] += 1
    union, flops, images = None, 0.0, 0.0
    for c, n in count.values():
        box = S.sushi_subnet_layers(arch, c)
        union = box if union is None else [tuple(max(p, q) for p, q in zip(a, b)) for a, b in zip(union, box)]
        flops += n * batch * _flops(arch, c)
        images += n * batch * (c.resolution ** 2 * arch.in_channels * es + 4.0 * arch.n_classes)
    return {"bytes": images + streams.box_bytes(union, es), "flops": flops}


def tolerance(case):
    """int8 is integer arithmetic with one right answer.  float32: the sums' order (2e-6 against sums in float64).
    bf16: every stored feature map is rounded to bf16, and another order of a layer's sums moves some of those
    roundings.  Measured between the execution modes, between kernels of different summation order and against the
    float32 mode on the same weights: up to 1.2e-3 on the bottleneck family, up to 3.5e-3 on the deepest
    inverted-residual SubNet."""
    if case["dtype"] == "int8":
        return "exact"
    if case["dtype"] == "fp32":
        return {"rel": 1e-5}
    return {"rel": 5e-3 if case["family"] == "resnet" else 1.2e-2}
