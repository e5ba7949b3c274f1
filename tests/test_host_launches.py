"""The library's launches, seen from the host: limits of a launch, per-device state, which kernel serves which layer.  No GPU:
the library runs on tests/fake_hip.cpp."""
import subprocess

from tests.fake_hip import ROOT, run
from workloads import arch as A


def test_large_lds_on_every_device_and_after_a_failure(tmp_path):
    """Kernels with more than 64 KiB of dynamic LDS need the limit raised on the device they run on, by every context that
    is the first there; a failure is reported and the next query tries again."""
    out = run(tmp_path, '''
arch = A.resnet_arch()
cfg = A.max_cfg(arch, 224)
for dtype in ("bf16", "int8"):
    for device in (0, 1):
        ctx = context(arch, dtype, device)
        if device == 1:
            fake.fake_fail_attributes(1)
            try:
                infer(ctx, cfg, 16)
                raise SystemExit("no error")
            except S.SushiError as e:
                assert e.code == -5, e
        big = [k for k in infer(ctx, cfg, 16) if k[4] > 65536]
        print(dtype, device, sorted({k[0] for k in big}))
        ctx.close()
''')
    want = ["conv_patch_kernel", "conv_tile_kernel"]
    assert out.splitlines() == ["%s %d %s" % (t, d, want) for t in ("bf16", "int8") for d in (0, 1)], out


def test_float32_maps_of_many_gib_are_launched(tmp_path):
    """A launch has fewer than 2^32 threads along a dimension.  A float32 layer with an output of 17 GiB (8.3 million pixels,
    512 filters, 64 input channels) has to stay below it, whichever kernel it gets."""
    out = run(tmp_path, '''
arch = dataclasses.replace(A.tiny_arch(), n_classes=8, stage_base_out=[64, 512], stage_stride=[1, 1], stage_max_depth=[1, 1],
                           stage_act=[A.ACT_RELU] * 2, stage_se=[0, 0], depth_drop_choices=[0], width_choices=[1.0], res_choices=[256])
ctx = context(arch, "fp32")
launches = infer(ctx, A.max_cfg(arch), 127)
print([k[0] for k in launches], max(k[2] * k[3] for k in launches) < 1 << 32)
ctx.close()
''')
    assert out.split("]")[1].strip() == "True", out


def test_patch_threshold_set_by_the_caller(tmp_path):
    """SUSHI_OPT_PATCH_CONV_MIN_PIXELS decides by itself once it is set, at every value: one threshold more or less moves no
    layer unless its pixel count lies between the two."""
    out = run(tmp_path, '''
arch = A.resnet_arch()
cfg = A.max_cfg(arch, 224)
for dtype in ("bf16", "int8"):
    ctx = context(arch, dtype)
    counts = []
    for value in (None, 3135, 3136, 3137, 0):
        if value is not None:
            ctx.sushi_set_option(S.OPT_PATCH_CONV_MIN_PIXELS, value)
        counts.append(sum(k[0] == "conv_patch_kernel" for k in infer(ctx, cfg, 17)))
    print(counts[1] == counts[2] == counts[3] > counts[0] > 0, counts[4] == 0, counts)
    ctx.close()
''')
    assert [line.split()[:2] for line in out.splitlines()] == [["True", "True"]] * 2, out


def test_statistics_name_the_kernels_that_ran(tmp_path):
    out = run(tmp_path, '''
from collections import Counter
POOL_FC = {"maxpool_i8_kernel", "gap_i8_kernel", "fc_i8_kernel"}
for arch, dtype, batch, res in ((A.resnet_arch(), "bf16", 1, 224), (A.resnet_arch(), "bf16", 16, 224), (A.mbv3_arch(), "bf16", 1, 224),
                                (A.mbv3_arch(), "bf16", 64, 224), (A.small_mbv3_arch(), "fp32", 2, 64), (A.resnet_arch(), "int8", 1, 224),
                                (A.resnet_arch(), "int8", 48, 224)):
    ctx = context(arch, dtype)
    ctx.sushi_set_option(S.OPT_KERNEL_TIMING, 1)
    ran = Counter("int8_pool_fc_kernels" if k[0] in POOL_FC else k[0] for k in infer(ctx, A.max_cfg(arch, res), batch))
    told = Counter({k["name"]: k["launches"] for k in ctx.sushi_get_kernel_stats() if k["launches"]})
    print(dtype, batch, "ok" if ran == told else (ran, told))
    ctx.close()
''')
    assert all(line.endswith(" ok") for line in out.splitlines()) and len(out.splitlines()) == 7, out


def _nets_of_gpu_tests():
    from tests import test_gpu_layer_kernels as t
    return dict(tiled=t.TILED, few=t.FEW_PIXELS, depthwise=[(t.depthwise_net(k, s, size, c), b) for k in (3, 5, 7) for s in (1, 2) for size, c, b in t.DEPTHWISE],
                stem=[(t.input_layer_net(r, s, w), b) for r, s, w, b in t.INPUT_LAYERS])


def test_nets_of_the_gpu_tests_reach_their_kernels(tmp_path):
    """Every variant of the tile, few-pixel, depthwise and input-layer kernels that a full-size SubNet reaches is reached by a net
    of test_gpu_layer_kernels.py."""
    out = run(tmp_path, '''
seen = {}
for dtype in ("bf16", "int8", "fp32"):
    tile, small = set(), set()
    for arch, batch in DATA["tiled"] if dtype != "fp32" else ():
        tile |= {(k[1][0], o["R"], o["stride"], o["res"]) for o, k in layers(arch, dtype, batch) if k[0] == "conv_tile_kernel"}
    for arch, batch in DATA["few"]:
        small |= {(k[3] // 64, o["R"], o["stride"], o["res"]) for o, k in layers(arch, dtype, batch) if k[0] == "conv_small_kernel" and o["kind"] == 0}
    seen[dtype] = (tile, small)
seen["dw"] = {(k[0], tuple(k[1])) for arch, batch in DATA["depthwise"] for o, k in layers(arch, "bf16", batch) if o["kind"] == 1}
seen["stem"] = {(k[0], tuple(k[1]) if k[0] == "stem_mfma_kernel" else (), o["stride"]) for arch, batch in DATA["stem"]
                for o, k in layers(arch, "bf16", batch)[:1]}
print(repr(seen))
''', _nets_of_gpu_tests())
    seen = eval(out)
    # (wave groups, taps per side, stride, residual)
    tile = {(1, 1, 1, 0), (1, 1, 1, 1), (1, 1, 2, 0), (2, 1, 1, 0), (2, 1, 1, 1), (2, 1, 2, 0), (1, 3, 1, 0), (1, 3, 2, 0), (2, 3, 1, 0), (2, 3, 2, 0),
            (4, 3, 2, 0)}  # (long 3x3 reductions with stride 1 run in conv_ksplit_kernel: test_gpu_split_reduction.py)
    assert seen["bf16"][0] >= tile and seen["int8"][0] >= tile | {(4, 1, 1, 0)}, seen
    for dtype in ("bf16", "int8", "fp32"):
        small = seen[dtype][1]
        assert {w for w, _, _, _ in small} >= {1, 2, 3, 4} | ({8} if dtype == "fp32" else set()) and {(r, s, res) for _, r, s, res in small} >= {(1, 1, 0), (1, 1, 1), (1, 2, 0), (3, 1, 0), (3, 2, 0)}, small
    want = {("dw_mfma_kernel", v) for v in ((3, 1, 1, 3), (3, 2, 1, 3), (5, 1, 1, 5), (5, 1, 8, 5), (5, 2, 1, 5), (5, 2, 4, 4), (7, 1, 1, 7), (7, 1, 7, 4),
                                            (7, 2, 1, 7), (7, 2, 4, 3))}
    assert seen["dw"] >= want and {(k, v[:2]) for k, v in seen["dw"]} >= {("dwconv_rows_kernel", (r, s)) for r in (3, 5, 7) for s in (1, 2)}, seen["dw"]
    assert seen["stem"] == {("stem_mfma_kernel", v, s) for v in ((1, 1), (1, 4), (2, 1), (2, 4)) for s in (1, 2)} | {("conv_direct_kernel", (), s) for s in (1, 2)}, seen["stem"]


def test_launches_do_not_write_what_they_read(tmp_path):
    """No launch writes memory that it reads (its workgroups run in any order), and what a launch reads is whole what one launch
    before it wrote and none has touched since: layer by layer and with layers fused, in the arena and in the static array,
    launched and recorded as a graph."""
    out = run(tmp_path, '''
from workloads import streams
from workloads.rng import Stream
SELF = 4096  # (where infer's caller keeps its image and its logits)


def overlap(a, b):
    return a[0] < b[0] + b[1] and b[0] < a[0] + a[1]


def faults(launches):
    found, written = [], []  # (of the memory written so far, what still holds)
    for i, (name, reads, writes) in enumerate(launches):
        for w in writes:
            found += [(i, name, "writes what it reads") for r in reads if overlap(r, w)]
            found += [(i, name, "writes twice") for v in writes if v is not w and overlap(v, w)]
        found += [(i, name, "reads what is not there") for r in reads if r[0] != SELF and r not in written]
        written = [v for v in written if not any(overlap(v, w) for w in writes)] + writes
    return found


p = ctypes.c_void_p(SELF)
seen = {}
for arch, dtype in ((A.mbv3_arch(), "bf16"), (A.resnet_arch(), "bf16"), (A.resnet_arch(), "int8"), (A.mbv3_arch(), "fp32"), (A.tiny_arch(), "fp32")):
    ctx = context(arch, dtype)
    nets = [A.min_cfg(arch), A.max_cfg(arch)] + [streams.uniform_cfg(arch, Stream(n), max(arch.res_choices)) for n in (3, 7)]
    for option in (None, 0) if dtype == "bf16" else (None,):  # (once the threshold is set every layer is a launch of its own)
        if option is not None:
            ctx.sushi_set_option(S.OPT_PATCH_CONV_MIN_PIXELS, option)
        for mode in (0, 1, "static"):
            if dtype == "int8" and mode == 1:
                continue
            if mode != "static":
                ctx.sushi_set_option(S.OPT_EXEC_MODE, mode)
            for k, cfg in enumerate(nets):
                for batch in (1, 5, 96):
                    c = ctx.marshal_cfg(cfg)
                    if mode == "static":
                        query = lambda: binding.lib().sushi_infer_static(ctx._h, ctypes.byref(c), p, batch, p) in (0, -2) or sys.exit("static")
                    else:
                        query = lambda: ctx.infer_marshalled(c, p, batch, p)
                    launches = memory(dtype, query)
                    for name, _, _ in launches:
                        seen[name, mode] = seen.get((name, mode), 0) + 1
                    bad = faults(launches)
                    if bad:
                        print(arch.family, dtype, option, mode, k, batch, len(bad), bad[0])
    ctx.close()
for name in ("expand_dw_kernel", "se_gate_kernel", "gate_kernel", "conv_patch_kernel", "conv_small_kernel", "conv_tile_kernel", "conv_ksplit_kernel"):
    print(name, min(seen.get((name, mode), 0) for mode in (0, 1)) > 30, seen.get((name, "static"), 0) > 0 or name in ("conv_patch_kernel", "conv_ksplit_kernel"))
''')
    names = ("expand_dw_kernel", "se_gate_kernel", "gate_kernel", "conv_patch_kernel", "conv_small_kernel", "conv_tile_kernel", "conv_ksplit_kernel")
    assert out.splitlines() == [name + " True True" for name in names], out


COUNT_SEARCHES = '''
#define __HIP_PLATFORM_AMD__ 1
#include "%s/paper_2306_17266_amd/csrc/kernels.h"
static int calls = 0;
extern "C" int searches() { return calls; }
sushi::ExpandDwGeom sushi::expand_dw_geom(const ExpandDwArgs &) {  // (in place of the library's)
    ExpandDwGeom g{};
    g.total = g.workers = g.groups = g.parts = 1;
    return ++calls, g;
}
'''


def test_tile_search_only_where_layers_run_fused(tmp_path):
    """The search for an expansion's tile costs a new SubNet's first query some microseconds per block: only queries that launch
    fused layers make it, not those of the persistent kernels or of a caller's threshold, which never launch one."""
    src, lib = str(tmp_path / "count.cpp"), str(tmp_path / "libcount.so")
    with open(src, "w") as f:
        f.write(COUNT_SEARCHES % ROOT)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-w", "-I/opt/rocm/include", src, "-o", lib], check=True)
    out = run(tmp_path, '''
count = ctypes.CDLL(DATA, mode=ctypes.RTLD_GLOBAL)  # (before the library is loaded)
arch = A.mbv3_arch()
for option, value in ((S.OPT_EXEC_MODE, 2), (S.OPT_EXEC_MODE, 3), (S.OPT_PATCH_CONV_MIN_PIXELS, 0), (S.OPT_EXEC_MODE, 1), (S.OPT_EXEC_MODE, 0)):
    ctx = context(arch)
    ctx.sushi_set_option(option, value)
    before = count.searches()
    try:
        infer(ctx, A.max_cfg(arch), 1)
    except S.SushiError:
        pass  # (the stand-in cannot run a persistent kernel; the plan was made)
    first = count.searches()
    if option == S.OPT_PATCH_CONV_MIN_PIXELS or value < 2:
        infer(ctx, A.max_cfg(arch), 1)
    print(first - before, count.searches() - first)
    ctx.close()
''', lib)
    first = [line.split()[0] for line in out.splitlines()]
    assert first[:3] == ["0"] * 3 and first[3] == first[4] and int(first[4]) > 10, out
    assert all(line.split()[1] == "0" for line in out.splitlines()), out


def test_gated_layer_of_the_gpu_tests_exceeds_one_round_of_the_chip(tmp_path):
    """A net of test_gpu_fused_blocks.py has a gated 1x1 layer with more workgroups than run at once (1024: four of 256 threads
    and 35 KB of LDS on each of 256 compute units)."""
    from tests import test_gpu_fused_blocks as t
    out = run(tmp_path, '''
arch, batch = DATA
print(max(k[2] for k in infer(context(arch), A.max_cfg(arch), batch) if k[0] == "conv_tile_kernel" and k[1][-1] == 1))
''', (t.block_net(6, 3, (1, 2), A.ACT_HSWISH, 56, 40), 96))
    assert int(out) > 1024, out
