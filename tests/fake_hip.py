"""Runs host code of the library on tests/fake_hip.cpp, a stand-in for the HIP runtime that checks launches against the
documented limits and logs them instead of running them.  The code runs in a process of its own, which never loads the
real runtime (so no torch there), with these helpers around it."""
import os
import pickle
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = '''
import ctypes, dataclasses, re, sys
sys.path.insert(0, %r)
import numpy as np
import paper_2306_17266_amd as S
from paper_2306_17266_amd import binding
from workloads import arch as A
from workloads import tensors as T
fake = ctypes.CDLL("libamdhip64.so.7")
fake.fake_log.restype = fake.fake_memory_log.restype = ctypes.c_char_p


def context(arch, dtype="bf16", device=0):
    table = S.sushi_describe_supernet(arch)
    ctx = S.Sushi(device, 0)
    if dtype == "int8":
        dense = [s for _, s, k in table if k in (T.KIND_CONV, T.KIND_FC)]
        words = [w for s in dense for w in (np.zeros(s[0]), np.ones(s[0]), np.zeros(s[0] + 8))]  # multipliers, shifts, the rest
        ctx.sushi_load_supernet_int8(arch, np.zeros(sum(int(np.prod(s)) for s in dense), np.int8), np.concatenate(words).astype(np.int32))
    else:
        ctx.sushi_load_supernet(arch, np.zeros(sum(int(np.prod(s)) for _, s, _ in table), np.float32), S.BF16 if dtype == "bf16" else S.FP32)
    return ctx


def kernel_name(mangled):
    """(the kernel's name, what stands behind it)"""
    at = next(m for m in re.finditer(r"(?<!\\d)\\d+", mangled) if mangled[m.end():m.end() + int(m.group())].endswith("_kernel"))
    end = at.end() + int(at.group())
    return mangled[at.end():end], mangled[end:]


def infer(ctx, cfg, batch):
    """One query; its launches as (kernel, template arguments, workgroups, threads per workgroup, bytes of dynamic LDS)."""
    fake.fake_clear_log()
    ctx.infer_marshalled(ctx.marshal_cfg(cfg), ctypes.c_void_p(4096), batch, ctypes.c_void_p(4096))
    out = []
    for line in fake.fake_log().decode().splitlines():
        _, wgs, threads, lds, name = line.split()
        short, rest = kernel_name(name)
        args = [int(v) for v in re.findall(r"L(?:[ib]|NS_\\w+?E)(\\d+)E", rest)]
        out.append((short, args, int(wgs), int(threads), int(lds)))
    return out


def memory(dtype, query):
    """query() and the activations that its launches read and write: [(kernel, reads, writes)], each a list of (address, bytes)."""
    fake.fake_element_bytes({"fp32": 4, "bf16": 2, "int8": 1}[dtype])
    fake.fake_clear_log()
    query()
    out = []
    for line in fake.fake_memory_log().decode().splitlines():
        name, *rest = line.split()
        ranges = [(how, int(at), int(n)) for how, at, n in zip(rest[::3], rest[1::3], rest[2::3])]
        out.append((kernel_name(name)[0], [r[1:] for r in ranges if r[0] == "r"], [r[1:] for r in ranges if r[0] == "w"]))
    return out


def layers(arch, dtype, batch):
    """The launches of the largest SubNet's query with what they compute: [(op of the plan, launch)]."""
    ctx = context(arch, dtype)
    cfg = A.max_cfg(arch)
    ops, launches = S.sushi_team_plan(arch, cfg, batch, 32), infer(ctx, cfg, batch)
    ctx.close()
    assert len(ops) == len(launches)
    return list(zip(ops, launches))
''' % ROOT


def run(tmp_path, code, data=None):
    """Runs PRELUDE and `code` with `data` (anything pickle takes) as DATA; returns what it printed."""
    lib = os.path.join(str(tmp_path), "libamdhip64.so.7")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-w", "-I/opt/rocm/include", "-Wl,-soname,libamdhip64.so.7",
                    "-Wl,--version-script=" + os.path.join(HERE, "fake_hip.map"), os.path.join(HERE, "fake_hip.cpp"), "-o", lib], check=True)
    with open(os.path.join(str(tmp_path), "data"), "wb") as f:
        pickle.dump(data, f)
    code = "import pickle\nDATA = pickle.load(open(%r, 'rb'))\n" % os.path.join(str(tmp_path), "data") + code
    env = dict(os.environ, LD_LIBRARY_PATH=str(tmp_path))
    res = subprocess.run([sys.executable, "-c", PRELUDE + code], env=env, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert res.returncode == 0, res.stdout
    return res.stdout
