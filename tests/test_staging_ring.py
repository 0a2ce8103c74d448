"""The ring of pinned staging buffers against a device that is always behind (CPU only): the host code is built with g++ on
tests/sanitize/queued_device.cpp, whose launches stay in a queue until the host waits for an event behind them and which notices
when words that a queued kernel has still to read are overwritten or freed."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_25412_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

CHILD = """
import ctypes as C, random, sys
import numpy as np
from paper_2510_25412_amd import binding
mode, seed = sys.argv[1], int(sys.argv[2])
lib = binding.load()
near = C.create_string_buffer(64 << 20)
at = C.addressof(near)

def context(layers, pages=4000):
    cfg = binding.make_config(8, 2, 128, 16, "bf16", pages, device=0, pool=at, workspace=at, workspace_bytes=64 << 20, decode_waves=256, n_layers=layers)
    return binding.Context(cfg)

if mode in ("mixed", "blind"):
    lib.queued_be_blind(mode == "blind")
    r, layers = random.Random(seed), 1 + 2 * (seed % 2)
    ctx, files = context(layers), []
    for step in range(400):
        op = r.choice(["append", "append", "pred", "pred", "pred", "raw", "extract", "merge", "fork", "remove", "read", "away"])
        live = r.sample(files, min(len(files), r.randint(1, 12)))
        if op == "append" or not files:
            if len(files) < 24:
                files.append(ctx.kv_open(None))
            ctx.kv_append(r.choice(files), r.choice([1, 17, 300, 2060 if ctx.free_pages() > 2000 else 5]), at, at, None)
        elif op == "pred":
            new = [r.choice([1, 1, 3, 40]) for _ in live]
            if layers == 1:
                ctx.pred_batch(live, new, at, at, at, at, None)
            else:
                ctx.pred_begin(live, new, None)
                for layer in range(layers):
                    ctx.pred_layer(layer, at, at, at, at, None)
        elif op == "raw" and layers == 1:
            live = [f for f in live if ctx.kv_len(f)]
            tables = [ctx.kv_pages(f) for f in live]
            if live:
                ctx.pred_batch_raw([1] * len(live), np.concatenate(tables), np.cumsum([0] + [len(t) for t in tables]), [ctx.kv_len(f) for f in live], at, at, None)
        elif op == "extract":
            idx = [r.sample(range(ctx.kv_len(f)), ctx.kv_len(f) // 2) for f in live]
            for h in ctx.kv_extract_batch(live, idx, None):
                ctx.kv_remove(h)
        elif op == "merge":
            ctx.kv_remove(ctx.kv_merge(live, None))
        elif op == "fork" and len(files) < 24:
            files.append(ctx.kv_fork(live[0]))
        elif op == "remove" and (len(files) > 20 or ctx.free_pages() < 2000):
            files.remove(live[0])
            ctx.kv_remove(live[0])
        elif op == "read" and ctx.kv_len(live[0]):
            ctx.kv_read(live[0], 0, ctx.kv_len(live[0]), at, at, None)
        elif op == "away":
            ctx.kv_offload(live, None)
            ctx.kv_restore(live, None)
        if ctx.free_pages() < 1200:
            for f in files[::2]:
                ctx.kv_remove(f)
            files = files[1::2]
else:
    layers = int(sys.argv[3])
    ctx = context(layers)
    files = [ctx.kv_open(None) for _ in range(3)]
    for f in files:
        ctx.kv_append(f, 20, at, at, None)
    for step in range(300):
        ctx.pred_begin(files, [1] * 3, None)
        for layer in range(layers):
            ctx.pred_layer(layer, at, at, at, at, None)
out = (C.c_int64 * 5)()
lib.queued_finish(out)
print("RESULT", *out)
"""


@pytest.fixture(scope="module")
def queued_lib(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ is not installed")
    out = str(tmp_path_factory.mktemp("queued") / "libsymphony_kv_queued.so")
    srcs = [os.path.join(CSRC, f) for f in ("kvfs.cpp", "desc.cpp", "sched.cpp", "capi.cpp")] + [os.path.join(ROOT, "tests", "sanitize", "queued_device.cpp")]
    cmd = ["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-w", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", f"-I{CSRC}", *srcs, "-o", out]
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout[-4000:]
    return out


def _run(lib, *args):
    p = subprocess.run([sys.executable, "-c", CHILD, *map(str, args)], cwd=ROOT, env=dict(os.environ, SYMPHONY_KV_LIB=lib), stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, text=True, timeout=300)
    assert p.returncode == 0, p.stdout[-4000:]
    line = [x for x in p.stdout.splitlines() if x.startswith("RESULT")][-1]
    return dict(zip(("overwritten", "launches", "records", "waits", "most_unrecorded"), map(int, line.split()[1:])))


@pytest.mark.parametrize("seed", range(4))
def test_no_staging_buffer_is_overwritten_before_it_is_read(queued_lib, seed):
    r = _run(queued_lib, "mixed", seed)
    assert r["launches"] > 300 and r["waits"] > 100      # the ring of four came round again and again
    assert r["overwritten"] == 0


def test_a_wait_that_does_not_wait_is_noticed(queued_lib):
    assert _run(queued_lib, "blind", 0)["overwritten"] > 0


@pytest.mark.parametrize("layers", [1, 3, 80])
def test_launches_between_two_records_are_bounded(queued_lib, layers):
    # the runtime keeps what it knows of finished launches until it meets a recorded event: 256 launches and the rest of a step
    r = _run(queued_lib, "layers", 0, layers)
    assert r["launches"] >= 300 * layers
    assert r["most_unrecorded"] <= 256 + 3 * layers + 1
    assert r["records"] <= r["launches"] / 128      # and a record is no packet of every step
