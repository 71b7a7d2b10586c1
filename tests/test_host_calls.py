"""What a call puts on the device and launches, checked on the CPU: the library runs against a HIP runtime that launches nothing
(fake_hip.cpp) in a process of its own, one per scenario (`python test_host_calls.py <library of the runtime> <scenario> <arguments>`)."""
from __future__ import annotations

import ctypes
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="session")
def run(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake_hip") / "libfake_hip.so")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-w", "-fPIC",
                    "-shared", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2604_16400_amd", "csrc"),
                    os.path.join(HERE, "fake_hip.cpp"), "-o", so], check=True, capture_output=True, text=True)

    def go(scenario, *args):
        r = subprocess.run([sys.executable, os.path.abspath(__file__), so, scenario, *map(str, args)], capture_output=True, text=True,
                           timeout=120)
        assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]

    return go


@pytest.mark.parametrize("dtype,n_adapters", [("bf16", 3), ("bf16", 130), ("f32", 3)])  # 130: more than a pass carries
@pytest.mark.parametrize("call", ["fwd", "bwd"])
def test_eager_calls_behind_a_replay_find_their_own_plan(run, call, dtype, n_adapters):
    run("behind_a_replay", call, dtype, n_adapters)


@pytest.mark.parametrize("call", ["fwd", "bwd"])
def test_a_replay_brings_its_own_plan(run, call):
    run("replay", call)


def test_plans_of_recorded_calls_beyond_the_room_for_them(run):
    run("many_recorded")


def test_calls_without_a_context_upload_when_recorded_and_ever_after(run):
    run("noalloc")


@pytest.mark.parametrize("dtype,n_adapters,call,fail", [
    ("f32", 3, "fwd", "plan_copy_kernel"), ("bf16", 130, "fwd", "plan_copy_kernel"), ("f32", 3, "bwd", "plan_copy_kernel"),
    ("bf16", 3, "fwd", "SkinnyPassArgs"), ("bf16", 3, "bwd", "SkinnyPassArgs"), ("bf16", 3, "fwd", "query"), ("bf16", 3, "bwd", "query")])
def test_a_call_behind_a_failed_upload_uploads(run, dtype, n_adapters, call, fail):
    run("failed_upload", dtype, n_adapters, call, fail)


@pytest.mark.parametrize("kind,kernel,call", [(k, n, c) for k, n in [("items", "skinny_kernel"), ("tiles", "WideArgs"), ("mixed", "MixedArgs")]
                                              for c in ("fwd", "bwd")] + [("decode", "decode_base", "fwd")])
def test_new_tables_carried_by_a_pass_leave_the_plan_of_a_whole_upload(run, kind, kernel, call):
    run("carried", kind, kernel, call)


def test_every_launch_has_asked_for_its_lds(run):
    run("lds")


@pytest.mark.parametrize("rows,d_in,d_out,streams,want", [
    (512, 4096, 4096, 1, "128, 128 sliced 4"), (512, 4096, 4096, 0, "128, 128 sliced 4"),  # K slices in the ring on either stream
    (640, 2048, 4096, 1, "128, 128 sliced 4"), (640, 2560, 10240, 1, "128, 128 sliced 0"),
    (1792, 4096, 4096, 1, "128, 128 whole 0"), (1792, 4096, 4096, 0, "256, 128 whole 3"),  # tiles for one round not beside gradients
    (256, 16384, 1016, 1, "128, 128 whole 0"), (256, 16384, 1016, 0, "128, 128 whole 4")])  # ... nor the ring uncut
def test_the_dx_gemm_beside_gradient_kernels(run, rows, d_in, d_out, streams, want):
    run("dx_gemm", rows, d_in, d_out, streams, want)


@pytest.mark.parametrize("rows,d_in,d_out,tiles,slices", [(247, 7384, 1792, 116, 2), (96, 4160, 1536, 33, 6), (1792, 4096, 4096, 448, 1)])
def test_the_launch_of_the_dx_gemm_and_the_gradients(run, rows, d_in, d_out, tiles, slices):
    run("shared_launch", rows, d_in, d_out, tiles, slices)


@pytest.mark.parametrize("rows,d_in,d_out,rank,want", [
    (1152, 1024, 1024, 64, 1), (1153, 1024, 1024, 64, 0), (4736, 512, 1024, 16, 1), (4737, 512, 1024, 16, 0), (1300, 4864, 9216, 64, 1), (1300, 4864, 8192, 64, 0)])
def test_gradients_of_many_rows_are_not_in_the_dx_gemm_s_launch(run, rows, d_in, d_out, rank, want):
    run("many_rows", rows, d_in, d_out, rank, want)


@pytest.mark.parametrize("rows,d_in,d_out,layout,rank,n,fwd,dx", [
    (64, 256, 1024, 0, 8, 1, "16x16", "16x16+dA"), (128, 1024, 512, 0, 8, 1, "16x16", "16x16+dA"),
    (256, 1024, 512, 0, 8, 1, "16x32", "16x64+dA"), (256, 1024, 512, 0, 128, 16, "16x16", "16x16+dA"),  # steps
    (512, 256, 512, 0, 8, 1, "16x64", "16x16+dA"), (512, 256, 512, 1, 64, 16, "16x16", "16x16+dA"),
    (272, 1024, 1024, 0, 8, 1, "32x64", "16x32+dA"), (272, 2048, 1024, 0, 8, 1, "32x64", "32x64"),
    (400, 512, 1024, 0, 64, 32, "16x16", "16x16+dA"), (400, 512, 1024, 1, 32, 32, "16x16", "16x64+dA"), (400, 1024, 1024, 1, 64, 32, "16x16", "16x32+dA"),
    (1100, 1024, 1024, 0, 8, 1, "32x64 late", "32x64 late"), (1100, 512, 1024, 0, 8, 1, "32x64", "32x64")])
def test_blocks_of_the_fp32_gemm(run, rows, d_in, d_out, layout, rank, n, fwd, dx):
    run("f32_blocks", rows, d_in, d_out, layout, rank, n, fwd, dx)


@pytest.mark.parametrize("rows,d_in,d_out,layout,adapter,low,high", [
    (8, 616, 13376, 1, -1, 0, 0), (8, 4096, 4096, 0, -1, 0, 0),  # no row with an adapter: the general path
    (16, 9656, 14256, 0, 0, 2 * 112, 256),    # 112 strips: one slice leaves more than half of the CUs idle
    (3, 18312, 16384, 0, 0, 2 * 128 + 1, 512),  # 128 strips and the shrink: one slice or a second, partial round
    (34, 15104, 768, 0, 0, 6 * 6, 6 * 17 + 8 * 3), (64, 1024, 4096, 0, 0, 32, 256)])  # few blocks add the slices
def test_blocks_of_a_decode_sized_call(run, rows, d_in, d_out, layout, adapter, low, high):
    run("decode_blocks", rows, d_in, d_out, layout, adapter, low, high)


@pytest.mark.parametrize("rows,d_in,d_out,rank,fetched", [
    (52, 7392, 672, 8, 1), (39, 11184, 928, 32, 1),  # uncut with the gradients in the launch (alone it would be cut)
    (96, 4160, 1536, 16, 0), (1792, 4096, 4096, 16, 1)])  # in slices; two streams' worth of tiles
def test_the_dh_pass_fetches_the_weight_for_the_gemm_that_runs(run, rows, d_in, d_out, rank, fetched):
    run("fetched_weight", rows, d_in, d_out, rank, fetched)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_a_dx_in_the_place_of_what_the_gradients_read_comes_behind_them(run, dtype):
    run("overlapping", dtype)


# ---------------------------------------------------------------------------------------------------------------------------
# the process of a scenario

STREAM = 0x5000


class Batch:
    """A batch, and its calls through a context; adapters' tables and gradients by layer."""

    def __init__(self, w, ctx, lens, ads, trn, ranks, d_in=256, d_out=512, dtype="bf16", layout=0):
        self.w, self.lib, self.ctx = w, w.lib, ctx
        self.T, S, self.N = sum(lens), len(lens), len(ranks)
        arr = lambda t, v: (t * max(len(v), 1))(*v)
        starts = [sum(lens[:k]) for k in range(S + 1)]
        self.seg = (arr(ctypes.c_int32, ranks), arr(ctypes.c_int32, starts), arr(ctypes.c_int32, ads), arr(ctypes.c_uint8, trn))
        self.shape = w.binding.collm_shape(d_in, d_out, self.T, S, self.N, 1 if dtype == "bf16" else 0, 1.0, layout)
        self.tok = [k for k in range(S) for _ in range(lens[k])]

    def _tab(self, layer, kind):
        return (ctypes.c_void_p * self.N)(*[0x100000000 * (1 + layer) + 0x10000000 * kind + 0x1000 * a for a in range(self.N)])

    def fwd(self, layer=0, stream=STREAM):
        return self.lib.collm_lora_linear_fwd(self.ctx, ctypes.byref(self.shape), 0x10000, 0x20000, self._tab(layer, 0), self._tab(layer, 1),
                                              *self.seg, 0x30000, 0x40000, stream)

    def bwd(self, layer=0, stream=STREAM, dx=0x60000000, grads=0, x=0x10000, dy=0x50000000, h=0x40000000):
        g = (self._tab(grads, 2), self._tab(grads, 3)) if grads is not None else (None, None)
        return self.lib.collm_lora_linear_bwd(self.ctx, ctypes.byref(self.shape), x, 0x20000000, self._tab(layer, 0), self._tab(layer, 1),
                                              *self.seg, dy, h, dx, *g, 0, stream)

    def on_device(self):
        """Whether the plan on the device is of this batch (it begins with the segment of every token)."""
        return self.w.fake.fake_plan()[: self.T] == self.tok


class World:
    def __init__(self, so):
        self.fake = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
        self.fake.fake_log.restype = ctypes.c_char_p
        self.fake.fake_plan.restype = ctypes.POINTER(ctypes.c_int32)
        self.fake.fake_capture.argtypes = [ctypes.c_void_p, ctypes.c_int]
        self.fake.fake_fail_launch.argtypes = [ctypes.c_char_p]
        sys.modules["torch"] = None  # (nothing else binds to this runtime)
        sys.path.insert(0, ROOT)
        from paper_2604_16400_amd import binding

        self.binding, self.lib = binding, binding.load_library(build_if_missing=False)

    def context(self, max_tokens=2048, max_segments=64, max_adapters=200, max_rank=128, max_d=16384):
        self.fake.fake_new_plan()
        self.fake.fake_new_graph()
        h = ctypes.c_void_p()
        assert self.lib.collm_ctx_create(ctypes.byref(h), 0, max_tokens, max_segments, max_adapters, max_rank, max_d) == 0
        self.launches()
        return h

    def batches(self, ctx, dtype="bf16", n_adapters=3):
        ranks = [8, 16, 8] + [16] * (n_adapters - 3)
        return [Batch(self, ctx, lens, [0, 1, 2, -1], [1, 0, 1, 0], ranks, dtype=dtype)
                for lens in ([40, 3, 50, 9], [30, 20, 60, 7], [11, 90, 33, 1])]

    def launches(self):
        """[(kernel, grid, LDS bytes, LDS bytes asked for by the attribute)] since the last call of this function"""
        out = []
        for line in self.fake.fake_log().decode().splitlines():
            f = line.split("\t")
            out.append((f[0], tuple(map(int, f[1].split())), int(f[2]), int(f[3])) if len(f) == 4 else (line, (), 0, 0))
        return out

    def stats(self, ctx):
        b, u, n, m = ctypes.c_float(), ctypes.c_float(), ctypes.c_int32(), ctypes.c_int32()
        assert self.lib.collm_debug_plan_stats(ctx, ctypes.byref(b), ctypes.byref(u), ctypes.byref(n), ctypes.byref(m)) == 0
        return m.value, n.value

    def record(self, *calls):
        self.fake.fake_capture(STREAM, 1)
        for c in calls:
            assert c() == 0
        self.fake.fake_capture(STREAM, 0)


def behind_a_replay(w, call, dtype, n_adapters):
    for forms in ([0, 0], [0, 1]):  # the eager calls' layers: nothing new, other tables
        ctx = w.context()
        x, y, _ = w.batches(ctx, dtype, int(n_adapters))
        go = lambda b, layer: (b.fwd if call == "fwd" else b.bwd)(layer)
        w.record(lambda: go(x, 0))
        assert go(y, forms[0]) == 0 and y.on_device()
        w.fake.fake_replay()
        assert x.on_device()
        for layer in forms + forms:
            assert go(y, layer) == 0 and y.on_device(), (forms, layer)
            assert w.stats(ctx)[1] > 4 * 3 * y.T  # all of it
            w.fake.fake_replay()
            assert x.on_device()
        w.lib.collm_ctx_destroy(ctx)


def replay(w, call):
    ctx = w.context()
    x, y, z = w.batches(ctx)
    go = lambda b, layer=0: (b.fwd if call == "fwd" else b.bwd)(layer)
    assert go(x) == 0  # (warmed up: nothing is new when it is recorded)
    whole, sent = w.stats(ctx)[1], []
    def note(b, layer):
        r = go(b, layer)
        sent.append(w.stats(ctx)[1])
        return r
    w.record(lambda: note(x, 0), lambda: note(x, 0), lambda: note(x, 1))
    assert sent == [whole, 0, whole]  # the second finds what the first brings, whatever ran between the replays
    for k in range(40):  # more uploads than staging slots
        b = (y, z)[k % 2]
        assert go(b, k % 3) == 0 and b.on_device()
    for _ in range(3):
        w.fake.fake_replay()
        assert x.on_device()
        assert go(y) == 0 and y.on_device()
    # two captures in a row: a graph brings its own plan, as the other need not have run before it
    w.fake.fake_new_graph()
    w.record(lambda: note(x, 1))
    w.fake.fake_new_graph()
    w.record(lambda: note(x, 1), lambda: note(x, 1))
    assert sent[3:] == [whole, whole, 0]
    # an eager call on another stream while one is captured
    w.fake.fake_new_graph()
    w.fake.fake_capture(STREAM, 1)
    assert note(x, 0) == 0 and (y.fwd if call == "fwd" else y.bwd)(0, STREAM + 1) == 0 and note(x, 0) == 0
    w.fake.fake_capture(STREAM, 0)
    assert sent[6:] == [whole, whole]
    w.fake.fake_replay()
    assert x.on_device()


def many_recorded(w):
    # 2048 tokens, recorded with new tables until the room for kept plans is used up: the rest travel in kernel arguments
    ctx = w.context()
    x = Batch(w, ctx, [2000, 48], [0, 1], [1, 0], [16, 8])
    w.fake.fake_capture(STREAM, 1)
    kinds = []
    for k in range(2 * (64 << 20) // 40000):
        assert x.fwd(k % 2) == 0
        names = [l[0] for l in w.launches()]
        kinds.append("words" if any("plan_words" in n for n in names) else "copy" if any("plan_copy" in n for n in names) else "none")
    w.fake.fake_capture(STREAM, 0)
    kept = kinds.index("words")
    assert set(kinds[:kept]) == {"copy"} and set(kinds[kept:]) == {"words"}
    assert 0.9 * (64 << 20) < kept * w.stats(ctx)[1] <= 64 << 20
    w.fake.fake_replay()
    assert x.on_device()


def noalloc(w):
    x, y, _ = w.batches(None)
    def go(b, layer=0):
        assert w.lib.collm_lora_linear_fwd_noalloc(0, ctypes.byref(b.shape), 0x10000, 0x20000, b._tab(layer, 0), b._tab(layer, 1), *b.seg,
                                                   0x30000, None, STREAM) == 0
        return sum("plan_words" in l[0] for l in w.launches())
    assert go(x) > 0 and go(x) == 0
    w.fake.fake_capture(STREAM, 1)
    assert go(x) > 0
    w.fake.fake_capture(STREAM, 0)
    assert go(x) > 0 and go(x) > 0


def failed_upload(w, dtype, n_adapters, call, fail):
    ctx = w.context()
    b = w.batches(ctx, dtype, int(n_adapters))[0]
    go = lambda layer: (b.fwd if call == "fwd" else b.bwd)(layer)
    assert go(0) == 0
    w.launches()
    w.fake.fake_fail_query(1) if fail == "query" else w.fake.fake_fail_launch(fail.encode())
    assert go(1) == -8
    w.fake.fake_fail_query(0)
    w.launches()
    assert go(1) == 0
    assert any("plan_copy" in l[0] or "PassArgs" in l[0] for l in w.launches()), "computed with the tables of the call before"
    assert go(1) == 0
    assert not any("plan_copy" in l[0] or "PassArgs" in l[0] for l in w.launches())


def carried(w, kind, kernel, call):
    # and a failed launch of the pass leaves no plan to reuse; a replay brings a plan of its own
    ranks = {"items": [8, 16, 16], "tiles": [64, 64, 64], "mixed": [12, 64, 20], "decode": [8, 64, 16]}[kind]
    lens, trn = ([1, 5, 9], [0, 0, 0]) if kind == "decode" else ([40, 33, 50], [1, 1, 1])
    go = lambda b, layer: (b.fwd if call == "fwd" else b.bwd)(layer)
    plans = []
    for layers in ([0, 1], [1]):
        ctx = w.context()
        b = Batch(w, ctx, lens, [0, 1, 2], trn, ranks, 1024, 1024)
        whole = 0
        for layer in layers:
            w.launches()
            assert go(b, layer) == 0
            whole = max(whole, w.stats(ctx)[1])
        names = [l[0] for l in w.launches()]
        if len(layers) == 2:
            assert any(kernel in n and "PassArgs" in n or "WideArgs" in n and kernel == "WideArgs" for n in names) and not any("plan_copy" in n for n in names), names
        plans.append(w.fake.fake_plan()[: whole // 4])
    assert plans[0] == plans[1]
    assert go(b, 0) == 0
    w.fake.fake_fail_launch(b"WideArgs" if kernel == "WideArgs" else b"SkinnyPassArgs")
    assert go(b, 1) == -8
    w.launches()
    assert go(b, 1) == 0 and any("plan_copy" in l[0] for l in w.launches()) and w.fake.fake_plan()[: whole // 4] == plans[0]
    x, y = Batch(w, ctx, lens, [0, 1, 2], trn, ranks, 1024, 1024), Batch(w, ctx, lens, [2, 1, 0], trn, ranks, 1024, 1024)
    w.record(lambda: go(x, 1))
    assert go(y, 0) == 0
    w.fake.fake_replay()
    assert w.fake.fake_plan()[: whole // 4] == plans[0]


def lds(w):
    # kernels of one signature whose LDS differs, the one with less first: K slices on two stages, then in the ring; the tiled
    # rank-wide pass over both layouts of the tables, with new addresses and without; the gradients beside GEMMs of both sizes
    seen = set()
    for d_in, d_out, T, rank, layout in [(4096, 11008, 64, 64, 0), (4096, 1024, 64, 64, 0), (4096, 1024, 64, 64, 1), (512, 512, 600, 64, 0),
                                         (4096, 4096, 1000, 16, 0), (4096, 4096, 2000, 128, 1), (12288, 16384, 2048, 16, 0)]:
        ctx = w.context()
        b = Batch(w, ctx, [T - 8, 8], [0, 1], [1, 0], [rank, 8], d_in, d_out, layout=layout)
        for layer in (0, 1):
            assert b.fwd(layer) == 0 and b.bwd(layer) == 0
        for name, grid, smem, asked in w.launches():
            assert smem <= max(asked, 65536), (name, smem, asked)
            seen.add((name.split("<", 1)[-1], smem))
        w.lib.collm_ctx_destroy(ctx)
    sliced = {(km, lds) for n, lds in seen for km in ("true", "false") if n.startswith(f"128, 128, 2, 2, {km}, false, false, true, false")}
    assert sliced >= {("false", 65536), ("false", 131072), ("true", 131072)}, seen


def dx_gemm(w, rows, d_in, d_out, streams, want):
    ctx = w.context()
    w.lib.collm_debug_set_grad_streams(ctx, int(streams))
    assert Batch(w, ctx, [int(rows)], [0], [1], [16], int(d_in), int(d_out)).bwd() == 0
    gemms = [l[0].split("<", 1)[1].split(", ") for l in w.launches() if "gemm_lora_kernel" in l[0]]
    gemms = [f"{a[0]}, {a[1]} {'sliced' if a[7] == 'true' else 'whole'} {a[9]}" for a in gemms if a[5] == "false"]
    assert gemms == [want], gemms


def shared_launch(w, rows, d_in, d_out, tiles, slices):
    # one dimension: workgroups start in the order of their ids, the GEMM's of every slice before the gradients'
    ctx = w.context()
    assert Batch(w, ctx, [int(rows)], [0], [1], [16], int(d_in), int(d_out)).bwd() == 0
    got = [(l[0], l[1]) for l in w.launches() if "GemmGradArgs" in l[0]]
    n = len(w.binding.host_shared_order(1, int(tiles), int(slices), int(d_out), -(-int(d_in) // 64) + -(-int(d_out) // 64))[0])
    assert len(got) == 1 and got[0][1] == (n, 1, 1), (got, n)


def many_rows(w, rows, d_in, d_out, rank, want):
    # one gradient block walks all rows of its adapter
    ctx = w.context(max_tokens=8192)
    assert Batch(w, ctx, [int(rows)], [0], [1], [int(rank)], int(d_in), int(d_out)).bwd() == 0
    assert sum("GemmGradArgs" in l[0] for l in w.launches()) == int(want)


def f32_blocks(w, rows, d_in, d_out, layout, rank, n, fwd, dx):
    rows, n = int(rows), int(n)
    ctx = w.context()
    b = Batch(w, ctx, [rows // n + (k < rows % n) for k in range(n)], list(range(n)), [1] * n, [int(rank)] * n, int(d_in), int(d_out), "f32", int(layout))
    def blocks():
        for name, *_ in w.launches():
            a = name.split("<", 1)[-1].rstrip(">").split(", ")
            if "gemm_f32_kernel" in name:
                return f"{16 * int(a[1])}x{16 * int(a[4])}{'' if a[5] == 'true' else ' late'}"
            if "dx_dA_f32_kernel" in name:
                return f"16x{16 * int(a[1])}+dA"
    assert b.fwd() == 0
    got = [blocks()]
    assert b.bwd() == 0
    got.append(blocks())
    assert got == [fwd, dx], got


def decode_blocks(w, rows, d_in, d_out, layout, adapter, low, high):
    ctx = w.context(max_d=20000)
    assert Batch(w, ctx, [int(rows)], [int(adapter)], [0], [16], int(d_in), int(d_out), layout=int(layout)).fwd() == 0
    blocks = [l[1][0] for l in w.launches() if "decode_base_kernel" in l[0]]
    assert int(low) <= sum(blocks) <= int(high) and len(blocks) == (int(high) > 0), blocks


def fetched_weight(w, rows, d_in, d_out, rank, fetched):
    # weights beyond 8 MiB; 256 blocks behind the items of the pass
    ctx = w.context()
    assert Batch(w, ctx, [int(rows)], [0], [1], [int(rank)], int(d_in), int(d_out)).bwd() == 0
    l = w.launches()
    gemm = [x for x in l if "GemmGradArgs" in x[0]]
    dh = [x for x in l if "skinny_kernel" in x[0] or "gemm_lora_kernel<128, 128, 4, 2" in x[0]]
    assert len(gemm) == 1 and len(dh) == 1 and (dh[0][1][0] >= 256) == bool(int(fetched)), l


def overlapping(w, dtype):
    ctx = w.context()
    b = Batch(w, ctx, [100, 28], [0, 1], [1, 0], [16, 16], 256, 512, dtype)
    e = 2 if dtype == "bf16" else 4
    names = ("GemmGradArgs", "dx_dA_f32")
    def shared(**where):
        assert b.bwd(**where) == 0
        return any(n in l[0] for l in w.launches() for n in names)
    x, h, dy, dx = 0x10000, 0x40000000, 0x50000000, 128 * 256 * e  # (dx: bytes)
    assert shared() and shared(dx=x + dx) and shared(x=x + dx, dx=x)  # beside one another
    assert not shared(dx=x) and not shared(dx=x + dx - 16) and not shared(x=x + dx - 16, dx=x)
    if dtype == "bf16":  # (fp32: dB has read them before)
        assert not shared(dx=dy + 16) and not shared(dx=h + 128 * 128 * 4 - 16) and shared(dx=h + 128 * 128 * 4)
        assert not shared(h=0x100000000 + 0x20000000) and shared(h=0x100000000 + 0x20000000 + 256 * 16 * 4)  # dA of adapter 0


if __name__ == "__main__":
    globals()[sys.argv[2]](World(sys.argv[1]), *sys.argv[3:])
