"""GPU parity of the decode-sized inference calls (kernels_decode.hip): rows, strips, slices and ranks at their edges, both
layouts, against the fp64 oracle (bar: TOL, as everywhere), and against the general path on the same inputs."""
import numpy as np
import pytest

import oracle
from paper_2604_16400_amd import workloads as wl

from gpu_util import TOL, DeviceLayer, make_ctx, maxrel, to_host

pytestmark = pytest.mark.gpu


def _batch(rows, n_adapters, seed, base=0.2):
    """Segments of one to a few tokens; a share of them without an adapter."""
    rng = np.random.default_rng(seed)
    lens = []
    while sum(lens) < rows:
        lens.append(min(int(rng.choice([1, 1, 1, 2, 19])), rows - sum(lens)))
    ads = [int(a) if rng.random() >= base else -1 for a in rng.integers(0, n_adapters, size=len(lens))]
    return lens, ads


def _forward(ctx, layer):
    """(y, kernels of the decode path ran) of one forward call"""
    ctx.profile_enable(True)
    layer.fwd(h_save=False)
    names = {n for n, _ in ctx.profile_read()}
    ctx.profile_enable(False)
    return to_host(layer.y), "decode" in names


def _check(rows, d_in, d_out, ranks, transposed, seed, base=0.2, want=True):
    lens, ads = _batch(rows, len(ranks), seed, base)
    w = wl.make_adhoc("decode", "bf16", d_in, d_out, ranks, lens, ads, [0] * len(lens), scale=0.7, seed=seed)
    t = wl.make_tensors(w)
    ctx = make_ctx(w)
    layer = DeviceLayer(w, t, ctx, transposed=transposed)
    y_ref, _ = oracle.lora_linear_fwd(t.x, t.W, t.A, t.B, layer.tok_adapter, w.scale)
    y, ran = _forward(ctx, layer)
    assert ran == want
    assert np.all(np.isfinite(y)), "unwritten"
    assert maxrel(y, y_ref) <= TOL["bf16"]
    layer.y.fill_(float("nan"))
    ctx.set_gemm_split(1)  # the general path, uncut
    y1, ran = _forward(ctx, layer)
    assert not ran
    # both round an fp32 sum once: at most a bf16 step (2^-8) of the larger value, plus the order of the sums
    assert maxrel(y, y1) <= 2.0 ** -8 + 1e-3
    ctx.close()


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("rows", [1, 15, 16, 17, 32, 33, 64])  # around the row tiles of a wave and the row groups of a block
def test_rows(rows, transposed):
    _check(rows, 1024, 392, [16, 8, 16], transposed, seed=rows)


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("d_in,d_out", [(8, 8), (24, 136), (72, 128), (4104, 8), (520, 1160), (6400, 264)])  # tails of K, of the strips
def test_sizes(d_in, d_out, transposed):
    for rows in (5, 40):
        _check(rows, d_in, d_out, [16, 32, 8], transposed, seed=d_in + rows)


@pytest.mark.parametrize("transposed,ranks,want", [
    (False, [8, 16, 64], True), (False, [72, 128, 256, 8], True), (False, [1, 12, 20, 63], True), (False, [100, 16], False),
    (True, [8, 16, 64], True), (True, [72, 128, 256, 8], True), (True, [12, 16], False)])
def test_ranks(transposed, ranks, want):
    for rows in (7, 50):
        _check(rows, 640, 520, ranks, transposed, seed=len(ranks) + rows, want=want)


@pytest.mark.parametrize("transposed", [False, True])
def test_all_rows_on_the_base_weight(transposed):
    _check(37, 256, 384, [16], transposed, seed=3, base=1.0, want=False)  # (no rank-wide pass: the general path)
    _check(37, 256, 384, [16], transposed, seed=3, base=0.0)


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("rows,ranks", [(1, [8]), (4, [16, 8]), (5, [16]), (13, [8, 16]), (64, [8] * 20)])
def test_many_slices(rows, ranks, transposed):
    # a narrow output: up to 32 slices, added eight at a time (items of up to four rows) or two at a time (more rows)
    for d_in, d_out in ((12296, 264), (16384, 136)):
        _check(rows, d_in, d_out, ranks, transposed, seed=rows + d_in, base=0.0 if rows < 8 else 0.2)


@pytest.mark.parametrize("transposed", [False, True])
def test_layers_in_turn_with_tables_of_their_own(transposed):
    # the batch's plan stays, new table addresses ride on the first kernel
    lens, ads = _batch(21, 5, 9)
    ws = [wl.make_adhoc("decode", "bf16", 512, 640, [16, 8, 32, 16, 8], lens, ads, [0] * len(lens), scale=0.7, seed=40 + k) for k in range(3)]
    ctx = make_ctx(ws[0])
    layers = [DeviceLayer(w, wl.make_tensors(w), ctx, transposed=transposed) for w in ws]
    modes = []
    for _ in range(8):  # more than there are staging slots
        for l in layers:
            l.fwd(h_save=False)
            modes.append(ctx.plan_stats()["mode"])
    assert modes[0] == 1 and set(modes[1:]) == {2}
    for l in layers:
        y_ref, _ = oracle.lora_linear_fwd(l.t.x, l.t.W, l.t.A, l.t.B, l.tok_adapter, l.w.scale)
        assert maxrel(to_host(l.y), y_ref) <= TOL["bf16"]
    ctx.close()


@pytest.mark.parametrize("transposed", [False, True])
def test_values_that_are_not_finite_stay_in_their_rows(transposed):
    import torch

    lens, ads = _batch(20, 3, 5, base=0.3)
    ads[0] = 0
    w = wl.make_adhoc("decode", "bf16", 256, 264, [12 if not transposed else 24, 16, 8], lens, ads, [0] * len(lens), scale=0.7, seed=5)
    ctx = make_ctx(w)
    layer = DeviceLayer(w, wl.make_tensors(w), ctx, transposed=transposed)
    layer.B[0].fill_(float("inf"))
    layer.x[0, 0] = float("nan")  # a token of adapter 0
    layer.fwd(h_save=False)
    bad = torch.tensor(layer.tok_adapter == 0, device="cuda")
    bad[0] = True
    assert bool(torch.isfinite(layer.y[~bad].float()).all()) and not bool(torch.isfinite(layer.y[bad].float()).all(1).any())
    ctx.close()


def test_recorded_call_replays_with_new_values():
    import torch

    lens, ads = _batch(21, 5, 9)
    w = wl.make_adhoc("decode", "bf16", 1032, 640, [16, 8, 32, 16, 8], lens, ads, [0] * len(lens), scale=0.7, seed=60)
    t = wl.make_tensors(w)
    ctx, eager = make_ctx(w), make_ctx(w)
    layer, other = DeviceLayer(w, t, ctx), DeviceLayer(w, t, eager)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        layer.fwd(h_save=False)
    s.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        layer.fwd(h_save=False)
    for k in range(3):
        layer.x.mul_(-0.5)
        other.x.copy_(layer.x)
        other.B[0].copy_(layer.B[0].mul_(1.5))
        layer.y.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        other.fwd(h_save=False)
        torch.cuda.synchronize()
        assert torch.equal(layer.y, other.y), k
    ctx.close()
    eager.close()
