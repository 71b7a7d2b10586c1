"""GPU parity of backward calls whose gradients run in blocks of the dX GEMM's launch (ranks up to 64, 128x128 tiles that leave places free),
uncut and in K slices: tails of rows, columns and ranks, many adapters, accumulation, h kept or not; against the oracle or fp32, and the two streams."""
import numpy as np
import pytest
import torch

from paper_2604_16400_amd import binding
from paper_2604_16400_amd import workloads as wl

from gpu_util import TOL, DeviceLayer, check_full, make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("d_in,d_out,ranks,lens,slices", [
    (200, 392, [64], [129], 1), (264, 136, [16], [257], 1), (1096, 2056, [16, 5], [65, 300], 9), (72, 1000, [40, 12], [1, 31, 33, 160], 4),
    (1032, 264, [64, 3, 24], [200, 1, 64, 17], 1), (264, 4104, [64, 24], [65, 30], 17),
    (256, 1024, [16] * 20, [8] * 20, 4), (256, 1024, [24] * 20, [8] * 20, 2),  # more trained adapters than travel as arguments
    (136, 520, [48] * 19, [3] * 38, 0)])  # too much work for the places
def test_small(d_in, d_out, ranks, lens, slices, transposed):
    n = len(lens)
    w = wl.make_adhoc("beside", "bf16", d_in, d_out, ranks, lens + [5], [i % len(ranks) for i in range(n)] + [-1], [1] * n + [0], scale=0.7, seed=n)
    t = wl.make_tensors(w)
    ctx = make_ctx(w)
    layer = DeviceLayer(w, t, ctx, transposed=transposed)
    layer.fwd(h_save=True)
    layer.bwd(h_save=True)
    assert ctx.last_call()["grad_slices"] == slices
    check_full(layer, TOL["bf16"])
    once = [g.clone() for g in layer.dA + layer.dB]
    layer.bwd(h_save=True, accumulate=True)
    for g, o in zip(layer.dA + layer.dB, once):
        assert torch.equal(g, o + o)
    layer.bwd(h_save=False)
    assert ctx.last_call()["grad_slices"] == slices
    check_full(layer, TOL["bf16"])
    ctx.close()


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("rows,d_in,d_out,rank,slices", [
    (768, 6944, 1864, 16, 1), (726, 5368, 912, 32, 1), (400, 5632, 2528, 32, 2), (386, 1280, 2816, 64, 6), (411, 1056, 5496, 16, 7),
    (77, 3072, 1208, 16, 5), (130, 7000, 8200, 12, 3), (1792, 4096, 1024, 16, 0), (1000, 2056, 4104, 64, 0)])
def test_large(rows, d_in, d_out, rank, slices, transposed):
    g = torch.Generator(device="cuda").manual_seed(rows)
    rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    st = (lambda a: a.t().contiguous()) if transposed else (lambda a: a)
    bf = lambda a: a.to(torch.bfloat16)
    x, dy, W = bf(rnd(rows, d_in)), bf(rnd(rows, d_out)), bf(0.02 * rnd(d_in, d_out))
    A, B = [bf(rnd(d_in, rank) * d_in ** -0.5) for _ in range(2)], [bf(0.05 * rnd(rank, d_out)) for _ in range(2)]
    cut = rows // 3
    batch = (np.array([rank, rank], np.int32), np.array([0, cut, rows], np.int32), np.array([1, 0], np.int32), np.ones(2, np.uint8), 2.0)
    h = torch.zeros((rows, rank), device="cuda")
    f32 = dict(dtype=torch.float32, device="cuda")
    want_dx, want = dy.float() @ W.float().T, {}
    for a, r in ((1, slice(0, cut)), (0, slice(cut, rows))):
        h[r] = x[r].float() @ A[a].float()
        dh = 2.0 * (dy[r].float() @ B[a].float().T)
        want_dx[r] += dh @ A[a].float().T
        want[a] = x[r].float().T @ dh, 2.0 * h[r].T @ dy[r].float()
    ctx = binding.Context(rows, 2, 2, rank, max(d_in, d_out))
    for streams in (-1, 1):
        ctx.set_grad_streams(streams)
        dx = torch.full((rows, d_in), float("nan"), dtype=torch.bfloat16, device="cuda")
        dA, dB = [torch.full_like(st(a), float("nan"), **f32) for a in A], [torch.full_like(st(b), float("nan"), **f32) for b in B]
        ctx.collm_lora_linear_bwd(x, st(W), [st(a) for a in A], [st(b) for b in B], *batch, dy, h, dx, dA, dB,
                                  layout=binding.LAYOUT_OUT_IN if transposed else binding.LAYOUT_IN_OUT)
        torch.cuda.synchronize()
        assert ctx.last_call()["grad_slices"] == (slices if streams < 0 else 0)
        close = lambda got, ref: float((got.float() - ref).abs().max()) <= TOL["bf16"] * float(ref.abs().max())
        assert close(dx, want_dx)
        for a in (0, 1):
            assert close(st(dA[a]) if transposed else dA[a], want[a][0]) and close(st(dB[a]) if transposed else dB[a], want[a][1])
    ctx.close()
