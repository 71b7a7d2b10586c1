"""GPU parity of the fp32 GEMM's block shapes (16 rows by 16, 32 or 64 columns, 32 rows) and of the backward passes that share
a launch, against the fp64 oracle (bar: TOL)."""
import numpy as np
import pytest

from paper_2604_16400_amd import workloads as wl

from gpu_util import TOL, DeviceLayer, check_full, make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("d_in,d_out,lens", [
    (520, 1028, [150, 31, 79]),    # forward 32 rows (289 blocks of 16 x 64), dX 64 columns (135), or 16 (K-major, steps)
    (1028, 524, [33, 150, 279]),   # forward 32 rows, K no multiple of 16; dX of 312 rows 32 columns (340, K 524)
    (68, 740, [700, 31, 369]),     # forward 32 rows (828 blocks), dX 64 columns of its 68
    (36, 1000, [700, 31, 369]),    # forward 32 rows (1104)
    (20, 12, [15, 1, 1]),          # a block wider than the output
    (1036, 292, [33, 150, 71]),    # forward 32 columns (80, K 1036)
    (1036, 516, [33, 150, 71]),    # forward 64 columns (144)
    (524, 1100, [700, 31, 369]),   # forward 32 rows, loads not ahead (1242, K 524)
])
def test_gemm_blocks(d_in, d_out, lens, transposed):
    w = wl.make_adhoc("f32", "f32", d_in, d_out, [5, 20, 16], lens, [0, 1, 2], [1, 0, 1], scale=0.5, seed=3)
    ctx = make_ctx(w)
    layer = DeviceLayer(w, wl.make_tensors(w), ctx, transposed=transposed)
    layer.fwd()
    layer.bwd()
    check_full(layer, TOL["f32"])
    ctx.close()


@pytest.mark.parametrize("grad_streams", [0, 1])
@pytest.mark.parametrize("transposed", [False, True])
def test_passes_in_one_launch_give_what_they_give_apart(transposed, grad_streams):
    # profiling keeps every pass a launch of its own: the same sums in the same order, to the bit
    import torch

    w = wl.make_adhoc("f32", "f32", 132, 200, [20, 8, 33, 4], [40, 3, 17, 30, 1], [0, 1, 2, 0, 3], [1, 0, 1, 1, 1], scale=0.5, seed=4)
    out = []
    for apart in (False, True):
        ctx = make_ctx(w)
        ctx.set_grad_streams(grad_streams)
        layer = DeviceLayer(w, wl.make_tensors(w), ctx, transposed=transposed)
        ctx.profile_enable(apart)
        layer.fwd()
        layer.bwd()
        layer.bwd(accumulate=True)
        got = [layer.dx.clone()] + [t.clone() for t in layer.dA + layer.dB]
        layer.bwd(h_save=False)
        layer.bwd(dx=False)
        got += [layer.dx] + layer.dA + layer.dB
        torch.cuda.synchronize()
        out.append(got)
        ctx.close()
    for a, b in zip(*out):
        assert torch.equal(a.nan_to_num(7.0), b.nan_to_num(7.0))
