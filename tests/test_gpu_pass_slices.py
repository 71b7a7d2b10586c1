"""GPU parity of the rank-wide passes cut into K slices: around the lengths and the numbers of items at which the rule changes its
mind (two, three and six round trips of 2048 values; 64 and 128 blocks), both layouts, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2604_16400_amd import workloads as wl

from gpu_util import TOL, DeviceLayer, check_full, make_ctx

pytestmark = pytest.mark.gpu


def _check(d_in, d_out, ranks, lens, transposed, seed, fwd=None, dh=None):
    """Every tensor of a forward and a backward call; every second segment trains.  fwd, dh: the slices of the passes over 16-row items."""
    n = len(lens)
    ads = [i % len(ranks) for i in range(n)]
    w = wl.make_adhoc("slices", "bf16", d_in, d_out, ranks, lens, ads, [i % 2 for i in range(n)], scale=0.7, seed=seed)
    t = wl.make_tensors(w)
    ctx = make_ctx(w)
    layer = DeviceLayer(w, t, ctx, transposed=transposed)
    layer.fwd(h_save=True)
    assert fwd in (None, ctx.last_call()["pass_slices"])
    layer.bwd(h_save=True)
    assert dh in (None, ctx.last_call()["pass_slices"])
    check_full(layer, TOL["bf16"], check_h=True)
    layer.bwd(h_save=False)  # h computed again by a pass of its own
    check_full(layer, TOL["bf16"], check_h=True)
    ctx.close()


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("K", [4096, 4104, 6152, 8200, 12288, 12296])  # the last slice is short, or the chain is long enough for the other rule
def test_lengths(K, transposed):
    want = {4096: 1, 12296: 3}.get(K, 4)
    _check(K, 72, [16, 8, 16], [33, 17, 1, 40], transposed, seed=K, fwd=want)
    _check(K, 40, [32, 24], [33, 17, 1, 40], transposed, seed=K, fwd=want)
    _check(40, K, [16, 8], [33, 17, 1, 40], transposed, seed=K, dh=want)
    _check(40, K, [32, 24], [33, 17, 1, 40], transposed, seed=K, dh=0)  # (tiled)


@pytest.mark.parametrize("items,slices", [(64, 4), (65, 2), (128, 2), (129, 1)])
def test_items(items, slices):
    # (an adapter to each row, so that a row is an item)
    _check(8200, 24, [8 + 8 * (i % 2) for i in range(items)], [1] * items, False, seed=items, fwd=slices)
    _check(24, 8200, [8 + 8 * (i // 2 % 2) for i in range(2 * items)], [1] * (2 * items), False, seed=items, dh=slices)


@pytest.mark.parametrize("transposed", [False, True])
def test_ranks_no_multiple_of_eight(transposed):
    _check(4104, 6152, [12, 20, 3], [33, 17, 1, 40, 5], transposed, seed=5, fwd=4, dh=4)
