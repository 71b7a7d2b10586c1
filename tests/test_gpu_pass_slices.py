"""GPU parity of the rank-wide passes cut into K slices: around the lengths and the numbers of items at which the rule changes its
mind (two, three and six round trips of 2048 values; 64 and 128 blocks), both layouts, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2604_16400_amd import workloads as wl

from gpu_util import TOL, DeviceLayer, check_full, make_ctx

pytestmark = pytest.mark.gpu


def _check(d_in, d_out, ranks, lens, transposed, seed):
    """Every tensor of a forward and a backward call; every second segment trains."""
    n = len(lens)
    ads = [i % len(ranks) for i in range(n)]
    w = wl.make_adhoc("slices", "bf16", d_in, d_out, ranks, lens, ads, [i % 2 for i in range(n)], scale=0.7, seed=seed)
    t = wl.make_tensors(w)
    ctx = make_ctx(w)
    layer = DeviceLayer(w, t, ctx, transposed=transposed)
    layer.fwd(h_save=True)
    layer.bwd(h_save=True)
    check_full(layer, TOL["bf16"], check_h=True)
    layer.bwd(h_save=False)  # h computed again by a pass of its own
    check_full(layer, TOL["bf16"], check_h=True)
    ctx.close()


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("K", [4096, 4104, 6152, 8200, 12288, 12296])  # the last slice is short, or the chain is long enough for the other rule
def test_lengths(K, transposed):
    _check(K, 72, [16, 8, 16], [33, 17, 1, 40], transposed, seed=K)
    _check(40, K, [32, 24], [33, 17, 1, 40], transposed, seed=K)


@pytest.mark.parametrize("items", [64, 65, 128, 129])  # four slices, two, none
def test_items(items):
    _check(8200, 24, [8, 16], [1] * items, False, seed=items)
    _check(24, 8200, [8, 32], [1] * (2 * items), False, seed=items)


@pytest.mark.parametrize("transposed", [False, True])
def test_ranks_no_multiple_of_eight(transposed):
    _check(4104, 6152, [12, 20, 3], [33, 17, 1, 40, 5], transposed, seed=5)
