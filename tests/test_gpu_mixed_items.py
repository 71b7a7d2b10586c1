"""GPU parity of rank-wide passes whose tiled and 16-row items share a launch (ranks that are no multiples of 8 beside wider ones): lengths at
which the number of slices changes, more blocks of one kind than of the other, both widths of the 16-row items; both layouts, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2604_16400_amd import workloads as wl

from gpu_util import TOL, DeviceLayer, check_full, make_ctx

pytestmark = pytest.mark.gpu


def _check(d_in, d_out, ranks, lens, transposed, seed, mixed=True):
    """Forward, backward with h and without; new adapter tables on a known batch ride on the pass.  mixed: whether the kinds share a launch."""
    n = len(lens)
    w = wl.make_adhoc("mixed", "bf16", d_in, d_out, ranks, lens, [i % len(ranks) for i in range(n)], [(i // len(ranks)) % 2 for i in range(n)], scale=0.7, seed=seed)
    t = wl.make_tensors(w)
    ctx = make_ctx(w)
    for _ in range(2):
        layer = DeviceLayer(w, t, ctx, transposed=transposed)  # (tables of their own)
        layer.fwd(h_save=True)
        assert ctx.last_call()["mixed_passes"] == mixed
        layer.bwd(h_save=True)
        assert ctx.last_call()["mixed_passes"] == mixed
        check_full(layer, TOL["bf16"], check_h=True)
    layer.bwd(h_save=False)
    assert ctx.last_call()["mixed_passes"] == 2 * mixed
    check_full(layer, TOL["bf16"], check_h=True)
    ctx.close()


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("K", [40, 4096, 4104, 8200, 12296])
def test_lengths(K, transposed):
    _check(K, 136, [12, 64, 20], [33, 17, 1, 150, 5, 40], transposed, seed=K)
    _check(72, K, [36, 72, 3], [17, 33, 40, 1, 130, 7], transposed, seed=K + 1)


@pytest.mark.parametrize("ranks,mixed", [([60, 128], True), ([12, 200], True), ([68, 64], False)])  # the last: too wide for the shared launch
def test_ranks(ranks, mixed):
    _check(1032, 2056, ranks, [20, 129, 1, 1, 35, 16], False, seed=ranks[0], mixed=mixed)


@pytest.mark.parametrize("n12,n64", [(130, 2), (2, 70)])  # more 16-row items than half of the places; more tiled ones than places are left
def test_counts(n12, n64):
    _check(1032, 520, [12] * n12 + [64] * n64, [2] * (2 * (n12 + n64)), False, seed=n12)
