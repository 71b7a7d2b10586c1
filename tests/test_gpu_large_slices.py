"""GPU parity of GEMMs in K slices of 256x256 tiles: rows and columns just short of and beyond a tile, contractions whose last slice is
short or no multiple of 64, steps of several groups of rank indices shared by the slices; forward and dX, both layouts, against fp32."""
import numpy as np
import pytest
import torch

from paper_2604_16400_amd import binding

from gpu_util import TOL

pytestmark = pytest.mark.gpu


def _layer(rows, K, cols, ranks, kmajor, train, seed):
    """x W with W [K][cols] (kmajor: stored as its transpose), rows dealt to the adapters in turn, every seventh on the base weight."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda shape, std: (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)
    n = len(ranks)
    cuts = np.unique(np.linspace(0, rows, 3 * n + 1).astype(np.int32))
    ads = np.array([-1 if k % 7 == 6 else k % n for k in range(len(cuts) - 1)], dtype=np.int32)
    is_train = np.array([1 if train and a >= 0 else 0 for a in ads], dtype=np.uint8)
    batch = (np.array(ranks, dtype=np.int32), cuts.astype(np.int32), ads, is_train, 0.7)
    tok_ad = np.repeat(ads, np.diff(cuts))
    st = lambda t: t.T.contiguous() if kmajor else t
    return dict(x=rnd((rows, K), 1.0), W=rnd((K, cols), 0.02), A=[rnd((K, r), K ** -0.5) for r in ranks], B=[rnd((r, cols), 0.1) for r in ranks],
                batch=batch, tok_ad=torch.from_numpy(tok_ad).cuda(), st=st, layout=binding.LAYOUT_OUT_IN if kmajor else binding.LAYOUT_IN_OUT,
                ctx=binding.Context(rows, len(ads), n, max(ranks), max(K, cols)))


CASES = [(1000, 2056, 9216, [16, 8]), (1025, 1800, 14336, [16]), (1020, 2056, 9224, [136, 12, 40]), (255, 8200, 17000, [24, 72])]


@pytest.mark.parametrize("kmajor", [False, True])
@pytest.mark.parametrize("rows,cols,K,ranks", CASES)
def test_forward(rows, cols, K, ranks, kmajor):
    L = _layer(rows, K, cols, ranks, kmajor, False, rows)
    tile, slices, _ = binding.host_plain_gemm(rows, cols, K, kmajor, steps=2 * sum((r + 15) // 16 for r in ranks))
    assert tile == binding.TILE_256x256 and slices > 1
    y = torch.full((rows, cols), float("nan"), dtype=torch.bfloat16, device="cuda")
    L["ctx"].collm_lora_linear_fwd(L["x"], L["st"](L["W"]), [L["st"](a) for a in L["A"]], [L["st"](b) for b in L["B"]], *L["batch"], y, None, layout=L["layout"])
    ref = L["x"].float() @ L["W"].float()
    for a in range(len(ranks)):
        m = L["tok_ad"] == a
        ref[m] += 0.7 * (L["x"][m].float() @ L["A"][a].float()) @ L["B"][a].float()
    assert torch.isfinite(y).all()
    assert (y.float() - ref).abs().max() <= TOL["bf16"] * ref.abs().max()
    L["ctx"].close()


@pytest.mark.parametrize("kmajor", [False, True])
@pytest.mark.parametrize("rows,cols,K,ranks", CASES[1:])
def test_backward(rows, cols, K, ranks, kmajor):
    """dx = dy W^T + s (dy B_a^T) A_a^T of the training rows: the contraction is d_out."""
    L = _layer(rows, cols, K, ranks, kmajor, True, rows)
    dy = torch.randn((rows, K), device="cuda", generator=torch.Generator(device="cuda").manual_seed(1)).to(torch.bfloat16)
    tr = L["tok_ad"] >= 0
    n_train = int(tr.sum())
    tile, slices, _ = binding.host_plain_gemm(n_train, cols, K, not kmajor, steps=2 * sum((r + 15) // 16 for r in ranks))
    assert tile == binding.TILE_256x256 and slices > 1
    dx = torch.full((rows, cols), float("nan"), dtype=torch.bfloat16, device="cuda")
    f32 = dict(dtype=torch.float32, device="cuda")
    tp = (lambda a, b: (b, a)) if kmajor else (lambda a, b: (a, b))
    dA = [torch.full(tp(cols, r), float("nan"), **f32) for r in ranks]
    dB = [torch.full(tp(r, K), float("nan"), **f32) for r in ranks]
    A, B = [L["st"](a) for a in L["A"]], [L["st"](b) for b in L["B"]]
    L["ctx"].collm_lora_linear_bwd(L["x"], L["st"](L["W"]), A, B, *L["batch"], dy, None, dx, dA, dB, layout=L["layout"])
    ref = dy.float() @ L["W"].float().T
    for a, r in enumerate(ranks):
        m = L["tok_ad"] == a
        dh = 0.7 * (dy[m].float() @ L["B"][a].float().T)
        ref[m] += dh @ L["A"][a].float().T
        dA_ref, dB_ref = L["x"][m].float().T @ dh, (0.7 * (L["x"][m].float() @ L["A"][a].float())).T @ dy[m].float()
        for got, want in ((dA[a], dA_ref), (dB[a], dB_ref)):
            got = got.T if kmajor else got
            assert (got - want).abs().max() <= TOL["bf16"] * want.abs().max()
    assert torch.isnan(dx[~tr]).all() and torch.isfinite(dx[tr]).all()
    assert (dx[tr].float() - ref[tr]).abs().max() <= TOL["bf16"] * ref[tr].abs().max()
    L["ctx"].close()
