"""CPU-side checks of the C-ABI library: it loads, exports what the header declares, and its
host-only integer bookkeeping equals the oracle's bit for bit."""
import ctypes
import os
import re
import sys

import numpy as np
import pytest

import oracle
from paper_2604_16400_amd import binding
from paper_2604_16400_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    lib = binding.load_library()
    hdr = open(os.path.join(ROOT, "include", "collm_lora.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    names = re.findall(r"\b(collm_[a-z_0-9]+)\s*\(", hdr)
    assert len(set(names)) >= 11
    for n in set(names):
        assert hasattr(lib, n), n
    assert lib.collm_status_string(0) == b"ok"
    assert lib.collm_status_string(-3) != lib.collm_status_string(-4)


def test_token_map_matches_oracle_bit_for_bit_fuzz():
    rng = np.random.default_rng(20260416)
    for it in range(10000):
        S = int(rng.integers(0, 40))
        kind = it % 4
        if kind == 0:
            lens = rng.integers(0, 4, size=S)
        elif kind == 1:
            lens = rng.integers(1, 300, size=S)
        elif kind == 2:
            lens = (rng.random(S) < 0.3) * rng.integers(0, 2000, size=S)
        else:
            lens = np.ones(S, dtype=np.int64)
        seg_start = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        tr = rng.integers(0, 2, size=S).astype(np.uint8)
        ad = rng.integers(-1, 7, size=S).astype(np.int32)
        ad[(tr != 0) & (ad < 0)] = 0
        got = binding.collm_token_map(seg_start, ad, tr, n_adapters=7)
        ref = oracle.token_map(seg_start, ad, tr)
        for g, r in zip(got, ref):
            assert g.dtype == r.dtype and np.array_equal(g, r)


@pytest.mark.parametrize("cfg", [1, 2, 3, 4, 5])
def test_token_map_configs(cfg):
    w = wl.make_config(cfg)
    got = binding.collm_token_map(w.seg_start, w.seg_adapter, w.seg_is_train, n_adapters=w.n_adapters)
    ref = oracle.token_map(w.seg_start, w.seg_adapter, w.seg_is_train)
    for g, r in zip(got, ref):
        assert np.array_equal(g, r)
    assert int(np.count_nonzero(got[2])) == w.n_train_tokens


def test_token_map_rejects_bad_tables():
    f = binding.collm_token_map
    with pytest.raises(binding.CollmError) as e:
        f([1, 3], [0], [0])  # does not start at 0
    assert e.value.status == -3
    with pytest.raises(binding.CollmError) as e:
        f([0, 3, 2], [0, 0], [0, 0])  # decreasing
    assert e.value.status == -3
    with pytest.raises(binding.CollmError) as e:
        f([0, 3], [0], [0], n_tokens=4)  # does not end at T
    assert e.value.status == -3
    with pytest.raises(binding.CollmError) as e:
        f([0, 3], [5], [0], n_adapters=5)  # adapter out of range
    assert e.value.status == -4
    with pytest.raises(binding.CollmError) as e:
        f([0, 3], [-1], [1], n_adapters=5)  # training segment without adapter
    assert e.value.status == -4
    with pytest.raises(binding.CollmError) as e:
        f([0, 3], [-2], [0], n_adapters=5)
    assert e.value.status == -4


# ---------------------------------------------------------------------------------------------
# the plan's row order (host logic): rows in runs of one adapter, low-rank K-steps per row tile
# ---------------------------------------------------------------------------------------------
def _steps_from_rows(row_tok, tok_adapter, ranks, tile_rows):
    """K-steps per row tile, counted from the row order: every maximal run of one adapter inside a
    tile costs ceil(rank / 16) steps; the steps are listed by groups of 64 rank indices, and every group
    but the tile's last is filled up to a multiple of four steps."""
    out = []
    for t0 in range(0, len(row_tok), tile_rows):
        ads = tok_adapter[row_tok[t0:t0 + tile_rows]]
        run_ranks = [int(ranks[a]) for i, a in enumerate(ads) if a >= 0 and (i == 0 or ads[i - 1] != a)]
        n, g = 0, 0
        while True:
            n += sum((min(r, g + 64) - g + 15) // 16 for r in run_ranks if r > g)
            g += 64
            if not any(r > g for r in run_ranks):
                break
            n = (n + 3) // 4 * 4
        out.append(n)
    return np.array(out, dtype=np.int32)


@pytest.mark.parametrize("cfg", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("tile_rows", [128, 256])
def test_plan_row_order_is_a_grouping_and_counts_its_steps(cfg, tile_rows):
    w = wl.make_config(cfg)
    _, ta, tt = oracle.token_map(w.seg_start, w.seg_adapter, w.seg_is_train)
    row_tok, steps = binding.host_row_order(w.ranks, w.seg_start, w.seg_adapter, w.seg_is_train, tile_rows)
    assert sorted(row_tok.tolist()) == list(range(w.n_tokens))           # every token exactly once
    ads = ta[row_tok]
    n_base = int((ta < 0).sum())
    assert np.all(ads[:n_base] < 0) and np.all(ads[n_base:] >= 0)        # base-only rows first
    for a in range(w.n_adapters):                                         # token order kept inside an adapter
        toks = row_tok[ads == a]
        assert np.all(np.diff(toks) > 0)
    assert np.array_equal(steps, _steps_from_rows(row_tok, ta, w.ranks, tile_rows))
    # training rows: one run per adapter (the gradient items are runs)
    row_tr, steps_tr = binding.host_row_order(w.ranks, w.seg_start, w.seg_adapter, w.seg_is_train, tile_rows, True)
    assert sorted(row_tr.tolist()) == np.flatnonzero(tt).tolist()
    ads_tr = ta[row_tr]
    changes = int((np.diff(ads_tr) != 0).sum()) + 1 if len(ads_tr) else 0
    assert changes == len(np.unique(ads_tr))
    assert np.array_equal(steps_tr, _steps_from_rows(row_tr, ta, w.ranks, tile_rows))


def test_plan_spreads_rare_adapters_over_the_row_tiles():
    # configuration 3: 32 adapters of rank 64 with Zipf popularity.  Listed by adapter index, the rare ones
    # would share the last tiles (11 adapters = 44 steps in one of them); dealt out, no tile carries more than
    # a few adapters beside the large ones that fill it.
    w = wl.make_config(3)
    _, ta, _ = oracle.token_map(w.seg_start, w.seg_adapter, w.seg_is_train)
    _, steps = binding.host_row_order(w.ranks, w.seg_start, w.seg_adapter, w.seg_is_train, 256)
    by_index = _steps_from_rows(np.argsort(ta, kind="stable").astype(np.int32), ta, w.ranks, 256)
    assert by_index.max() >= 40
    assert steps.max() <= 20 and steps.max() <= by_index.max() // 2
    assert steps.sum() <= by_index.sum() + 4 * len(steps)   # at most one more run per tile, of rank 64


def test_gemm_tiling_covers_the_rows_and_matches_the_measured_choices():
    rng = np.random.default_rng(5)
    for _ in range(2000):
        rows = int(rng.integers(1, 40000))
        cols = int(rng.integers(1, 4000)) * 8
        K = int(rng.integers(1, 2000)) * 8
        tile, big, tail, tail_cols = binding.host_tiling(rows, cols, K, bool(rng.integers(0, 2)))
        assert tile in (binding.TILE_256x256, binding.TILE_128x128) and big >= 1 and tail >= 0 and tail_cols >= 0
        tr = 256 if tile == binding.TILE_256x256 else 128
        assert tr * big + 128 * tail >= rows                      # every row is in some tile
        if tail:
            assert tile == binding.TILE_256x256 and 256 * big < rows          # the tail starts inside the rows
            assert 256 * big + 128 * (tail - 1) < rows                        # and has no empty row tile
        else:
            assert tr * (big - 1) < rows or rows <= tr
        if tail_cols:
            # large tiles over whole rounds of the 256 CUs, then at most one round of small tiles (two per CU)
            tn = (cols + 255) // 256
            assert tile == binding.TILE_256x256 and tail == 0 and 0 < tail_cols < tn
            assert big * (tn - tail_cols) <= 256 * (big * tn // 256)
            assert ((rows + 127) // 128) * ((cols - 256 * (tn - tail_cols) + 127) // 128) <= 512
    # choices the measurements on the five configurations gave
    assert binding.host_tiling(2048, 4096, 4096) == (binding.TILE_128x128, 16, 0, 0)    # c2 forward: one round of 512 small tiles
    assert binding.host_tiling(16384, 8192, 8192) == (binding.TILE_256x256, 64, 0, 0)   # c5: whole rounds of large tiles
    assert binding.host_tiling(3277, 5120, 5120) == (binding.TILE_256x256, 12, 2, 0)    # c4 dX: 240 large tiles + the last 205 rows
    assert binding.host_tiling(8192, 5120, 5120) == (binding.TILE_256x256, 32, 0, 4)    # c4 forward: 2 rounds + 512 tiles of 128x128
    assert binding.host_tiling(4096, 11008, 4096) == (binding.TILE_256x256, 16, 0, 0)   # c3 forward: 2.7 rounds, no split pays
    assert binding.host_tiling(64, 4096, 4096)[0] == binding.TILE_128x128               # decode-sized


def _sanitizer_run(tmp_path, compiler, std, sources, args):
    """Builds the sources with the address and undefined-behaviour sanitizers (static runtimes, so that nothing
    preloaded into this process matters) and runs the result."""
    import subprocess

    exe = str(tmp_path / "sanitized")
    cmd = [compiler, std, "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-static-libasan",
           "-static-libubsan", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2604_16400_amd", "csrc"),
           *sources, "-lm", "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0", LD_PRELOAD="")
    r = subprocess.run([exe, *args], capture_output=True, text=True, env=env, timeout=240)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return r.stdout


def test_planner_under_address_and_undefined_behaviour_sanitizers(tmp_path):
    # 10^4 random segment tables through build_plan with every option (tile sizes, item sizes, the tiled pass,
    # sibling ranks), each plan checked against what the table fixes: csrc/planner.cpp is offset arithmetic into
    # one int32 block
    out = _sanitizer_run(tmp_path, "g++", "-std=c++17",
                         [os.path.join(ROOT, "tests", "sanitize_planner.cpp"),
                          os.path.join(ROOT, "paper_2604_16400_amd", "csrc", "planner.cpp")], ["10000"])
    assert "planner ok 10000" in out


def test_oracle_under_address_and_undefined_behaviour_sanitizers(tmp_path):
    out = _sanitizer_run(tmp_path, "gcc", "-std=c11",
                         [os.path.join(ROOT, "tests", "sanitize_oracle.c"), os.path.join(ROOT, "oracle", "collm_oracle.c")],
                         ["300"])
    assert "oracle ok 300" in out


def test_gemm_tile_order_visits_every_tile_once_and_keeps_bands_together():
    # The workgroup id -> tile map of the GEMM kernels, run on the host: a bijection for every grid and band, a band's
    # tiles contiguous in workgroup ids, and the walk of every XCD through a band.
    rng = np.random.default_rng(5)
    shapes = [(64, 112, 32), (64, 32, 32), (64, 4, 0), (13, 20, 0), (13, 20, 8), (40, 7, 16), (33, 5, 24), (1, 1, 0), (7, 3, 8)]
    shapes += [(int(rng.integers(1, 70)), int(rng.integers(1, 40)), int(rng.integers(0, 5)) * 8) for _ in range(60)]
    for tiles_m, tiles_n, band in shapes:
        used, tm, tn = binding.host_tile_order(256, tiles_m, tiles_n, 8192, band)
        assert used == band
        seen = np.zeros((tiles_m, tiles_n), dtype=np.int32)
        np.add.at(seen, (tm, tn), 1)
        assert (seen == 1).all(), (tiles_m, tiles_n, band)
        if 0 < band < tiles_m:
            ids = np.arange(tiles_m * tiles_n)
            assert np.array_equal(tm // band, ids // (band * tiles_n)), (tiles_m, tiles_n, band)
        # an XCD (workgroup ids 8 i + x) walks the groups of 8 row tiles of a band in ascending order, and inside a
        # group column by column
        b = band if 0 < band < tiles_m else tiles_m
        for x in range(8):
            m, n = tm[x::8].astype(np.int64), tn[x::8].astype(np.int64)
            key = ((m // b) * (tiles_m + 8) + (m % b) // 8) * tiles_n + n
            assert (np.diff(key) >= 0).all(), (tiles_m, tiles_n, band, x)
    # the band the library chooses: the rows of configuration 5 (16384 x 8192) in bands of 32 row tiles; none where all
    # rows fit the cache anyway (few row tiles) or where not even 16 row tiles do (K = 28672)
    assert binding.host_tile_order(256, 64, 112, 8192)[0] == 32
    assert binding.host_tile_order(256, 64, 32, 8192)[0] == 32
    assert binding.host_tile_order(256, 32, 54, 5120)[0] == 0
    assert binding.host_tile_order(256, 32, 32, 28672)[0] == 0
    assert binding.host_tile_order(128, 16, 32, 4096)[0] == 0



@pytest.mark.parametrize("tiles_m,tiles_n,n_slices", [(2, 30, 4), (1, 212, 2), (3, 11, 8), (1, 1, 3), (5, 13, 1), (40, 11, 1)])
def test_gradients_in_the_gemm_s_launch_start_behind_all_of_its_slices(tiles_m, tiles_n, n_slices):
    tiles, grads = tiles_m * tiles_n, 19
    sl, tm, tn, gr = (a.astype(np.int64) for a in binding.host_shared_order(tiles_m, tiles_n, n_slices, 4096, grads))
    gemm = tiles * n_slices
    first = (gemm + 7) // 8 * 8
    assert (gr[:first] == -1).all() and (gr[first:] == np.arange(grads)).all() and (sl[gemm:] == -1).all()
    assert sorted((sl * tiles + tm * tiles_n + tn)[:gemm]) == list(range(gemm))  # every tile of every slice once
    if n_slices == 1:
        _, m, n = binding.host_tile_order(128, tiles_m, tiles_n, 4096)
        assert (m == tm[:gemm]).all() and (n == tn[:gemm]).all()
        return
    # an XCD (the id's last three bits) has one run of the tiles of one slice after the other
    run = [sl[x:gemm:8] * tiles + (tm[x:gemm:8] // 8) * 8 * tiles_n + tn[x:gemm:8] * np.minimum(8, tiles_m - tm[x:gemm:8] // 8 * 8) + tm[x:gemm:8] % 8
           for x in range(8)]
    assert (np.concatenate(run) == np.arange(gemm)).all()


def test_marshalling_takes_the_plain_forms_and_leaves_the_rest():
    """The compiled marshalling calls the library for contiguous int32 / uint8 arrays and pointer tables (here it reports
    the missing context) and hands everything else back to the binding's general path."""
    import torch

    binding.load_library()
    m = binding._marshal
    x, W = torch.zeros(3, 8, dtype=torch.bfloat16), torch.zeros(8, 16, dtype=torch.bfloat16)
    tab = binding.PointerTable([torch.zeros(8), None])
    rank, ss = np.array([8, 4], np.int32), np.array([0, 1, 3], np.int32)
    sa, st = np.array([0, -1], np.int32), np.array([1, 0], np.uint8)
    good = [None, x, W, tab, tab, rank, ss, sa, st, 2.0, 0, 0, W, None]
    assert m.linear_fwd(*good) == -1                                   # COLLM_E_NULL: no context
    back = good[:13] + [None, None, tab, tab, 0]
    assert m.linear_bwd(*back) == -1 and m.linear_bwd(*(back[:15] + [None, None, 1])) == -1
    for at, other in [(3, [torch.zeros(8), None]), (4, None), (5, [8, 4]), (5, rank.astype(np.int64)), (5, np.array([8, 1, 4, 1], np.int32)[::2]),
                      (6, ss.astype(">i4")), (6, ss[:2]), (7, sa.reshape(1, 2)), (8, st.astype(bool)), (8, st[:1]), (9, "2"), (10, 1 << 40),
                      (1, x.half()), (1, x[0]), (2, None), (12, None), (13, 5)]:
        args = list(good)
        args[at] = other
        assert m.linear_fwd(*args) is None, (at, other)
    with pytest.raises(TypeError):
        m.linear_fwd(*good[:-1])
    e = torch.zeros(0)
    assert m.adapter_adamw(e, e, e, e, 1e-4, 0.9, 0.999, 1e-8, 0.0, 1, None, 0) == 0     # nothing to do
    assert m.adapter_adamw(e, e, e, e, 1e-4, 0.9, 0.999, 1e-8, 0.0, 0, None, 0) == -2    # COLLM_E_SHAPE: steps count from 1
    assert m.adapter_adamw(e, e, e, e, 1e-4, 0.9, 0.999, 1e-8, 0.0, 1.5, None, 0) is None
    assert m.adapter_adamw(e.half(), e, e, e, 1e-4, 0.9, 0.999, 1e-8, 0.0, 1, None, 0) is None
    copies = binding.PointerTable([x, x])
    assert m.adapter_fedavg(copies, 0, x, 0) == -2 and m.adapter_fedavg([x, x], 2, x, 0) is None


@pytest.mark.parametrize("rows,cols,K,tile", [
    (512, 8448, 4096, binding.TILE_128x128),     # 264 small tiles: one round of them, not 66 large ones on 256 CUs
    (1024, 4224, 4096, binding.TILE_128x128),
    (2048, 4096, 4096, binding.TILE_128x128),    # 512: exactly one round
    (3000, 3000, 3000, binding.TILE_256x256),    # 576 would start a second round
    (4096, 4096, 4096, binding.TILE_256x256),
])
def test_tile_choice_below_one_round(rows, cols, K, tile):
    assert binding.host_tiling(rows, cols, K)[0] == tile


@pytest.mark.parametrize("rows,cols,K,want", [
    (5427, 3920, 5192, (0, 16, 11, 0)), (1107, 16952, 17488, (0, 3, 3, 0)),  # more than two rounds of small tiles
    (5427, 3920, 1023, (2, 43, 0, 0)),                                       # too short for K slices
    (1498, 10880, 6040, (2, 12, 0, 0)), (636, 24704, 6808, (2, 5, 0, 0))])   # 1020 and 965 small tiles: at most two rounds
def test_small_tiles_behind_large_ones_beat_a_third_round(rows, cols, K, want):
    assert binding.host_tiling(rows, cols, K) == want


@pytest.mark.parametrize("tiles_m,tiles_n,K,want", [
    (1, 4, 512, 1), (8, 16, 768, 1), (1, 4, 1016, 1), (1, 8, 1024, 3), (8, 4, 1024, 3),                      # from K = 1024 on
    (8, 8, 1400, 1), (8, 8, 1408, 4), (8, 12, 1408, 2), (3, 11, 1400, 1), (1, 33, 1024, 3),                 # 1408 with several row tiles
    (1, 16, 3072, 10), (1, 32, 2048, 7), (1, 64, 2048, 4), (1, 64, 4096, 5), (2, 100, 4096, 2), (16, 16, 8192, 2),
    (1, 64, 6144, 8), (1, 64, 8192, 7), (1, 32, 8192, 11), (1, 32, 16384, 15), (1, 64, 16384, 7), (1, 64, 28672, 8), (8, 16, 8192, 4),
    (1, 257, 16376, 1), (1, 257, 16384, 3), (11, 31, 16384, 3), (11, 31, 16376, 1), (18, 19, 16384, 1),     # 257, 341, 342 tiles
    (4, 66, 11264, 3), (4, 66, 11256, 1), (2, 129, 11264, 1), (3, 96, 11264, 1), (8, 43, 11264, 2), (8, 43, 11256, 1),
    (8, 45, 28672, 2), (19, 19, 28672, 1), (6, 64, 28672, 1), (3, 115, 28672, 1), (5, 77, 28672, 1), (16, 32, 28672, 1)])
def test_gemm_slices_at_the_lines_of_the_rule(tiles_m, tiles_n, K, want):
    assert binding.host_gemm_slices(tiles_m, tiles_n * 128, K) == want
    assert binding.host_gemm_slices(tiles_m, tiles_n * 128 - 120, K, True) == want  # (the same tiles, the last one ragged)


@pytest.mark.parametrize("tiles_m,tiles_n,K,steps,want", [
    (1, 32, 512, 0, 1), (1, 32, 512, 15, 1), (1, 32, 512, 16, 3), (1, 32, 512, 96, 8), (2, 32, 512, 56, 4), (2, 32, 512, 55, 1),
    (1, 32, 256, 96, 4), (1, 16, 2048, 96, 16), (1, 64, 2048, 96, 7), (1, 300, 512, 96, 1)])
def test_gemm_slices_count_the_extension_steps(tiles_m, tiles_n, K, steps, want):
    # a decode batch of many adapters has more steps in its row tile than K tiles; slices of 64 K values at least
    assert binding.host_gemm_slices(tiles_m, tiles_n * 128, K, steps=steps) == want


@pytest.mark.parametrize("rows,cols,K,steps,want", [
    (1003, 5120, 5120, 0, (binding.TILE_128x192, 1, 0)),                   # 320 small tiles -> 216 blocks
    (1003, 5120, 5120, 168, (binding.TILE_128x128, 1, 0)),                 # ... not with 21 steps a row tile
    (1792, 4096, 4096, 0, (binding.TILE_256x128, 1, 0)),                   # 448 -> 224
    (2048, 4096, 4096, 0, (binding.TILE_256x128, 1, 0)),                   # 512 -> 256
    (2049, 4096, 4096, 0, (binding.TILE_256x192, 1, 0)),                   # 544 -> 198
    (901, 11008, 4104, 0, (binding.TILE_256x192, 1, 0)),                   # 688 -> 232
    (16384, 1024, 8192, 0, (binding.TILE_256x256, 1, 0)), (4096, 4096, 4096, 0, (binding.TILE_256x256, 1, 0)),
    (733, 5408, 16384, 0, (binding.TILE_128x128, 3, 0)), (733, 5408, 16376, 0, (binding.TILE_128x192, 1, 0)),  # 258 tiles: three slices
    (256, 16384, 1024, 0, (binding.TILE_128x128, 1, 1)), (256, 16512, 1024, 0, (binding.TILE_128x192, 1, 0)),  # 256 and 258 tiles
    (8, 4096, 4096, 0, (binding.TILE_128x128, 8, 1)), (8, 4096, 1536, 0, (binding.TILE_128x128, 8, 1)), (8, 4096, 1024, 0, (binding.TILE_128x128, 5, 1)),
    (8, 4096, 1016, 0, (binding.TILE_128x128, 1, 1)),                      # one block per CU, not cut
    (64, 11008, 4096, 64, (binding.TILE_128x128, 5, 0)),                   # 86 tiles: five slices on two blocks per CU
    (64, 4096, 4096, 64, (binding.TILE_128x128, 8, 1)), (64, 4096, 4096, 65, (binding.TILE_128x128, 8, 0)),     # the steps outweigh K
    (714, 1536, 26112, 0, (binding.TILE_128x128, 7, 0)), (714, 1536, 4096, 0, (binding.TILE_128x128, 3, 1)),  # long contractions
    (64, 10880, 4096, 0, (binding.TILE_128x128, 3, 1)), (64, 11008, 4096, 0, (binding.TILE_128x128, 5, 0)),     # 85 and 86 tiles,
    (64, 11008, 3072, 0, (binding.TILE_128x128, 2, 1)), (64, 16384, 4096, 0, (binding.TILE_128x128, 2, 1)),     # 86 and 128 tiles: two
    (512, 4096, 4096, 0, (binding.TILE_128x128, 2, 1)), (64, 16512, 4096, 0, (binding.TILE_128x128, 3, 0)),     # slices; 129 tiles
    (64, 16384, 10240, 0, (binding.TILE_128x128, 4, 0))])
def test_plain_gemm_choice_at_the_lines_of_the_rule(rows, cols, K, steps, want):
    assert binding.host_plain_gemm(rows, cols, K, steps=steps) == want


def test_gemm_slices_by_layout_and_workspace():
    for K, in_out, out_in in [(20472, 1, 1), (20480, 2, 1), (28672, 2, 1)]:
        assert (binding.host_gemm_slices(4, 86 * 128, K), binding.host_gemm_slices(4, 86 * 128, K, True)) == (in_out, out_in)
    # 341 tiles in three slices just fit 64 MiB; a workspace for two of the three leaves the contraction whole, one for
    # four of seven slices leaves four
    assert binding.host_gemm_slices(11, 31 * 128, 16384, workspace_bytes=3 * 341 * 65536) == 3
    assert binding.host_gemm_slices(11, 31 * 128, 16384, workspace_bytes=3 * 341 * 65536 - 1) == 1
    assert binding.host_gemm_slices(1, 64 * 128, 8192, workspace_bytes=4 * 64 * 65536) == 4
    assert binding.host_gemm_slices(1, 64 * 128, 8192, workspace_bytes=0) == 1


@pytest.mark.parametrize("rank", [1, 16, 17, 32, 48, 64, 65, 256])
def test_gradient_blocks_leave_room_for_two_gemm_blocks(rank):
    """A CU's LDS, first fit: gradient blocks, GEMM blocks of 128x128 tiles in what they leave, then the gradient blocks end.
    Two GEMM blocks must fit however many gradient blocks there were."""
    cu, gemm = 160 << 10, 64 << 10

    def place(held, size):
        at = 0
        for lo, hi in sorted(held):
            if lo - at >= size:
                break
            at = max(at, hi)
        return (at, at + size) if at + size <= cu else None

    grad = binding.host_grad_lds(rank, True)
    assert grad >= binding.host_grad_lds(rank, False)
    for n in range(1, cu // grad + 1):
        grads, gemms = [(k * grad, (k + 1) * grad) for k in range(n)], []
        for held in (grads, []):
            while (b := place(held + gemms, gemm)) is not None:
                gemms.append(b)
        assert len(gemms) == 2, (n, grad, gemms)


_BINDING_COPY = """
import importlib.util, os, sys, types
import torch

def load(path, name):
    spec = importlib.util.spec_from_file_location(name, os.path.join(path, "__init__.py"), submodule_search_locations=[path])
    sys.modules[name] = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(sys.modules[name])
    b = importlib.import_module(name + ".binding")
    b.load_library()
    return b

# a tensor on a device that does not exist: the library reports it and launches nothing
class T:
    dtype, device = torch.float32, types.SimpleNamespace(index=9999)
    def data_ptr(self): return 4096
    def numel(self): return 8

stream = types.SimpleNamespace(cuda_stream=0)
def adamw(b):
    try:
        b.collm_adapter_adamw(T(), T(), T(), T(), 1e-4, 0.9, 0.999, 1e-8, 0.0, 1, stream=stream)
    except b.CollmError as e:
        return str(e)
"""


def _run_binding_copy(tmp_path, keep_marshal, code, **env):
    import shutil
    import subprocess

    src = os.path.dirname(binding.LIB_PATH)
    copy = tmp_path / "copy"
    copy.mkdir()
    for f in ("__init__.py", "binding.py", "build.py", os.path.basename(binding.LIB_PATH)) + \
            ((os.path.basename(binding.MARSHAL_PATH),) if keep_marshal else ()):
        shutil.copy2(os.path.join(src, f), copy / f)
    shutil.copytree(os.path.join(src, "csrc"), copy / "csrc")
    r = subprocess.run([sys.executable, "-W", "ignore", "-c", _BINDING_COPY + code, src, str(copy)], capture_output=True, text=True,
                       env={**os.environ, **env}, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def test_the_binding_works_without_its_compiled_marshalling(tmp_path):
    """A library without the extension and without a compiler to build it: every call takes the ctypes route."""
    out = _run_binding_copy(tmp_path, False, """
b = load(sys.argv[2], "alone")
assert b._marshal is None
e = torch.zeros(0)
b.collm_adapter_adamw(e, e, e, e, 1e-4, 0.9, 0.999, 1e-8, 0.0, 1, stream=stream)
print(adamw(b))
""", CXX="/nonexistent/c++")
    assert "collm_adapter_adamw: status" in out, out


def test_the_extension_is_named_after_its_interpreter():
    import sysconfig

    assert binding.MARSHAL_PATH.endswith(sysconfig.get_config_var("EXT_SUFFIX")) and os.path.exists(binding.MARSHAL_PATH)


def test_each_binding_calls_its_own_library(tmp_path):
    """Two copies of the package in one process: the compiled marshalling of each calls the library its binding has loaded (the
    text of the last error is kept per library)."""
    out = _run_binding_copy(tmp_path, True, """
first, second = load(sys.argv[1], "first"), load(sys.argv[2], "second")
assert first._marshal is not None and second._marshal is not None and first.LIB_PATH != second.LIB_PATH
assert adamw(second) and second._lib.collm_last_error() and not first._lib.collm_last_error(), "called the other library"
assert adamw(first) and first._lib.collm_last_error()
print("ok")
""")
    assert out.strip().endswith("ok"), out


@pytest.mark.parametrize("n_train,d_in,d_out,dtype,rank,streams", [
    (768, 2048, 2048, binding.COLLM_BF16, 16, 2), (384, 1024, 4096, binding.COLLM_BF16, 16, 1),     # 6 and 3.75 MiB
    (768, 1024, 1024, binding.COLLM_BF16, 32, 2), (192, 1024, 4096, binding.COLLM_BF16, 32, 1),     # 3 and 1.9 MiB
    (1280, 1024, 1024, binding.COLLM_BF16, 16, 1), (1281, 1024, 1024, binding.COLLM_BF16, 16, 2),   # at and above 5 MiB
    (512, 1024, 1024, binding.COLLM_BF16, 17, 1), (513, 1024, 1024, binding.COLLM_BF16, 32, 2),     # at and above 2 MiB
    (1, 256, 256, binding.COLLM_BF16, 33, 2),
    (1024, 1024, 1024, binding.COLLM_F32, 256, 1), (1025, 1024, 1024, binding.COLLM_F32, 4, 2)])    # at and above 8 MiB
def test_streams_of_the_backward_call(n_train, d_in, d_out, dtype, rank, streams):
    assert binding.host_grad_streams(n_train, d_in, d_out, dtype, rank) == streams
