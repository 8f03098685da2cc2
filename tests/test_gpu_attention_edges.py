"""Tree attention where its kernels change course: every workgroup shape from one key tile upwards (the pipelines' first and
last tiles, tiles that are partly prefix, partly tree or cut short), row counts that leave wavefronts idle, batches cut into
runs, and the merge of few and many key splits for few and many rows.  Bounds as in test_gpu_attention."""
import numpy as np
import pytest

import oracle
import paper_2512_23858_amd as ygg
import ygg_workloads as wl
from gpu_util import run_attention, shape_of
from test_gpu_attention import _cfg, _check, _inputs

pytestmark = pytest.mark.gpu


@pytest.fixture
def plan():
    yield ygg.set_attention_plan
    ygg.set_attention_plan()


# query heads on one kv head and a tree of 41 nodes: 246 rows, or 41 with one query head.  The 256-row shape, and at head_dim 128 that of
# 192 rows, run their wavefronts in opposite phases where the longest prefix leaves a workgroup many tiles, whatever the lengths then are.
@pytest.mark.parametrize("waves,kshares,Hq,longest", [(8, 1, 6, 0), (8, 1, 4, 0), (8, 1, 6, 8300), (8, 1, 4, 8300), (6, 1, 6, 0),
                                                      (6, 1, 6, 8300), (6, 1, 4, 8300),
                                                      (4, 1, 6, 0), (8, 2, 6, 0), (4, 2, 2, 0), (2, 2, 1, 0)])
@pytest.mark.parametrize("Dh", [128, 64])
@pytest.mark.parametrize("nsplit", [1, 2])
def test_every_workgroup_shape_from_one_tile_upwards(plan, waves, kshares, Hq, longest, Dh, nsplit):
    plan(waves=waves, rblocks=1, kshares=kshares, nsplit=nsplit)
    for keys in (41, 63, 64, 65, 100, 129, 192, 200, 257, 320, 330, 385, 450, 513, 640, 705, 1000):
        L = keys - 41
        cfg, host, parent = _inputs(_cfg(1, Hq, 1, 5, 8, Dh=Dh, seed=31), [L], max(L, longest, 1), tree_gain=2.0)
        shape = shape_of(cfg, max_seq_len=max(L, longest, 1))
        got = ygg.attention_plan(shape)
        assert (got["waves"], got["key_shares"]) == (waves, kshares)
        tiles = (keys + 63) // 64 // got["key_splits"]
        phases = longest > 0 or tiles >= (10 if Dh == 128 else 24)
        assert ygg.attention_launch(shape)["opposite_phases"] == (phases and kshares == 1 and (waves == 8 or (waves == 6 and Dh == 128)))
        _check(cfg, host, parent, max(L, longest, 1))


# two wavefronts fetch the rows of up to 32 in turns of four: 2, 3, 4, 5, 8, 9, 12, 13, 28, 31 and 32 rows to a kv head
@pytest.mark.parametrize("group,D,W", [(1, 1, 1), (1, 1, 2), (2, 1, 1), (1, 1, 4), (4, 1, 1), (3, 1, 2), (4, 1, 2), (1, 3, 4), (4, 2, 3), (1, 5, 6),
                                       (2, 3, 5)])
@pytest.mark.parametrize("nsplit", [1, 3])
def test_rows_of_two_wavefronts(plan, group, D, W, nsplit):
    plan(nsplit=nsplit)
    for L in (0, 50, 257):
        cfg, host, parent = _inputs(_cfg(2, 2 * group, 2, D, W, seed=33), [L, L // 2], max(L, 1), tree_gain=2.0)
        got = ygg.attention_plan(shape_of(cfg, max_seq_len=max(L, 1)))
        assert (got["waves"], got["key_shares"]) == (2, 2)
        _check(cfg, host, parent, max(L, 1))


@pytest.mark.parametrize("waves", [8, 6, 4])
def test_the_widest_tree_under_a_forced_shape(plan, waves):
    plan(waves=waves, rblocks=1, kshares=1)
    cfg, host, parent = _inputs(_cfg(1, 2, 2, 31, 33, seed=37), [100], 100, tree_gain=2.0)
    assert cfg.n_nodes == 1024
    _check(cfg, host, parent, 100)


# at least eight tiles to a workgroup of the longest sequence: the batch is cut into equal runs of tiles, as many as fill 256
# workgroups (the last case's workgroups are pairs, which runs do not serve: equal splits of each sequence)
@pytest.mark.parametrize("B,Hq,Hkv,D,W,lens,Dh,runs", [
    (5, 32, 4, 6, 8, [5000, 0, 64, 1500, 333], 128, 32),            # two row tiles, an empty and a one-tile prefix
    (9, 32, 8, 5, 7, [4000, 100, 15, 15, 2000, 1, 700, 64, 3999], 128, 32),
    (16, 24, 4, 5, 8, [64 * i * 4 % 4096 for i in range(16)], 64, 64),
    (16, 32, 4, 6, 8, [0] * 9 + [5000] + [3] * 6, 128, 32),         # many sequences of one tile: runs without a tile of their own
    (2, 32, 4, 6, 8, [9000, 0], 128, 32),                           # exactly eight tiles, an empty prefix at the end
    (6, 48, 8, 5, 8, [7500, 0, 64, 1500, 15, 333], 128, 32),        # runs of up to 22 tiles: opposite phases
    (6, 48, 8, 5, 8, [23000, 0, 64, 1500, 15, 333], 64, 32),        # up to 67: opposite phases at head_dim 64
    (2, 28, 4, 5, 8, [3000, 0], 128, 0),
])
def test_batches_in_runs(B, Hq, Hkv, D, W, lens, Dh, runs):
    cfg, host, parent = _inputs(_cfg(B, Hq, Hkv, D, W, Dh=Dh, seed=41), lens, max(lens), tree_gain=2.0)
    got = ygg.attention_plan(shape_of(cfg, max_seq_len=max(lens)))
    equal_splits = 256 // (B * Hkv * got["row_tiles"])
    assert got["key_splits"] == (runs or equal_splits) and equal_splits != runs
    assert ygg.attention_launch(shape_of(cfg, max_seq_len=max(lens)))["opposite_phases"] == (B == 6 or (B, Dh) == (16, 128))
    _check(cfg, host, parent, max(lens))


# equal lengths with a whole number of runs to a sequence (runs end where sequences do), from fewer tiles than runs upwards; one that differs
@pytest.mark.parametrize("lens", [[0] * 4, [15] * 4, [16] * 4, [300] * 4, [463] * 4, [464] * 4, [4300] * 4, [4300] * 3 + [4200], [9000] * 2])
@pytest.mark.parametrize("Dh", [128, 64])
def test_equal_lengths_in_runs(lens, Dh):
    B, longest = len(lens), max(4300, max(lens))
    cfg, host, parent = _inputs(_cfg(B, 32, 4, 6, 8, Dh=Dh, seed=43), lens, longest, tree_gain=2.0)
    assert ygg.attention_plan(shape_of(cfg, max_seq_len=longest))["key_splits"] == 32 and 32 % B == 0
    _check(cfg, host, parent, longest)


# merge: whole wavefronts per row up to 4096 rows, fewer lanes above; rounds of 8, 16 or 32 splits
@pytest.mark.parametrize("nsplit", [2, 7, 8, 9, 16, 17, 33, 64])
@pytest.mark.parametrize("Dh", [128, 64])
def test_merge_of_few_and_many_splits(plan, nsplit, Dh):
    plan(nsplit=nsplit)
    for Hq, Hkv, D, W in ((3, 3, 3, 5), (64, 4, 5, 13)):        # 48 and 4224 rows
        cfg, host, parent = _inputs(_cfg(1, Hq, Hkv, D, W, Dh=Dh, seed=53), [4200], 4200)
        assert ygg.attention_plan(shape_of(cfg, max_seq_len=4200))["key_splits"] == nsplit
        _check(cfg, host, parent, 4200)


# fp32 takes a split per key tile while its rows are few; no more than 4096 rows are ever split
@pytest.mark.parametrize("nsplit", [2, 7, 8, 9, 16, 17, 33, 64])
@pytest.mark.parametrize("Dh", [128, 64])
def test_merge_of_fp32_splits(nsplit, Dh):
    L = 64 * nsplit - 16
    cfg, host, parent = _inputs(_cfg(1, 3, 3, 3, 5, dtype="f32", Dh=Dh, seed=53), [L], L)
    assert cfg.n_nodes == 16 and ygg.attention_plan(shape_of(cfg, max_seq_len=L))["key_splits"] == nsplit
    _check(cfg, host, parent, L)


# where a workgroup's share of the keys is short the launch plan takes another shape than the one of fewest padded rows:
# (wavefronts, key shares) of these are (8, 1), (8, 1), (8, 1), (6, 1) and (8, 2)
@pytest.mark.parametrize("Hq,Hkv,D,W,L,shape", [(32, 8, 6, 8, 4096, (4, 2)), (32, 8, 6, 8, 500, (4, 2)), (64, 8, 6, 8, 4096, (8, 2)),
                                                (32, 8, 8, 16, 1024, (4, 2)), (32, 32, 10, 32, 4096, (6, 1))])
def test_short_runs_of_many_rows(Hq, Hkv, D, W, L, shape):
    cfg, host, parent = _inputs(_cfg(1, Hq, Hkv, D, W, seed=61), [L], L, tree_gain=2.0)
    got = ygg.attention_plan(shape_of(cfg, max_seq_len=L))
    assert (got["waves"], got["key_shares"]) == shape and got["key_splits"] > 1
    _check(cfg, host, parent, L)


@pytest.mark.parametrize("Dh", [128, 64])
def test_partial_sums_up_to_the_largest_floats(plan, Dh):
    """All scores are 0, so a split's partial output is the plain sum of its V rows: about 2^126.4, and the reciprocal of that is a
    subnormal float.  The two partials together stay below 2^128.  The result is the mean of the V rows; bound as in _check,
    in units of V."""
    plan(nsplit=2)
    cfg, host, parent = _inputs(_cfg(1, 8, 2, 6, 8, Dh=Dh, seed=71), [600], 600)
    host["q"] = np.zeros_like(host["q"])
    unit = 2.0 ** 118
    for stream, name in ((1, "v_cache"), (2, "v_tree")):
        v = unit * (1.0 + 0.4 * wl.rng(71, stream).random(host[name].shape))
        host[name] = wl.to_storage(v.astype(np.float32), cfg.dtype)
    shape = shape_of(cfg, max_seq_len=600)
    assert ygg.attention_plan(shape)["key_splits"] == 2
    ref, _ = oracle.tree_attention(host["q"], host["k_cache"], host["v_cache"], host["seq_lens"], host["k_tree"], host["v_tree"],
                                   parent, cfg.softmax_scale)
    out, _ = run_attention(shape, host, parent)
    assert np.isfinite(out).all()
    assert np.abs(out - ref).max() / unit <= 2e-2, np.abs(out - ref).max() / unit


def test_fp32_splits_keep_their_weights_at_large_scores():
    """Scores near 2^20, each exact in fp32 (one element of q and k is not zero; 1/8 is their spacing and the scale is 1/8), and
    V = 1 in the first half of the prefix, -1 in the second, so that every split's weight shows.  Differences of references are
    exact; an output is off by at most one unit in the last place for each of its three factors expf and for each addition of
    1149 keys, as is its sum of weights: 1152 * 2^-23 = 1.4e-4 at most."""
    cfg, host, parent = _inputs(_cfg(1, 4, 4, 6, 8, dtype="f32", Dh=64, seed=72), [1100], 1100)
    assert cfg.softmax_scale == 0.125
    for name in ("q", "k_cache", "k_tree"):
        host[name] = np.zeros_like(host[name])
    host["q"][..., 5] = 8.0
    for stream, name in ((1, "k_cache"), (2, "k_tree")):
        tile = (np.arange(host[name].shape[1]) // 64 * 53 % 25)[None, :, None]      # splits of different maxima
        host[name][..., 5] = 2.0 ** 20 + (tile + wl.rng(72, stream).integers(0, 9, host[name].shape[:-1])) / 8.0
    host["v_cache"][:, :550], host["v_cache"][:, 550:], host["v_tree"][:] = 1.0, -1.0, 0.5
    shape = shape_of(cfg, max_seq_len=1100)
    assert ygg.attention_plan(shape)["key_splits"] > 4
    ref, ref_lse = oracle.tree_attention(host["q"], host["k_cache"], host["v_cache"], host["seq_lens"], host["k_tree"],
                                         host["v_tree"], parent, cfg.softmax_scale)
    out, lse = run_attention(shape, host, parent)
    assert np.abs(out - ref).max() <= 1.4e-4, np.abs(out - ref).max()
    assert np.abs(lse - ref_lse).max() <= 2.0 ** -3, np.abs(lse - ref_lse).max()   # one unit in the last place at 2^20


@pytest.mark.parametrize("waves", [8, 4, 2])
@pytest.mark.parametrize("Dh", [128, 64])
@pytest.mark.parametrize("nsplit", [1, 2])
def test_pairs_whose_second_share_sees_little(plan, waves, Dh, nsplit):
    """At most 32 keys in a split's only tile: the second wavefront of a pair has no visible key, yet finishes its half of the row."""
    plan(waves=waves, rblocks=1, kshares=2, nsplit=nsplit)
    for L in (0, 23, 24, 64, 87):   # nine tree nodes: 9, 32, 33 keys; the same behind a whole tile
        cfg, host, parent = _inputs(_cfg(1, 3, 1, 4, 2, Dh=Dh, seed=47), [L], max(L, 1), tree_gain=4.0)
        _check(cfg, host, parent, max(L, 1))


@pytest.mark.parametrize("waves", [8, 4, 2])
@pytest.mark.parametrize("Dh", [128, 64])
def test_partial_rows_of_pairs_that_cancel(plan, waves, Dh):
    """All scores are 0 and V is whole numbers of 0 to 3, but for 1.75 * 2^23 at one key of a pair's first share and its negative at one of
    the second's: every sum is exact in fp32, and a split's partial row is at most 3 * 64 = 192 large.  Stored to 2^-12 of that, both
    splits' partials and the rounding to bf16 (8 significant bits: half a unit is 2^-8 of the value at most) put an output off by no more
    than 2 * 192 * 2^-12 / keys + 2^-8 of its value; a scale of the size of the shares' own sums would put it off by up to 2 * 0.875 / keys."""
    plan(waves=waves, rblocks=1, kshares=2, nsplit=2)
    cfg, host, parent = _inputs(_cfg(1, 3, 1, 4, 2, Dh=Dh, seed=73), [119], 119)       # nine tree nodes: two tiles of 64 keys
    host["q"] = np.zeros_like(host["q"])
    for stream, name in ((1, "v_cache"), (2, "v_tree")):
        v = wl.rng(73, stream).integers(0, 4, host[name].shape).astype(np.float32)
        if name == "v_cache":
            for at, sign in ((5, 1.0), (40, -1.0), (70, 1.0), (100, -1.0)):
                v[:, at] = sign * 1.75 * 2.0 ** 23
        host[name] = wl.to_storage(v, cfg.dtype)
    shape = shape_of(cfg, max_seq_len=119)
    got = ygg.attention_plan(shape)
    assert (got["waves"], got["key_shares"], got["key_splits"]) == (waves, 2, 2)
    ref, _ = oracle.tree_attention(host["q"], host["k_cache"], host["v_cache"], host["seq_lens"], host["k_tree"], host["v_tree"],
                                   parent, cfg.softmax_scale)
    out, _ = run_attention(shape, host, parent)
    bound = 2 * 192 * 2.0 ** -12 / 120 + 2.0 ** -8 * np.abs(ref)     # (120 to 123 keys to a row)
    assert (np.abs(out - ref) <= 1.001 * bound).all(), (np.abs(out - ref) / bound).max()


# The last split's share is smaller by what the tree's keys cost it, down to one tile, and the others' differ by one: trees of one, two
# and four tiles over prefixes that leave splits empty, leave them one tile, and (the longest, where the splits are few) give them
# enough for opposite phases.
@pytest.mark.parametrize("waves,Dh", [(8, 128), (6, 128), (4, 128), (8, 64), (6, 64)])
@pytest.mark.parametrize("D,W,nsplit", [(5, 8, 3), (6, 16, 5), (10, 20, 5), (10, 20, 16)])
def test_shares_of_the_last_split(plan, waves, Dh, D, W, nsplit):
    plan(waves=waves, rblocks=1, kshares=1, nsplit=nsplit)
    longest = 64 * (11 if Dh == 128 else 25) * nsplit if nsplit < 10 else 700
    for L in (0, 63, 200, 64 * nsplit - 1 - D * W % 64, 640, 1111, longest):
        cfg, host, parent = _inputs(_cfg(1, 4, 1, D, W, Dh=Dh, seed=47), [L], max(L, 64 * nsplit), tree_gain=2.0)
        _check(cfg, host, parent, max(L, 64 * nsplit))
    got = ygg.attention_launch(shape_of(cfg, max_seq_len=longest))
    assert got["opposite_phases"] == (nsplit < 10 and (waves == 8 or (waves == 6 and Dh == 128)))
    tiles = (1 + D * W + 63) // 64
    assert got["tree_cost"] == (1 + 6 * tiles // 5 if got["opposite_phases"] else 1 + tiles // 4)


# Pairs of head_dim 64: the last split gives a tile away where the tree's keys then still lie in it alone.  Prefixes around that, with one
# to three tiles of tree.
@pytest.mark.parametrize("waves", [8, 4, 2])
@pytest.mark.parametrize("D,W,nsplit", [(2, 4, 3), (5, 8, 4), (10, 13, 3), (10, 13, 10)])
def test_tiles_given_away_by_pairs(plan, waves, D, W, nsplit):
    plan(waves=waves, rblocks=1, kshares=2, nsplit=nsplit)
    tree = 1 + D * W
    for tiles in (2 * nsplit, 2 * nsplit + 1, 3 * nsplit - 2, 3 * nsplit - 1):
        for keys in (64 * tiles, 64 * tiles - 1, 64 * tiles - 63):
            L = keys - tree
            cfg, host, parent = _inputs(_cfg(1, 2, 1, D, W, Dh=64, seed=67), [L], L, tree_gain=2.0)
            assert ygg.attention_plan(shape_of(cfg, max_seq_len=L))["key_splits"] == nsplit
            _check(cfg, host, parent, L)
