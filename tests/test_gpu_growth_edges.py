"""Both growth rules where their kernels change shape: chunk lengths of 1024 / 2048 / 4096 / several passes, tails of a few
logits, rows that are no multiple of four logits, fewer lists than new nodes, more equal logits than a candidate pool holds,
and logits whose exponentials need a reference other than zero.  Indices bit for bit against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_23858_amd as ygg
import ygg_workloads as wl
from gpu_util import DEV, shape_of, to_dev, workspace
from test_gpu_attach import attach_both, read_pool
from test_gpu_expand_accept import _expand_both

pytestmark = pytest.mark.gpu


def _cfg(B, D, W, V, seed=23):
    return wl.Config("case", B, 4, 2, 64, "bf16", 16, (), D, W, V, (0.6,), "dirichlet", 0.5, 1, seed)


@pytest.mark.parametrize("B,D,W,V", [(1, 2, 8, 1023), (1, 2, 8, 1024), (1, 3, 8, 1025), (1, 2, 9, 4099), (2, 2, 33, 2048),
                                     (1, 2, 64, 2050), (1, 3, 12, 3001),
                                     # second step in chunks of 1024 (512 lists), of 2048 (288 to 768) and of 4096 (416)
                                     (2, 2, 16, 16384), (2, 2, 16, 16388), (2, 2, 16, 16389), (2, 2, 16, 49152), (2, 2, 16, 49156),
                                     (1, 2, 3, 70000), (12, 2, 16, 5001), (40, 2, 3, 9001),      # chunks of 2048
                                     (40, 2, 8, 5000), (40, 2, 8, 5002),                         # chunks of 4096
                                     # few lists in a row for many new nodes: half or less of them, 17 to 31 lists, hardly any
                                     (1, 2, 60, 14000), (2, 2, 47, 50257), (1, 2, 64, 20000), (1, 2, 50, 24001), (1, 2, 62, 1000),
                                     (1, 2, 58, 70001), (1, 2, 33, 131080)])                     # several passes per chunk
def test_growth_at_the_edges_of_the_chunks(B, D, W, V):
    _expand_both(_cfg(B, D, W, V))
    if W * W + W * D <= 4096:
        attach_both(_cfg(B, D, W, V))


@pytest.mark.parametrize("V", [700, 5000, 70000])
@pytest.mark.parametrize("W", [3, 20])
def test_growth_with_more_ties_than_a_pool_holds(W, V):
    cfg = _cfg(1, 3, W, V)

    def equal(d):
        return np.full((1, 1 if d == 1 else W, V), 1.5, np.float32)
    _expand_both(cfg, logits_fn=equal, check_margin=False)
    attach_both(cfg, logits_fn=equal, check_margin=False)


@pytest.mark.parametrize("shift,masked", [(0.0, -1e9), (650.0, None), (-650.0, None), (0.0, -600.0), (3e4, -3e4)])
def test_growth_with_logits_far_from_zero(shift, masked):
    """Large offsets, and all but a stretch of the vocabulary pushed far down: whole chunks then carry a reference of their
    own beside chunks that need none.  The second row is left as it is."""
    cfg = _cfg(2, 3, 6, 9000, seed=29)

    def fn(d):
        x = wl.expansion_inputs(cfg, d)
        y = x[:, :1] if d == 1 else x[:, ::2]
        y += np.float32(shift)
        if masked is not None:
            y[:, :, :4200] = np.float32(masked) + x[:, :1, :4200]
            y[:, :, 4500:] = np.float32(masked) + x[:, :1, 4500:]
        return x
    _expand_both(cfg, logits_fn=fn, check_margin=False)


# forced tokens and rows without any: one logit of size `big` in each row of the first sequence, in the first, a middle or the last place;
# nothing but -big in the second's (the last chunk partly past the end); both by turns in the third's.  Chunks of 1024, 2048, 4096 and
# several passes.  From 2^34 on fp32 numbers are more than 746 apart.  Sums differ in the last places, and a row's log-sum-exp is
# rounded alike on both sides.
@pytest.mark.parametrize("W,V", [(6, 1000), (6, 3000), (6, 40001), (6, 131001), (33, 131081)])
@pytest.mark.parametrize("big", [2.0 ** 33, 2.0 ** 34, 1.8e10, 1e12])
def test_growth_with_forced_tokens_and_rows_without_any(W, V, big):
    cfg = _cfg(3, 2, W, V, seed=31)

    def fn(d):
        x = wl.expansion_inputs(cfg, d)
        for p in range(x.shape[1]):
            at = (0, V // 2 + 7, V - 1)[p % 3]
            x[0, p, at] = big
            x[1, p] = -big
            if p % 2:
                x[2, p] = -big
            else:
                x[2, p, at] = big
        return x
    _expand_both(cfg, logits_fn=fn, check_margin=False)
    if W < 33:
        attach_both(cfg, logits_fn=fn, check_margin=False)


@pytest.mark.parametrize("W,V", [(6, 3000), (20, 5000), (40, 9000)])
@pytest.mark.parametrize("share", [1.0, 0.9])
def test_nan_logits_stay_inside_their_sequence(W, V, share):
    """NaN logits leave a sequence's own tree undefined, but no call may leave the buffers: the sequences beside it come out as
    ever, and the carried pool says no more than it can hold.  share: how much of the middle sequence's logits is NaN."""
    B, D = 3, 3
    cfg = _cfg(B, D, W, V)
    for op, name in ((ygg.OP_EXPAND, "expand"), (ygg.OP_ATTACH, "attach")):
        parent = np.full((B, cfg.n_nodes), -9, np.int32); token = parent.copy(); cum = np.zeros((B, cfg.n_nodes), np.float32)
        parent[:, 0], token[:, 0] = -1, 1
        gp, gt, gc = to_dev(parent.copy()), to_dev(token.copy()), to_dev(cum.copy())
        shape = shape_of(cfg)
        ws = workspace(shape, op)
        gpool = torch.full((ygg.attach_pool_bytes(shape),), 0xA5, dtype=torch.uint8, device=DEV)
        pool = oracle.attach_pool(B, D, W)
        for t in range(1, D + 1):
            x = wl.expansion_inputs(cfg, t)
            y = x.copy()
            y[1][wl.rng(23, t).random(y[1].shape) < share] = np.nan
            if name == "expand":
                oracle.expand(D, W, t, x, parent, token, cum)
                ygg.equal_growth_expand(shape, t, to_dev(y), gp, gt, gc, ws)
            else:
                oracle.attach(D, W, t, x, parent, token, cum, pool)
                ygg.equal_growth_attach(shape, t, to_dev(y), gp, gt, gc, gpool, ws)
            torch.cuda.synchronize()
            if name == "attach":
                assert all(0 <= count <= W * (D - t) for count, _ in read_pool(gpool, B, D, W))
        for got, want in ((gp, parent), (gt, token)):
            assert np.array_equal(got.cpu().numpy()[[0, 2]], want[[0, 2]])
        assert np.abs(gc.cpu().numpy()[[0, 2]] - cum[[0, 2]]).max() <= 1e-5


# all but a few logits of the vocabulary at one value, as a grammar mask leaves them: spread over the chunks, all in one, fewer than
# new nodes; one pass per chunk and several (width 33 of 131080)
@pytest.mark.parametrize("W,V,keep", [(8, 5000, 300), (8, 32000, 5), (33, 9001, 20), (20, 70001, 400), (33, 131080, 900), (64, 3000, 70)])
@pytest.mark.parametrize("value", [-np.inf, -1e9])
@pytest.mark.parametrize("spread", [True, False])
def test_growth_over_a_masked_vocabulary(W, V, keep, value, spread):
    cfg = _cfg(1, 2, W, V, seed=37)

    def fn(d):
        x = wl.expansion_inputs(cfg, d)
        for p in range(x.shape[1]):
            at = wl.rng(37, 100 * d + p).permutation(V)[:keep] if spread else (V // 3 + 17 * p) % (V - keep) + np.arange(keep)
            masked = np.full(V, np.float32(value))
            masked[at] = x[0, p, at]
            x[0, p] = masked
        return x
    _expand_both(cfg, logits_fn=fn, check_margin=False)
    if W < 64:
        attach_both(cfg, logits_fn=fn, check_margin=False)


@pytest.mark.parametrize("low", [-1.0, -2.0])
def test_growth_with_equal_logits_in_later_passes(low):
    """Several passes per chunk: later logits equal to the threshold of the passes before must lose against those, and the first
    larger ones come in the middle of a chunk."""
    cfg = _cfg(1, 2, 33, 131080)

    def fn(d):
        x = np.full((1, 1 if d == 1 else 33, 131080), np.float32(low))
        x[:, :, 6000::7] = -1.0
        return x
    _expand_both(cfg, logits_fn=fn, check_margin=False)
