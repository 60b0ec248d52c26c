"""The drafter's levels (top-k per row, pool, next frontier) at vocabularies and top-k widths off the usual ones, and an extend in which some
sequences have no new entries.

The LM head has one column that is not zero, so a row's logits are a[j] * f exactly, rounded once, f being one number of the drafter's output:
the order of the candidates, ties included, is known on the host, f follows from the two best ones' distance, and the scores from f in
64 bits."""
import dataclasses

import numpy as np
import pytest
import torch

from synth import TINY, fill_kv_pool

from gpu_util import make_engine, make_models

pytestmark = pytest.mark.gpu

U = 2.0 ** -24   # half a unit of fp32


def _inputs(cfg, B, stride, n_new, seed):
    rng = np.random.default_rng(seed)
    dev = lambda a: torch.from_numpy(a).cuda()
    tok = rng.integers(0, cfg.vocab, size=(B, stride)).astype(np.int32)
    src = rng.integers(0, 3, size=(B, stride)).astype(np.int32)
    hid = rng.normal(size=(B, 3, cfg.hidden)).astype(np.float32)
    return dev(tok), dev(src), dev(np.array(n_new, np.int32)), dev(hid)


def _check_row(tokens, logp, a, K, slack):
    """tokens, logp [K] of one row against the K best of a[j] * f; returns the largest score error."""
    sign = 1.0 if a[tokens[0]] > 0 else -1.0
    order = np.lexsort((np.arange(len(a)), -sign * a))[:K]          # value descending, index ascending
    np.testing.assert_array_equal(tokens, order)
    f = (logp[0] - logp[1]) / (a[order[0]] - a[order[1]])
    l = a * f
    lse = l.max() + np.log(np.exp(l - l.max()).sum())
    err = np.abs(logp - (l[order] - lse)).max()
    # the two scores that f comes from and the score itself are rounded once each, f is twice their distance and counts in the logit and
    # in the sum; the sum's own roundings and the logarithm's are a few of its 40 or so in a row, relative to 1 and to the result
    assert err <= U * (10 * slack + 2 * abs(lse) + 16), (err, slack, lse)
    return float(err)


# segments of 2048 logits and K of them per lane of a merging wave: 5, 10 and 20 in registers, or none; more than 128 segments; rows whose
# last segment is short, whose length is not a multiple of four, shorter than a wave; rows of one segment, whole and in part, in 16-byte pieces
@pytest.mark.parametrize("V,K,D,B", [(4099, 2, 3, 3), (50, 5, 3, 2), (152064, 4, 2, 2), (152064, 8, 3, 1), (152064, 10, 3, 2), (152063, 16, 2, 1),
                                     (200001, 16, 3, 1), (270336, 2, 3, 2), (270339, 10, 2, 2), (6144, 16, 3, 2),
                                     (1024, 4, 4, 2), (1024, 16, 3, 3), (2048, 16, 3, 2), (2044, 8, 3, 2), (2047, 10, 3, 2)])
def test_levels_hold_the_best_candidates_and_their_scores(V, K, D, B):
    cfg = dataclasses.replace(TINY, n_layers=1, hidden=64, mlp=64, vocab=V)
    tw, dw, _, _ = make_models(cfg, 5, "fp32", std=0.2)
    rng = np.random.default_rng(V)
    a = rng.integers(-3 << 17, (3 << 17) + 1, size=V) * 2.0 ** -20   # in [-0.375, 0.375]
    if V > 1000:
        a[rng.integers(0, V, size=V // 8)] = 0.375                   # many equal ones near the top, on both sides
        a[rng.integers(0, V, size=V // 8)] = -0.375
    ends = rng.permutation(V - 1)[:3]
    a[ends[0]], a[ends[1]], a[ends[2]], a[V - 1] = 1.0, 0.5, -0.5, -1.0
    tw["lm_head"].zero_()
    tw["lm_head"][:, 0] = torch.from_numpy(a).float().cuda()
    tw["final_norm"][0] = 9.0
    ctxs = np.arange(3, 3 + B, dtype=np.int32) * 7
    e, _, _ = make_engine(cfg, "fp32", tw, dw, B, 8, D, K, 128, seed=3, seq_len=ctxs)
    dk, dv = fill_kv_pool(1, e.dkv.k_pool.shape[1], cfg.n_kv_heads, cfg.page_size, cfg.head_dim, 6)
    e.dkv.k_pool.copy_(dk)
    e.dkv.v_pool.copy_(dv)
    print(f"draft levels V={V} K={K} D={D} B={B}", flush=True)
    tok, src, n_new, hid = _inputs(cfg, B, 2, [1 + b % 2 for b in range(B)], 1)
    e.ctx.draft_expand(B, D, K, 4, tok, src, n_new, hid, None, e.dkv, e.tree(4))
    pool_tok, pool_par, pool_sc = (x.cpu().numpy() for x in e.ctx.draft_pool(B, D, K))
    pool_sc, KK, worst = pool_sc.astype(np.float64), K * K, 0.0
    for b in range(B):
        assert np.all(pool_par[b, :K] == -1)
        worst = max(worst, _check_row(pool_tok[b, :K], pool_sc[b, :K], a, K, np.abs(pool_sc[b, :K]).max()))
        frontier = np.arange(K)
        for level in range(1, D):
            base = K + (level - 1) * KK
            np.testing.assert_array_equal(pool_par[b, base: base + KK], np.repeat(frontier, K))
            for r in range(K):
                at = slice(base + r * K, base + (r + 1) * K)
                sc = pool_sc[b, at]
                worst = max(worst, _check_row(pool_tok[b, at], sc - pool_sc[b, frontier[r]], a, K, np.abs(sc).max()))
            sc = pool_sc[b, base: base + KK]
            frontier = base + np.lexsort((np.arange(KK), -sc))[:K]
    print(f"  largest error of a score {worst:.2e}", flush=True)
    e.ctx.close()


@pytest.mark.parametrize("V,K", [(50, 5), (1024, 4), (2048, 16), (4099, 4)])     # one segment, in 16-byte pieces or not; several
@pytest.mark.parametrize("bad", ["all NaN", "one NaN", "one infinite", "all infinite"])
def test_logits_without_an_order_leave_scores_and_a_tree_that_have_one(bad, V, K):
    """What is no number is no candidate, scores are numbers or -inf, and the tree has its n nodes, each behind its parent, and nothing behind them."""
    cfg = dataclasses.replace(TINY, n_layers=1, hidden=64, mlp=64, vocab=V)
    tw, dw, _, _ = make_models(cfg, 5, "fp32", std=0.2)
    if bad == "all NaN":
        tw["lm_head"].fill_(float("nan"))
    elif bad == "one NaN":
        tw["lm_head"][V // 2] = float("nan")
    else:       # (one column: plus or minus infinity, as the drafter's output has it)
        rows = slice(None) if bad == "all infinite" else V // 2
        tw["lm_head"][rows] = 0
        tw["lm_head"][rows, 0] = float("inf")
    B, D, n = 2, 3, 6
    e, _, _ = make_engine(cfg, "fp32", tw, dw, B, 8, D, K, 128, seed=3, seq_len=np.array([9, 40], np.int32))
    e.dkv.k_pool.normal_(generator=torch.Generator(device="cuda").manual_seed(1))
    e.dkv.v_pool.normal_(generator=torch.Generator(device="cuda").manual_seed(2))
    wide = e.tree(n).empty(B + 1, n)
    for x in vars(wide).values():
        x.fill_(77)
    t = type(wide)(**{k: x[:B] for k, x in vars(wide).items()})
    print(f"draft levels without an order: {bad} V={V} K={K}", flush=True)
    e.ctx.draft_expand(B, D, K, n, *_inputs(cfg, B, 2, [1, 2], 1), None, e.dkv, t)
    tok, par, sc = (x.cpu().numpy() for x in e.ctx.draft_pool(B, D, K))
    assert not np.isnan(sc).any() and (sc < 1e-5).all()
    assert (tok >= -1).all() and (tok < V).all()
    if bad == "all NaN":
        assert (tok == -1).all() and np.isneginf(sc).all()
    parent = t.parent.cpu().numpy()
    assert (parent[:, 0] == -1).all() and (parent[:, 1:] >= 0).all() and (parent < np.arange(n)).all()
    assert not torch.isnan(t.score).any()
    for k, x in vars(wide).items():
        assert (x[B] == 77).all(), k
    e.ctx.close()


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_sequences_without_new_entries_keep_their_row_and_cache(dtype):
    cfg = dataclasses.replace(TINY, n_layers=1, hidden=256, head_dim=128 if dtype == "bf16" else 64, vocab=4096)
    B, K, D = 4, 4, 2
    ctxs = np.array([9, 40, 0, 21], np.int32)
    tw, dw, _, _ = make_models(cfg, 5, dtype, std=0.1)
    e, table, dtable = make_engine(cfg, dtype, tw, dw, B, 8, D, K, 128, seed=3, seq_len=ctxs)
    e.dkv.k_pool.normal_(generator=torch.Generator(device="cuda").manual_seed(1))
    e.dkv.v_pool.normal_(generator=torch.Generator(device="cuda").manual_seed(2))
    print(f"extend without new entries {dtype}", flush=True)
    e.ctx.draft_expand(B, D, K, 6, *_inputs(cfg, B, 3, [3, 1, 2, 2], 1), None, e.dkv, e.tree(6))
    first = [x.clone() for x in e.ctx.draft_pool(B, D, K)]
    e.dkv.seq_len_bound += 3
    e.dkv.seq_len[2] = 0                                             # sequence 2: a kept row, nothing in its cache
    lens = e.dkv.seq_len.clone()
    before = [p.clone() for p in (e.dkv.k_pool, e.dkv.v_pool)]
    n_new = [0, 2, 0, 0]
    inputs = _inputs(cfg, B, 3, n_new, 2)
    e.ctx.draft_expand(B, D, K, 6, *inputs, None, e.dkv, e.tree(6))
    second = e.ctx.draft_pool(B, D, K)
    torch.cuda.synchronize()
    assert torch.equal(e.dkv.seq_len, lens + torch.tensor(n_new, dtype=torch.int32, device="cuda"))
    for b in (0, 2, 3):
        # the root's distribution is that of the row kept last time; deeper levels see the same committed entries but for sequence 2,
        # emptied (in bf16 their attention may be cut otherwise, and a tie fall the other way)
        m = K if b == 2 or dtype == "bf16" else first[0].shape[1]
        assert torch.equal(first[0][b, :m], second[0][b, :m])
        assert float((first[2][b, :m] - second[2][b, :m]).abs().max()) <= (1e-5 if dtype == "fp32" else 2e-2)
        slots = np.arange(int(lens[b]))                              # committed entries as they were
        pg, off = torch.from_numpy(dtable[b, slots // cfg.page_size].astype(np.int64)), torch.from_numpy(slots % cfg.page_size)
        for old, new in zip(before, (e.dkv.k_pool, e.dkv.v_pool)):
            assert torch.equal(old.cpu()[:, pg, :, off], new.cpu()[:, pg, :, off])
    # the sequence with new entries as in a batch of its own
    f, _, _ = make_engine(cfg, dtype, tw, dw, 1, 8, D, K, 128, seed=3, seq_len=ctxs[1:2])
    f.dkv.k_pool.copy_(before[0][:, : f.dkv.k_pool.shape[1]])
    f.dkv.v_pool.copy_(before[1][:, : f.dkv.v_pool.shape[1]])
    need = (int(lens[1]) + cfg.page_size - 1) // cfg.page_size
    f.dkv.block_table[0, :].copy_(torch.arange(f.dkv.block_table.shape[1], dtype=torch.int32))
    for p in range(need):
        for old, new in zip(before, (f.dkv.k_pool, f.dkv.v_pool)):
            new[:, p] = old[:, int(dtable[1, p])]
    f.dkv.seq_len.copy_(lens[1:2])
    f.dkv.seq_len_bound = int(lens[1])
    f.ctx.draft_expand(1, D, K, 6, *(x[1:2].contiguous() for x in inputs), None, f.dkv, f.tree(6))
    alone = f.ctx.draft_pool(1, D, K)
    torch.cuda.synchronize()
    tol = 1e-4 if dtype == "fp32" else 2e-2
    if dtype == "fp32":
        assert torch.equal(alone[0][0], second[0][1])
    assert float((alone[2][0, 0] - second[2][1, 0]).abs()) <= tol * float(alone[2].abs().max())
