"""Prompts through tlt_prefill (several chunks of a sequence per pass) against the same prompts chunk by chunk: caches, lengths,
slots that no prompt token owns, and the step that follows."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import decoder as dec
from synth import TINY, prompts

from gpu_util import dense_cache, make_engine, make_models

pytestmark = pytest.mark.gpu

WIDE = dataclasses.replace(TINY, hidden=512, n_q_heads=6, n_kv_heads=2, head_dim=128, mlp=1024, vocab=4096)   # MFMA attention
PLAIN = dataclasses.replace(TINY, vocab=32768)   # wave-per-row attention; fp32 products


# bodies of two chunks, of a chunk and one token, of many chunks with a short last one; more than one pass; a cache that already
# holds something, of different length per sequence
@pytest.mark.parametrize("dtype,cfg,B,P,chunk,lens", [
    ("bf16", WIDE, 2, 129, None, None), ("bf16", WIDE, 1, 66, None, None), ("bf16", WIDE, 3, 302, None, [0, 5, 83]),
    ("bf16", WIDE, 1, 40, 7, [17]), ("bf16", WIDE, 8, 700, None, None), ("fp32", PLAIN, 2, 150, None, [3, 40]),
    ("fp32", PLAIN, 3, 67, 16, None)])
def test_prefill_equals_chunk_by_chunk(dtype, cfg, B, P, chunk, lens, monkeypatch):
    tw, dw, _, _ = make_models(cfg, 5, dtype, std=0.05)
    tol = 1e-4 if dtype == "fp32" else 2e-2
    pr = prompts(B, P, cfg.vocab, seed=3)
    start = np.zeros(B, np.int32) if lens is None else np.array(lens, np.int32)
    K, D, N = 3, 3, 8
    engines = []
    for chunkwise in (True, False):
        e, table, dtable = make_engine(cfg, dtype, tw, dw, B, 64, D, K, P + 220, seed=4, seq_len=start)
        gen = torch.Generator(device="cuda").manual_seed(1)
        for kv, tab in ((e.kv, table), (e.dkv, dtable)):   # what the caches hold is random, what they do not is NaN: it must not be read
            for pool in (kv.k_pool, kv.v_pool):
                pool.fill_(float("nan"))
                for b in range(B):
                    for s in range(int(start[b])):
                        row = pool[:, int(tab[b, s // cfg.page_size]), :, s % cfg.page_size]
                        row.normal_(generator=gen)
        used = []
        real = e.ctx.prefill
        monkeypatch.setattr(e.ctx, "prefill", lambda *a, real=real, no=chunkwise: False if no else used.append(real(*a)) or used[-1])
        print(f"prefill {dtype} B {B} P {P} chunkwise {chunkwise}", flush=True)
        e.prefill(pr, chunk)
        torch.cuda.synchronize()
        assert chunkwise or used == [True]
        engines.append(e)
    a, b = engines
    for x, y in ((a.kv, b.kv), (a.dkv, b.dkv)):
        assert torch.equal(x.seq_len, y.seq_len) and x.seq_len_bound == y.seq_len_bound
        assert torch.equal(x.seq_len.cpu(), torch.from_numpy(start + P - 1))
        for p, q in ((x.k_pool, y.k_pool), (x.v_pool, y.v_pool)):
            hole = torch.isnan(p)
            assert torch.equal(hole, torch.isnan(q))   # the same slots written
            d = (p.float() - q.float())[~hole].abs().max() / p.float()[~hole].abs().max()
            assert float(d) <= tol, float(d)
    assert torch.equal(a.root, b.root)
    al = [e.step(K, D, N) for e in engines]
    if dtype == "fp32":
        assert all(np.array_equal(x, y) for x, y in zip(*al))
        ta, tb = (e.tree(N) for e in engines)   # grown from the drafter's output at the prompt's last position
        assert torch.equal(ta.token, tb.token) and float((ta.score - tb.score).abs().max()) <= tol * max(1.0, float(ta.score.abs().max()))


# passes of 2048 rows at most, the last with fewer chunks and a shorter last one; bf16 and fp32
@pytest.mark.parametrize("dtype,cfg,B,P", [("bf16", WIDE, 2, 129), ("bf16", WIDE, 3, 302), ("bf16", WIDE, 8, 700), ("fp32", PLAIN, 8, 700)])
def test_step_after_prefill_starts_from_the_last_position(dtype, cfg, B, P, monkeypatch):
    tw, dw, _, _ = make_models(cfg, 5, dtype, std=0.05)
    tol = 1e-4 if dtype == "fp32" else 2e-2
    pr = prompts(B, P, cfg.vocab, seed=3)
    K, pools = 10, []
    for chunkwise in (True, False):
        e, _, _ = make_engine(cfg, dtype, tw, dw, B, 64, 2, K, P + 80, seed=4)
        used, real = [], e.ctx.prefill
        monkeypatch.setattr(e.ctx, "prefill", lambda *a, no=chunkwise: False if no else used.append(real(*a)) or used[-1])
        print(f"step after prefill {dtype} B {B} P {P} chunkwise {chunkwise}", flush=True)
        e.prefill(pr)
        assert chunkwise or used == [True]
        e.step(K, 1, 4)
        pools.append([x.cpu().numpy() for x in e.ctx.draft_pool(B, 1, K)])
        e.ctx.close()
    for b in range(B):
        (ta, _, sa), (tb, _, sb) = ((x[b] for x in p) for p in pools)
        # a logit may be off by tol * max|logit|, the row's log-sum-exp by as much; log V + the best log-probability is at most the largest logit
        # here (the logits are centred on zero, and a log-sum-exp is at least the mean plus log V)
        T = 2 * tol * (np.log(cfg.vocab) + float(sa[0]))
        assert sa[0] > sa[-1] + T           # (the inputs' own: the best token of another row, missing in the other list, breaks the last bound)
        for t1, s1, t2, s2 in ((ta, sa, tb, sb), (tb, sb, ta, sa)):
            for k in range(K):
                same = np.flatnonzero(t2 == t1[k])
                if len(same):
                    assert abs(s1[k] - s2[same[0]]) <= T
                else:
                    assert s1[k] <= s2[-1] + T                         # one that the other side left out is no better than its last


@pytest.mark.parametrize("B,P", [(1, 602), (5, 400)])
def test_keys_and_values_are_as_near_to_64_bits_as_chunk_by_chunk(B, P, monkeypatch):
    """First block's keys and values of a pass of more than 256 rows, whose q/k/v product is stored in the model dtype, and of chunks of 64
    rows, whose product arrives at the rotary kernel as fp32 slices: both round it to bf16 there and the rotated result again."""
    cfg = WIDE
    tw, dw, tw64, _ = make_models(cfg, 5, "bf16", std=0.05, qkv_bias=True)
    pr = prompts(B, P, cfg.vocab, seed=3)
    lw, rms, want = tw64["layers"][0], lambda d: float(np.sqrt((d * d).mean())), []
    for b in range(B):
        x = dec.round_to_bf16(dec.rmsnorm(tw64["embed"][pr[b, :-1]], lw["attn_norm"], cfg.rms_eps))
        rows = (x @ lw["wqkv"].T + lw["bqkv"])[:, cfg.q_dim:].reshape(P - 1, 2 * cfg.n_kv_heads, cfg.head_dim)
        want.append((dec.rope(rows[:, : cfg.n_kv_heads], np.arange(P - 1), cfg.rope_theta), rows[:, cfg.n_kv_heads:]))
    seen = []
    for chunkwise in (True, False):
        e, table, _ = make_engine(cfg, "bf16", tw, dw, B, 64, 2, 2, P + 20, seed=4)
        if chunkwise:
            monkeypatch.setattr(e.ctx, "prefill", lambda *a: False)
        print(f"prefill, keys against 64 bits B {B} P {P} chunkwise {chunkwise}", flush=True)
        e.prefill(pr)
        torch.cuda.synchronize()
        seen.append([[rms(dense_cache(pool, table, b, P - 1, cfg.page_size)[0] - w)
                      for pool, w in zip((e.kv.k_pool, e.kv.v_pool), want[b])] for b in range(B)])
        e.ctx.close()
    for b in range(B):
        for i in range(2):
            once = rms(dec.round_to_bf16(want[b][i]) - want[b][i])
            print(f"  {'kv'[i]}: rounded once {once:.3e}, chunk by chunk {seen[0][b][i]:.3e}, in one pass {seen[1][b][i]:.3e}", flush=True)
            # two roundings of the same size (1.41), a few elements of the rows that the norm rounds the other way
            assert seen[1][b][i] <= 1.02 * seen[0][b][i] and seen[1][b][i] <= 1.5 * once


def test_prompts_of_another_count_than_the_engines_change_nothing():
    e, _, _ = make_engine(WIDE, "bf16", *make_models(WIDE, 5, "bf16", std=0.05)[:2], 3, 64, 2, 2, 400, seed=4)
    for B in (2, 4):
        with pytest.raises(RuntimeError):
            e.prefill(prompts(B, 200, WIDE.vocab, seed=3))
        torch.cuda.synchronize()
        for kv in (e.kv, e.dkv):
            assert kv.seq_len_bound == 0 and not kv.seq_len.any() and not kv.k_pool.any()
    e.prefill(prompts(1, 200, WIDE.vocab, seed=3))                     # (one prompt: the first sequence's)
    assert e.kv.seq_len.tolist() == e.dkv.seq_len.tolist() == [199, 0, 0]
    e.ctx.close()
