"""Prompts through tlt_prefill (several chunks of a sequence per pass) against the same prompts chunk by chunk: caches, lengths,
slots that no prompt token owns, and the step that follows."""
import dataclasses

import numpy as np
import pytest
import torch

from synth import TINY, prompts

from gpu_util import make_engine, make_models

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
