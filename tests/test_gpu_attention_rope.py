"""fp32 attention that rotates its rows and writes the new keys and values itself (few rows per sequence), against the rotary kernel and the row
attention one after the other: outputs and cache."""
import dataclasses

import numpy as np
import pytest
import torch

from synth import TINY

from gpu_util import make_engine, make_models

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,ctxs", [
    (64, 8, [0, 1, 300]), (64, 1, [63]), (64, 5, [59, 64, 255, 1025]),      # an angle per thread; a tile that ends with old, new and no keys
    (128, 4, [30, 257]), (192, 2, [64, 5]), (256, 2, [127, 700]),           # lanes without a value row at 192
])
def test_as_in_two_kernels(d, n, ctxs):
    """A tree of n rows, and the same tree followed by rows that nothing sees, which makes it too long for the fused kernel."""
    cfg = dataclasses.replace(TINY, name=f"tiny-d{d}", head_dim=d, hidden=256, mlp=320, vocab=97)
    pad = 64 * 4 // (d // 2) + 1     # one row more than there are threads for
    tw, dw, _, _ = make_models(cfg, 11, "fp32", std=0.05)
    rng = np.random.default_rng(d + n)
    B = len(ctxs)
    out, cache = [], []
    for rows in (n, pad):
        e, _, _ = make_engine(cfg, "fp32", tw, dw, B, 64, 2, 2, 1200, seed=3, seq_len=np.array(ctxs, np.int32))
        g = torch.Generator(device="cuda").manual_seed(5)
        e.kv.k_pool.normal_(0, 1, generator=g)
        e.kv.v_pool.normal_(0, 1, generator=g)
        t = e.tree(rows)
        rng = np.random.default_rng(d + n)
        parent, token = np.full((B, rows), -1, np.int32), np.zeros((B, rows), np.int32)
        for b in range(B):
            for i in range(n):
                parent[b, i] = rng.integers(max(0, i - 3), i) if i else -1
                token[b, i] = rng.integers(cfg.vocab)
            parent[b, n:] = 0        # children of the root behind the tree: no row of it sees them
        t.parent.copy_(torch.from_numpy(parent))
        t.token.copy_(torch.from_numpy(token))
        e.ctx.tree_finalize(B, t)
        hid = torch.zeros((B, rows, cfg.hidden), device="cuda")
        print(f"rotating attention d={d} rows={rows} ctx={ctxs}", flush=True)
        e.ctx.verify_forward(B, t, e.kv, out_hidden=hid)
        torch.cuda.synchronize()
        out.append(hid[:, :n].cpu())
        cache.append([x.clone() for x in (e.kv.k_pool, e.kv.v_pool)])
        slots = [(e.kv.block_table[b, (c + i) // 16].item(), (c + i) % 16) for b, c in enumerate(ctxs) for i in range(n)]
        e.ctx.close()
    scale = out[1].abs().max()
    # (the products of so few rows and of more sum in one order, the norms in two: the same within the roundings of a forward of two blocks)
    assert float((out[0] - out[1]).abs().max()) <= 64 * 2.0 ** -24 * float(scale) * cfg.n_layers * 8
    for x, y in zip(*cache):
        for page, row in slots:
            assert float((x[0, page, :, row] - y[0, page, :, row]).abs().max()) <= 64 * 2.0 ** -24 * float(y.abs().max())


def _pools(e):
    return [x.clone() for kv in (e.kv, e.dkv) for x in (kv.k_pool, kv.v_pool)]


@pytest.mark.parametrize("bias", [False, True])
@pytest.mark.parametrize("d,n,ctxs,hole", [
    (64, 8, [504], None), (64, 5, [0, 59, 255, 507], 1), (64, 1, [0, 1, 511], 2),     # 512 keys, the most; a page short in a context or under the new rows
    (128, 4, [30, 257], 1), (192, 2, [64, 510], None), (256, 2, [127, 5], 0),
])
def test_verification_has_the_bits_of_the_two_kernels(d, n, ctxs, hole, bias):
    """A larger bound of the lengths sends the same rows through the rotary kernel and the row attention: hidden states, and every row of both
    caches in every layer, are the same bit for bit; one key more than 512 goes there by itself."""
    cfg = dataclasses.replace(TINY, name=f"tiny-d{d}", head_dim=d, hidden=256, mlp=320, vocab=97, n_layers=3)
    tw, dw, _, _ = make_models(cfg, 11, "fp32", std=0.05, qkv_bias=bias)
    B, rng, out = len(ctxs), np.random.default_rng(d + n), []
    parent, token = np.full((B, n), -1, np.int32), rng.integers(cfg.vocab, size=(B, n)).astype(np.int32)
    for b in range(B):
        for i in range(1, n):
            parent[b, i] = rng.integers(max(0, i - 3), i)
    for bound in (max(ctxs), 1100):
        e, _, _ = make_engine(cfg, "fp32", tw, dw, B, 16, 2, 2, 1200, seed=3, seq_len=np.array(ctxs, np.int32))
        g = torch.Generator(device="cuda").manual_seed(5)
        for x in (e.kv.k_pool, e.kv.v_pool):
            x.normal_(0, 1, generator=g)
        if hole is not None:
            e.kv.block_table[hole, ctxs[hole] // cfg.page_size] = -1
        e.kv.seq_len_bound = bound
        t = e.tree(n)
        t.parent.copy_(torch.from_numpy(parent))
        t.token.copy_(torch.from_numpy(token))
        e.ctx.tree_finalize(B, t)
        hid = torch.full((B, n, cfg.hidden), float("nan"), device="cuda")
        print(f"rotating attention d={d} n={n} ctx={ctxs} bound={bound} bias={bias}", flush=True)
        e.ctx.verify_forward(B, t, e.kv, out_hidden=hid)
        torch.cuda.synchronize()
        out.append([hid.clone()] + _pools(e))
        e.ctx.close()
    for x, y in zip(*out):
        assert torch.equal(x, y)


@pytest.mark.parametrize("d,stride,n_new,K,D", [(64, 8, [8, 3, 0, 1], 4, 4), (64, 3, [1, 3, 2], 8, 3), (128, 4, [4, 2], 3, 4)])
def test_drafter_levels_have_the_bits_of_the_two_kernels(d, stride, n_new, K, D):
    """Extension rows that are not active, and provisional rows behind other ones: the candidates, their scores and the drafter's cache."""
    cfg = dataclasses.replace(TINY, name=f"tiny-d{d}", head_dim=d, hidden=256, mlp=320, vocab=97)
    tw, dw, _, _ = make_models(cfg, 11, "fp32", std=0.05)
    B, out = len(n_new), []
    for bound in (90, 1100):
        e, _, _ = make_engine(cfg, "fp32", tw, dw, B, 16, D, K, 1300, seed=3, seq_len=np.arange(B, dtype=np.int32) * 29 + 3)
        g = torch.Generator(device="cuda").manual_seed(5)
        for x in (e.dkv.k_pool, e.dkv.v_pool):
            x.normal_(0, 1, generator=g)
        dev = lambda a: torch.from_numpy(np.asarray(a, np.int32)).cuda()
        hid = torch.randn((B, stride, cfg.hidden), generator=g, device="cuda")
        rng = np.random.default_rng(d)
        tok, src = rng.integers(cfg.vocab, size=(B, stride)), rng.integers(stride, size=(B, stride))
        for step in range(2):        # (the second: a sequence without new entries has a row that was kept)
            e.dkv.seq_len_bound = bound + 8 * step
            print(f"rotating attention, drafter d={d} stride={stride} bound={bound} step={step}", flush=True)
            e.ctx.draft_expand(B, D, K, 9, dev(tok), dev(src), dev(np.maximum(n_new, 1) if step == 0 else n_new), hid, None, e.dkv, e.tree(9))
            out.append([x.clone() for x in e.ctx.draft_pool(B, D, K)] + _pools(e))
        e.ctx.close()
    for a, b in ((out[0], out[2]), (out[1], out[3])):
        for x, y in zip(a, b):
            assert torch.equal(x, y)
