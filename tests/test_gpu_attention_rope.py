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
