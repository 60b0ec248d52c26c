"""tlt_attention (the tree-attention kernels on their own) against the oracle's attention, element by
element, on random trees over random paged caches: both kernels, several key chunks, ragged tails,
a one-row tree, empty contexts, 5 and 7 query heads per kv head."""
import numpy as np
import pytest
import torch

from oracle import decoder as dec
from paper_2511_16665_amd import binding as tlt
from synth import fill_kv_pool, random_block_table

from gpu_util import dense_cache, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,n,ctxs,impl", [
    (8, 2, 13, [0, 37, 150], 1),
    (8, 2, 13, [0, 37, 150], 0),
    (28, 4, 48, [700, 90, 4099], 1),        # 336 query rows per kv head: three row tiles per wave
    (40, 8, 32, [1500, 64, 63, 65], 1),     # 160 rows: waves with one and with two row tiles
    (28, 4, 64, [2100, 5], 1),              # 448 rows: two row groups
    (4, 4, 1, [1, 16, 1000], 1),            # one row, one query head per kv head
    (14, 2, 8, [9000], 1),                  # one long sequence cut into many chunks
    (28, 4, 1, [8191], 1),                  # one row: chunks of the shortest length, more than 16 of them
    (4, 1, 2, [17 * (i % 9) for i in range(70)], 1),   # more sequences than a wave has lanes, many of one tile
    (4, 1, 1, [20001], 1),                  # 79 chunks: more than the merging wave has lanes
])
def test_attention_matches_oracle(Hq, Hkv, n, ctxs, impl):
    d, page = 128, 16
    B = len(ctxs)
    ctxs = np.array(ctxs, dtype=np.int32)
    rng = np.random.default_rng(Hq * 100 + n)
    table, n_pages = random_block_table(ctxs + n + 8, page, seed=3, extra_pages=3)
    k, v = fill_kv_pool(1, n_pages, Hkv, page, d, seed=9, dtype=torch.bfloat16)
    qkv_dim = (Hq + 2 * Hkv) * d
    qkv = (torch.randn((B, n, qkv_dim), generator=torch.Generator().manual_seed(1)) * 1.5).bfloat16()
    parent = np.full((B, n), -1, dtype=np.int64)
    mask = np.zeros((B, n), dtype=np.uint64)
    for b in range(B):
        for i in range(n):
            if i > 0:
                parent[b, i] = rng.integers(max(0, i - 4), i)
            mask[b, i] = (mask[b, parent[b, i]] if i > 0 else np.uint64(0)) | np.uint64(1 << i)
    kv = tlt.KV(k[0].cuda(), v[0].cuda(), torch.from_numpy(table.astype(np.int32)).cuda(), torch.from_numpy(ctxs).cuda(),
                int(ctxs.max()))
    out = torch.full((B, n, Hq * d), 7.0, dtype=torch.bfloat16, device="cuda")
    ws = tlt.attention_workspace(B, n, Hq, Hkv, d, int(ctxs.max()) + n + 8)
    print(f"attention Hq={Hq} Hkv={Hkv} n={n} ctx={list(ctxs)} impl={impl}", flush=True)
    rc = tlt.attention(tlt.TLT_BF16, Hq, page, qkv.cuda(), torch.from_numpy(mask.view(np.int64)).cuda(), kv, out, ws, impl)
    assert rc == 0, tlt.ERRORS.get(rc, rc)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().reshape(B, n, Hq, d)
    q = qkv[:, :, : Hq * d].double().numpy().reshape(B, n, Hq, d)
    for b in range(B):
        c = int(ctxs[b])
        K = dense_cache(k, table, b, c + n, page)[0]
        V = dense_cache(v, table, b, c + n, page)[0]
        visible = np.zeros((n, c + n), dtype=bool)
        visible[:, :c] = True
        for i in range(n):
            for j in range(n):
                visible[i, c + j] = bool((int(mask[b, i]) >> j) & 1)
        want = dec.attention(q[b], K, V, visible)
        assert rel_err(got[b], want) <= 2e-2, (b, rel_err(got[b], want))


@pytest.mark.parametrize("ctx,missing", [
    (900, (1, 40)),    # in a chunk's first two tiles, whose pages come with the work item, and in another chunk's third tile
    (900, (40,)),      # past the first two tiles only
    (30, (1,)),        # a chunk of one tile
])
def test_attention_with_a_page_missing_from_the_table(ctx, missing):
    """A page the block table does not back (a caller's mistake): the kernel takes its keys and values as zero, also after it has
    fetched a chunk's first tiles, and the other sequence is not touched."""
    Hq, Hkv, n, d, page = 8, 2, 5, 128, 16
    ctxs = np.array([ctx, 700], dtype=np.int32)
    table, n_pages = random_block_table(ctxs + n + 8, page, seed=3, extra_pages=3)
    broken = table.copy()
    for i, p in enumerate(missing):
        broken[0, p] = (-1, n_pages)[i % 2]
    k, v = fill_kv_pool(1, n_pages, Hkv, page, d, seed=9, dtype=torch.bfloat16)
    qkv = torch.randn((2, n, (Hq + 2 * Hkv) * d), generator=torch.Generator().manual_seed(1)).bfloat16()
    mask = torch.tensor([[(2 << i) - 1 for i in range(n)]] * 2, dtype=torch.int64).cuda()
    outs = []
    for t in (table, broken):
        kv = tlt.KV(k[0].cuda(), v[0].cuda(), torch.from_numpy(t.astype(np.int32)).cuda(), torch.from_numpy(ctxs).cuda(), int(ctxs.max()))
        out = torch.full((2, n, Hq * d), 7.0, dtype=torch.bfloat16, device="cuda")
        ws = tlt.attention_workspace(2, n, Hq, Hkv, d, int(ctxs.max()) + n + 8)
        print("attention, pages missing:", missing if t is broken else (), flush=True)
        assert tlt.attention(tlt.TLT_BF16, Hq, page, qkv.cuda(), mask, kv, out, ws, 1) == 0
        torch.cuda.synchronize()
        outs.append(out)
    assert torch.equal(outs[0][1], outs[1][1])
    K, V = (dense_cache(x, table, 0, ctx + n, page)[0] for x in (k, v))
    for p in missing:
        K[p * page:(p + 1) * page] = V[p * page:(p + 1) * page] = 0
    visible = np.tril(np.ones((n, ctx + n), dtype=bool), ctx)
    want = dec.attention(qkv[0, :, : Hq * d].double().numpy().reshape(n, Hq, d), K, V, visible)
    assert rel_err(outs[1][0].float().cpu().numpy().reshape(n, Hq, d), want) <= 2e-2


def test_attention_with_more_sequences_than_the_planner_keeps_in_lds():
    B, Hq, Hkv, d, page = 4200, 2, 1, 128, 16
    ctxs = np.array([17 * (i % 9) + (300 if i % 400 == 5 else 0) for i in range(B)], dtype=np.int32)
    table, n_pages = random_block_table(ctxs + 1, page, seed=3, extra_pages=3)
    k, v = fill_kv_pool(1, n_pages, Hkv, page, d, seed=9, dtype=torch.bfloat16)
    qkv = torch.randn((B, 1, (Hq + 2 * Hkv) * d), generator=torch.Generator().manual_seed(1)).bfloat16()
    kv = tlt.KV(k[0].cuda(), v[0].cuda(), torch.from_numpy(table.astype(np.int32)).cuda(), torch.from_numpy(ctxs).cuda(), int(ctxs.max()))
    out = torch.full((B, 1, Hq * d), 7.0, dtype=torch.bfloat16, device="cuda")
    ws = tlt.attention_workspace(B, 1, Hq, Hkv, d, int(ctxs.max()) + 1)
    print(f"attention, {B} sequences", flush=True)
    assert tlt.attention(tlt.TLT_BF16, Hq, page, qkv.cuda(), torch.ones((B, 1), dtype=torch.int64, device="cuda"), kv, out, ws, 1) == 0
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().reshape(B, 1, Hq, d)
    q = qkv[:, :, : Hq * d].double().numpy().reshape(B, 1, Hq, d)
    for b in sorted(set(range(0, B, 5)) | set(range(4080, B))):
        T = int(ctxs[b]) + 1
        K, V = (dense_cache(x, table, b, T, page)[0] for x in (k, v))
        assert rel_err(got[b], dec.attention(q[b], K, V, np.ones((1, T), dtype=bool))) <= 2e-2, b
