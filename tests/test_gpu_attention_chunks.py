"""The cut of the cached keys into chunks, at sizes where a round of the chip decides: the planner's lists against its rule,
and the merge with four waves per row (where a sequence can have 17 chunks or more, up to 512 rows)."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import attention_plan_model as model  # noqa: E402
from gpu_util import check_draft_tree_against_forced_oracle, dense_cache, make_engine, make_models  # noqa: E402
from oracle import decoder as dec  # noqa: E402
from oracle import sd  # noqa: E402
from paper_2511_16665_amd import binding as tlt  # noqa: E402
from synth import MID, fill_kv_pool, lognormal_contexts, random_block_table  # noqa: E402

pytestmark = pytest.mark.gpu


def _run(Hq, Hkv, n, ctxs, check):
    d, page, B = 128, 16, len(ctxs)
    lens = np.array(ctxs, dtype=np.int32)
    table, n_pages = random_block_table(lens + n + 8, page, seed=5, extra_pages=3)
    gen = torch.Generator(device="cuda").manual_seed(n + B)
    k, v = (torch.empty((n_pages, Hkv, page, d), dtype=torch.bfloat16, device="cuda").normal_(0.0, 1.0, generator=gen) for _ in range(2))
    qkv = (1.5 * torch.randn((B, n, (Hq + 2 * Hkv) * d), generator=gen, device="cuda")).bfloat16()
    mask = torch.tensor([(1 << (i + 1)) - 1 for i in range(n)], dtype=torch.int64, device="cuda").repeat(B, 1)   # a chain
    table = torch.from_numpy(table.astype(np.int32)).cuda()
    kv = tlt.KV(k, v, table, torch.from_numpy(lens).cuda(), int(lens.max()))
    out = torch.full((B, n, Hq * d), 7.0, dtype=torch.bfloat16, device="cuda")
    ws = tlt.attention_workspace(B, n, Hq, Hkv, d, int(lens.max()) + n + 8)
    print(f"attention chunks Hq={Hq} Hkv={Hkv} n={n} B={B} longest={lens.max()}", flush=True)
    assert tlt.attention(tlt.TLT_BF16, Hq, page, qkv, mask, kv, out, ws, 1) == 0
    torch.cuda.synchronize()
    planned = ws[:16 + 8 * B].view(torch.int32).cpu().numpy()   # items, three words of padding, first slots, chunks of each sequence
    for b in check:
        c, G = int(lens[b]), Hq // Hkv
        pages = table[b, :(c + n + page - 1) // page].long()
        K, V = (x[pages].permute(1, 0, 2, 3).reshape(Hkv, -1, d)[:, :c + n].float() for x in (k, v))
        q = qkv[b, :, :Hq * d].float().view(n, Hkv, G, d)
        visible = torch.arange(c + n, device="cuda")[None, :] <= c + torch.arange(n, device="cuda")[:, None]
        for h in range(Hkv):
            s = (q[:, h].reshape(n * G, d) @ K[h].T) / d ** 0.5
            s = s.view(n, G, -1).masked_fill(~visible[:, None, :], float("-inf")).view(n * G, -1)
            want = (torch.softmax(s, -1) @ V[h]).view(n, G, d)
            got = out[b].float().view(n, Hkv, G, d)[:, h]
            # (P and the output are rounded to bf16: 2^-8 of the largest output)
            assert ((got - want).abs().max() <= 1e-2 * want.abs().max()).item(), (b, h)
    assert planned[0] == planned[4 + B:].sum()
    return planned[4 + B:]


# several rounds of items and one: equal lengths, single tiles and short sequences among them, lognormal ones, lengths at multiples of the chunk length
@pytest.mark.parametrize("heads,ctxs", [
    (32, [8200] * 8), (6, [6500] * 38 + [1, 700]), (16, [16383] * 12 + [16400, 5000, 64]), (16, lognormal_contexts(15, 3846, 0.2, 15384, 256, 0)),
    (8, lognormal_contexts(14, 8200, 0.8, 32768, 256, 0)), (4, [8191] * 64), (16, [16383] * 15 + [64]), (1, [1267 * 64 - 1] * 35 + [367 * 64 - 1])])
def test_planned_chunks(heads, ctxs):
    tiles = model.tiles_of(ctxs, 1)
    got = _run(heads, heads, 1, ctxs, [0, len(ctxs) - 3, len(ctxs) - 2, len(ctxs) - 1])
    assert got.tolist() == model.counts(tiles, model.chunk_size(tiles, heads)).tolist()


# sequences of 16, 17, 65 and 129 chunks of the shortest length, one of two, one long sequence among short ones; 512 and 513 rows (one row beyond the limit)
@pytest.mark.parametrize("Hq,Hkv,n,ctxs,chunks", [
    (4, 4, 1, [64 * 64 - 1], [16]), (4, 4, 1, [64 * 64], [17]), (2, 1, 3, [64 * 260 - 3], [65]), (1, 1, 1, [64 * 513 - 1], [129]), (4, 1, 2, [9000, 500], [36, 2]),
    (28, 4, 1, [30000, 1500, 700, 0], [53, 3, 2, 1]), (16, 2, 32, [8000], [32]), (27, 1, 19, [8000], [32])])
def test_merge_of_many_chunks(Hq, Hkv, n, ctxs, chunks):
    assert _run(Hq, Hkv, n, ctxs, range(len(ctxs))).tolist() == chunks


@pytest.mark.parametrize("ctxs", [[8192], [30000]])
def test_one_and_four_waves_per_row_give_the_same_bits(ctxs):
    """18 nodes of 28 heads are 504 rows, which four waves merge, 19 are 532.  Of a kv head's 7 rows per node, the first 16 nodes' fill seven row tiles, which hold
    the same rows either way."""
    Hq, Hkv, d, page, outs = 28, 4, 128, 16, []
    gen = torch.Generator(device="cuda").manual_seed(4)
    lens = np.array(ctxs, dtype=np.int32)
    table, n_pages = random_block_table(lens + 27, page, seed=5, extra_pages=3)
    table = torch.from_numpy(table.astype(np.int32)).cuda()
    k, v = (torch.empty((n_pages, Hkv, page, d), dtype=torch.bfloat16, device="cuda").normal_(0.0, 1.0, generator=gen) for _ in range(2))
    qkv = (1.5 * torch.randn((1, 19, (Hq + 2 * Hkv) * d), generator=gen, device="cuda")).bfloat16()
    mask = torch.tensor([[(2 << i) - 1 for i in range(19)]], dtype=torch.int64, device="cuda")
    kv = tlt.KV(k, v, table, torch.from_numpy(lens).cuda(), int(lens.max()))
    for n in (18, 19):
        out = torch.full((1, n, Hq * d), 7.0, dtype=torch.bfloat16, device="cuda")
        ws = tlt.attention_workspace(1, n, Hq, Hkv, d, int(lens.max()) + 27)
        print(f"attention chunks merged, n={n} of {ctxs}", flush=True)
        assert tlt.attention(tlt.TLT_BF16, Hq, page, qkv[:, :n].contiguous(), mask[:, :n].contiguous(), kv, out, ws, 1) == 0
        torch.cuda.synchronize()
        outs.append((out[:, :16], ws[20:24].view(torch.int32).item()))   # (the chunks)
    assert outs[0][1] == outs[1][1] > 16
    assert torch.equal(outs[0][0].view(torch.int16), outs[1][0].view(torch.int16))


def test_four_waves_per_row_with_inactive_rows():
    """The drafter's catch-up, whose rows beyond a sequence's new entries are inactive, all of them in a sequence without any, behind caches of 20 chunks: the trees
    that come of it, against the oracle's drafter."""
    cfg = dataclasses.replace(MID, name="mid-g7", n_q_heads=14, n_layers=1)
    B, K, D, N, stride = 2, 3, 3, 8, 4
    ctxs = np.array([5000, 3000], dtype=np.int32)
    assert model.chunk_size(model.tiles_of(ctxs, 1), cfg.n_kv_heads) == 4 and B * stride * cfg.n_q_heads <= 512
    tw_dev, dw_dev, tw, dw = make_models(cfg, 5, "bf16", std=0.05)
    cap = int(ctxs.max()) + 60
    e, _, dtable = make_engine(cfg, "bf16", tw_dev, dw_dev, B, N, D, K, cap, seed=3, seq_len=ctxs)
    dk, dv = fill_kv_pool(1, e.dkv.k_pool.shape[1], cfg.n_kv_heads, cfg.page_size, cfg.head_dim, 6, dtype=torch.bfloat16)
    e.dkv.k_pool.copy_(dk)
    e.dkv.v_pool.copy_(dv)
    e.ctx.set_attention_impl(1)
    e.dkv.seq_len_bound = int(ctxs.max())
    rng = np.random.default_rng(1)
    dev = lambda a: torch.from_numpy(a).cuda()
    states, last, lens = [], [0] * B, ctxs.copy()
    for b, c in enumerate(ctxs):
        st = sd.SeqState(cfg, cap, dec.round_to_bf16)
        st.draft.k[:c], st.draft.v[:c] = dense_cache(dk, dtable, b, c, cfg.page_size)[0], dense_cache(dv, dtable, b, c, cfg.page_size)[0]
        st.draft_len = int(c)
        states.append(st)
    for n_new in ([3, 1], [0, 2]):
        n_new = np.array(n_new, dtype=np.int32)
        tok, src = rng.integers(0, cfg.vocab, size=(B, stride)).astype(np.int32), rng.integers(0, 5, size=(B, stride)).astype(np.int32)
        hidden, tree = rng.normal(size=(B, 5, cfg.hidden)).astype(np.float32), e.tree(N)
        print(f"drafter behind long caches, new entries {n_new.tolist()}", flush=True)
        e.ctx.draft_expand(B, D, K, N, dev(tok), dev(src), dev(n_new), dev(hidden), None, e.dkv, tree)
        pool = [x.cpu().numpy() for x in e.ctx.draft_pool(B, D, K)]
        e.dkv.seq_len_bound += stride
        lens += n_new
        np.testing.assert_array_equal(e.dkv.seq_len.cpu().numpy(), lens)
        g_tree = [x.cpu().numpy() for x in (tree.token, tree.parent, tree.depth, tree.score)]
        for b in range(B):
            if n_new[b]:
                toks = [int(t) for t in tok[b, :n_new[b]]]
                sd.draft_extend(cfg, tw, dw, states[b], toks, hidden[b][src[b, :n_new[b]]].astype(np.float64))
                last[b] = toks[-1]
                check_draft_tree_against_forced_oracle(sd, cfg, tw, dw, states[b], last[b], K, D, N, tuple(x[b] for x in pool), tuple(x[b] for x in g_tree), 2e-2)
    e.ctx.close()
