"""The work that a rollout program has this library do, as measured cases.

Every case drives the public entry points (paper_2511_16665_amd.engine and .binding) the way a rollout loop does: one pass
is a few consecutive steps of a batch from a fixed starting state (lengths and pending tokens are put back at the start of
a pass; the cache rows that a pass writes are the same ones each time).

kind "decode"   plain decoding: one-node trees, verification forward + greedy acceptance + commit, token fed back on the device
kind "step"     Engine.step: learned drafter, dynamic top-k tree, verification, greedy acceptance, commit
kind "sampled"  Engine.step_sampled: sampled drafting on a static template, rejection-sampling acceptance
kind "ngram"    model-free drafter on the host (NGram.propose) + Engine.step_trees, the learned drafter's cache following along
kind "prefill"  Engine.prefill: a prompt through target and drafter in chains of 64

The model.  Weights are random with the published shapes; so that the tokens behave as in a trained model's rollout (a
clear favourite at most positions, a drafter that is mostly right and sometimes lost) the token tables have structure:
the LM head's row of token v is the sum of the embeddings of the eight tokens that v follows as first, second, ... choice,
and the drafter's input projection passes an embedding on, except for a quarter of the vocabulary (embeddings in a subspace
of its own) whose continuation it cannot see.  Drafts are then accepted for about three tokens on average, and a token that
is emitted leads the next one by many times what rounding can move, so emitted tokens are a fair thing to compare.
What is returned of the hidden states are the rows of the emitted tokens, which is what a drafter's trainer collects from
a rollout: the tree's other rows are guesses whose order hangs on near-ties between scores.  The later steps of a pass
attend to the cache rows that the earlier ones committed.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2511_16665_amd import binding as tlt
from paper_2511_16665_amd import engine as eng
from synth import QWEN7B, QWEN32B, TINY, lognormal_contexts, random_block_table, uniform_contexts

# (32 billion parameters and their cache three times over do not fit one card: a quarter of the blocks, full width)
MODELS = {"tiny": TINY, "7b": QWEN7B, "32b": dataclasses.replace(QWEN32B, n_layers=16)}
CHOICES = (2.0, 1.0, 0.9, 0.8, 0.7, 0.6, 0.5, 0.4)   # weight of a token's first, second, ... successor in the LM head
TEMPERATURE = 0.9


def listed():
    return [
        # the smallest calls: a two-layer fp32 decoder with chain drafts, where launches and host work are everything
        dict(name="tiny fp32 chain", kind="step", model="tiny", batch=2, ctx=128, ctx_kind="fixed", depth=4, topk=1, nodes=5, steps=8),
        # speculation off: one sequence (latency), a middling batch, and the large batch of a rollout's first phase
        dict(name="decode 1", kind="decode", model="7b", batch=1, ctx=8192, ctx_kind="fixed", steps=4),
        dict(name="decode 16", kind="decode", model="7b", batch=16, ctx=8192, ctx_kind="fixed", steps=4),
        dict(name="decode 64", kind="decode", model="7b", batch=64, ctx=8192, ctx_kind="fixed", steps=2),
        # the tail of a rollout: the last sequence with a small tree, then a few with mid-sized ones of odd size
        dict(name="step 1 x 8", kind="step", model="7b", batch=1, ctx=8192, ctx_kind="fixed", depth=7, topk=8, nodes=8, steps=3),
        dict(name="step 3 x 23", kind="step", model="7b", batch=3, ctx=5000, ctx_kind="lognormal", depth=4, topk=4, nodes=23, steps=3),
        # the common case of a rollout with speculation on, a small tree for many sequences and the benchmark's workload
        dict(name="step 16 x 16", kind="step", model="7b", batch=16, ctx=8192, ctx_kind="fixed", depth=8, topk=8, nodes=16, steps=2),
        dict(name="step 32 x 48", kind="step", model="7b", batch=32, ctx=4096, ctx_kind="lognormal", depth=6, topk=8, nodes=48, steps=2),
        # few sequences of 24k-32k tokens, sampled, the largest trees
        dict(name="sampled 4 x 64", kind="sampled", model="7b", batch=4, ctx=32768, ctx_kind="tail", depth=8, topk=10, nodes=64, steps=2),
        # the wider model's blocks
        dict(name="step 16 x 32 wide", kind="step", model="32b", batch=16, ctx=8192, ctx_kind="lognormal", depth=6, topk=8, nodes=32, steps=2),
        # sibling rollouts of a prompt: trees retrieved on the host
        dict(name="ngram 7 x 12", kind="ngram", model="7b", batch=7, ctx=3000, ctx_kind="lognormal", depth=5, topk=3, nodes=12, steps=3),
        # prompts of a group of rollouts into both caches (a ragged last chunk)
        dict(name="prefill 4 x 301", kind="prefill", model="7b", batch=4, ctx=301, ctx_kind="fixed"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "step", "step", "step", "sampled", "ngram", "prefill", "tiny"])
    if kind == "tiny":
        return dict(kind="step", model="tiny", batch=_log(rng, 1, 8), ctx=_log(rng, 40, 600), ctx_kind="lognormal",
                    depth=rng.randint(2, 6), topk=rng.randint(1, 4), nodes=rng.randint(3, 16), steps=8)
    if kind == "decode":
        batch = _log(rng, 1, 64)
        return dict(kind=kind, model=rng.choice(["7b", "7b", "32b"]), batch=batch, ctx=_log(rng, 300, min(16384, 524288 // batch)),
                    ctx_kind=rng.choice(["fixed", "lognormal"]), steps=2)
    if kind == "prefill":
        batch = _log(rng, 1, 8)
        return dict(kind=kind, model="7b", batch=batch, ctx=_log(rng, 40, 1200 // batch), ctx_kind="fixed")
    if kind == "ngram":
        return dict(kind=kind, model="7b", batch=_log(rng, 1, 24), ctx=_log(rng, 500, 8192), ctx_kind="lognormal",
                    depth=rng.randint(3, 6), topk=rng.randint(2, 4), nodes=rng.randint(4, 24), steps=2)
    depth, topk = rng.randint(3, 8), rng.randint(2, 10)
    nodes = min(_log(rng, 6, 64), 1 + topk + (depth - 1) * topk * topk)
    if kind == "sampled":
        return dict(kind=kind, model="7b", batch=rng.randint(1, 4), ctx=_log(rng, 4000, 32768), ctx_kind=rng.choice(["tail", "lognormal"]),
                    depth=depth, topk=topk, nodes=nodes, steps=1)
    batch = _log(rng, 1, min(32, 1536 // nodes))
    model = rng.choice(["7b", "7b", "7b", "32b"])
    return dict(kind=kind, model=model, batch=batch if model == "7b" else min(batch, 16), ctx=_log(rng, 500, 8192 if batch <= 16 else 4096),
                ctx_kind=rng.choice(["fixed", "lognormal"]), depth=depth, topk=topk, nodes=nodes, steps=1)


def _contexts(case, seed):
    B, c = case["batch"], case["ctx"]
    if case["ctx_kind"] == "fixed":
        return np.full(B, c, dtype=np.int32)
    if case["ctx_kind"] == "tail":                     # the long tail: everything but the longest sequences has ended
        return uniform_contexts(B, c * 3 // 4, c, seed)
    # (lengths of a rollout in progress: which sequence has which length comes from the seed, the lengths themselves do not,
    # so that every seed is the same amount of work)
    lens = lognormal_contexts(B, c, 0.8, max(c, min(4 * c, 32768)), min(256, c), 0)
    return np.random.default_rng(seed).permutation(lens).astype(np.int32)


def _mean_context(case):
    return float(np.mean(_contexts(case, 0)))


def _accept_bound(case):
    if case["kind"] == "decode":
        return 1
    return min(case["depth"], case["nodes"] - 1) + 1


def _weights(cfg, gen, dtype):
    """Target and drafter parameters on the GPU (see the module's docstring)."""
    h, V, L = cfg.hidden, cfg.vocab, cfg.n_layers

    def normal(shape, std):
        return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=gen)

    def gain():
        return (1.0 + 0.1 * torch.randn(h, generator=gen, device="cuda")).to(dtype)

    out_std = 0.02 / math.sqrt(2 * L)                  # the usual scaling of the projections that write the residual stream

    def layer():
        return {"attn_norm": gain(), "wqkv": normal((cfg.qkv_dim, h), 0.02), "wo": normal((h, cfg.q_dim), out_std),
                "mlp_norm": gain(), "wg": normal((cfg.mlp, h), 0.02), "wu": normal((cfg.mlp, h), 0.02),
                "wd": normal((h, cfg.mlp), out_std)}

    seen = 3 * h // 4                                  # dimensions of the tokens that the drafter can continue
    lost = torch.rand(V, generator=gen, device="cuda") < 0.25
    embed = normal((V, h), 1.0)
    embed[:, :seen].masked_fill_(lost[:, None], 0)
    embed[:, seen:].masked_fill_(~lost[:, None], 0)
    embed[:, seen:] *= math.sqrt(h / (h - seen))
    embed[:, :seen] *= math.sqrt(h / seen)
    before = [torch.randperm(V, generator=gen, device="cuda") for _ in CHOICES]   # before[k][v]: whose choice k is token v
    scale = 16.0 / (h * (CHOICES[0] - CHOICES[1])) * 1.45   # the first choice leads by about 16
    head = torch.empty((V, h), dtype=dtype, device="cuda")
    for o in range(0, V, 16384):
        part = sum(c * embed[p[o:o + 16384]].float() for c, p in zip(CHOICES, before))
        head[o:o + 16384] = (scale * part).to(dtype)
    fc = torch.zeros((h, 2 * h), dtype=dtype, device="cuda")
    fc[:, h:].normal_(0.0, 0.2 / math.sqrt(h), generator=gen)
    fc[:seen, :seen].fill_diagonal_(1.0)
    turn = torch.linalg.qr(torch.randn((h - seen, h - seen), generator=gen, device="cuda"))[0]
    fc[seen:, seen:h] = turn.to(dtype)
    target = {"embed": embed, "lm_head": head, "final_norm": gain(), "layers": [layer() for _ in range(L)]}
    follow = torch.empty(V, dtype=torch.int64, device="cuda")   # a token's first choice of successor
    follow[before[0]] = torch.arange(V, device="cuda")
    return target, {"fc": fc, "layer": layer()}, follow.cpu().numpy()


def _cache(cfg, L, caps, lens, seed, gen, dtype, code):
    table, pages = random_block_table(caps, cfg.page_size, seed, extra_pages=8)
    shape = (L, pages, cfg.n_kv_heads, cfg.page_size, cfg.head_dim)
    k, v = (torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, 1.0, generator=gen) for _ in range(2))
    return eng.alloc_kv(cfg, code, L, table, pages, lens, fill=(k, v))


def prepare(case, seed):
    cfg = MODELS[case["model"]]
    code = tlt.TLT_F32 if case["model"] == "tiny" else tlt.TLT_BF16
    dtype = tlt.torch_dtype(code)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B, kind, steps = case["batch"], case["kind"], case.get("steps", 1)
    tw, dw, follow = _weights(cfg, gen, dtype)
    if kind == "prefill":
        D, K, N = 1, 1, 64
        lens = np.zeros(B, dtype=np.int32)
        caps = np.full(B, case["ctx"] + 2 * N, dtype=np.int32)
    else:
        D, K, N = case.get("depth", 1), case.get("topk", 1), case.get("nodes", 1)
        lens = _contexts(case, seed)
        caps = lens + (steps + 1) * _accept_bound(case) + N + (D - 1) * K + 80
    kv = _cache(cfg, cfg.n_layers, caps, lens, seed, gen, dtype, code)
    if kind == "decode":
        dw, dkv = None, None
    else:
        dkv = _cache(cfg, 1, caps, lens, seed + 1, gen, dtype, code)
    e = eng.Engine(cfg, code, tw, dw, B, N, D, K, int(caps.max()) + 64, kv, dkv)
    state = {"case": case, "engine": e, "lens": kv.seq_len.clone(), "bound": kv.seq_len_bound}
    host = np.random.default_rng(seed)
    last = host.integers(0, cfg.vocab, size=B)         # the token each sequence ended with
    if kind == "prefill":
        state["prompts"] = host.integers(0, cfg.vocab, size=(B, case["ctx"])).astype(np.int32)
        return state
    state["last"] = torch.from_numpy(last.astype(np.int32)).cuda().view(B, 1)
    if kind == "decode":
        e.tree(1).parent.fill_(-1)
        e.ctx.tree_finalize(B, e.tree(1))
        return state
    state["hidden"] = 1.2 * torch.randn((B, 1, cfg.hidden), generator=gen, device="cuda")
    state["src"] = torch.zeros((B, 1), dtype=torch.int32, device="cuda")
    state["one"] = torch.ones((B,), dtype=torch.int32, device="cuda")
    if kind == "sampled":
        n = len(tlt.template_build(K, D, N)[0])
        u32 = lambda *s: torch.randint(-2**31, 2**31 - 1, s, generator=gen, device="cuda", dtype=torch.int32)  # noqa: E731
        state["uniform"] = [(u32(B, n), u32(B, n), u32(B)) for _ in range(steps)]
    if kind == "ngram":
        # eight finished responses per prompt: the target's own continuations with a departure now and then
        db = tlt.NGram(4)
        for b in range(B):
            for r in range(8):
                t, seq = int(last[b]), []
                for _ in range(200):
                    seq.append(t)
                    t = int(follow[t]) if len(seq) < 8 or host.random() < 0.9 else int(host.integers(cfg.vocab))
                db.insert(b, np.array(seq, dtype=np.int32))
        state["db"], state["last_host"] = db, last.astype(np.int32)
    return state


def _emitted_hidden(e, n):
    """Hidden-state rows of the tokens that the last step emitted: [B, stride, h], path entries past the end read row 0."""
    idx = e.path_idx.clamp(min=0).long().unsqueeze(-1).expand(-1, -1, e.cfg.hidden)
    return torch.gather(e._buf("hid", n), 1, idx)


def run(state):
    case, e = state["case"], state["engine"]
    B, kind, steps = case["batch"], case["kind"], case.get("steps", 1)
    e.kv.seq_len.copy_(state["lens"])
    e.kv.seq_len_bound = state["bound"]
    if kind == "decode":
        t, hid, am = e.tree(1), e._buf("hid", 1), e._buf("am", 1)
        t.token.copy_(state["last"])
        tokens, hidden = [], []
        for _ in range(steps):
            e.ctx.verify_forward(B, t, e.kv, out_argmax=am, out_hidden=hid)
            e.ctx.accept(B, 0, 1.0, t, None, am, None, None, None, e.stride, e.accept_len, e.path_idx, e.out_tokens, e.n_out)
            e.ctx.kv_commit(B, e.kv, e.accept_len, e.path_idx, e.stride)
            e.kv.seq_len_bound += 1
            t.token.copy_(e.out_tokens[:, :1])
            tokens.append(e.out_tokens[:, 0].clone())
            hidden.append(hid.clone())
        return {"tokens": torch.stack(tokens), "hidden": torch.stack(hidden), "lens": e.kv.seq_len}
    e.dkv.seq_len.copy_(state["lens"])
    e.dkv.seq_len_bound = state["bound"]
    if kind == "prefill":
        e.prefill(state["prompts"])
        return {"k": e.kv.k_pool, "v": e.kv.v_pool, "dk": e.dkv.k_pool, "dv": e.dkv.v_pool, "lens": e.kv.seq_len}
    K, D, N = case["topk"], case["depth"], case["nodes"]
    e.set_pending(state["last"], state["src"], state["one"], state["hidden"], 1)
    tokens, accepted, hidden = [], [], []
    if kind == "ngram":
        # (the first proposal continues the prompt's last token; the drafter's cache catches up inside step_trees)
        context = [np.array([x], dtype=np.int32) for x in state["last_host"]]
        for _ in range(steps):
            trees = [state["db"].propose(b, context[b], D, K, N) for b in range(B)]
            al, out = e.step_trees(np.stack([x[0] for x in trees]), np.stack([x[1] for x in trees]), keep_drafter=True)
            context = [np.concatenate([context[b], out[b, :al[b] + 1]])[-4:] for b in range(B)]
            tokens.append(out)
            accepted.append(al)
            hidden.append(_emitted_hidden(e, N))
    else:
        for i in range(steps):
            if kind == "sampled":
                al, out = e.step_sampled(K, D, N, TEMPERATURE, *state["uniform"][i])
                n = len(tlt.template_build(K, D, N)[0])
            else:
                al, out = e.step(K, D, N)
                n = min(N, 1 + K + (D - 1) * K * K)
            tokens.append(out)
            accepted.append(al)
            hidden.append(_emitted_hidden(e, n))
    return {"tokens": np.stack(tokens), "accepted": np.stack(accepted), "hidden": torch.stack(hidden), "lens": e.kv.seq_len}


def work(case):
    """Bytes: the weights of every forward once (a drafter level needs the one before it, so each reads its weights), the
    cached keys and values once per forward.  Flops: the products of every row, and attention over the cached tokens."""
    cfg = MODELS[case["model"]]
    elt = 4 if case["model"] == "tiny" else 2
    B, kind, h, V = case["batch"], case["kind"], cfg.hidden, cfg.vocab
    block = h * cfg.qkv_dim + cfg.q_dim * h + 3 * h * cfg.mlp
    head = h * V

    def forward(rows, layers, ctx, with_head, extra=0):
        params = layers * block + (head if with_head else 0) + extra
        byt = params * elt + 2 * layers * cfg.kv_dim * elt * (B * ctx + rows) + rows * h * 4
        return np.array([byt, 2.0 * rows * params + 4.0 * layers * cfg.q_dim * ctx * rows])

    total = np.zeros(2)
    if kind == "prefill":
        body = case["ctx"] - 1
        for o in range(0, body, 64):
            m = min(64, body - o)
            total += forward(B * m, cfg.n_layers, o, False) + forward(B * m, 1, o, False, 2 * h * h)
        return {"bytes": float(total[0]), "flops": float(total[1])}
    ctx, steps = _mean_context(case), case["steps"]
    if kind == "decode":
        total = steps * forward(B, cfg.n_layers, ctx, True)
    else:
        K, D, N = case["topk"], case["depth"], case["nodes"]
        total = forward(B * N, cfg.n_layers, ctx, True) + forward(B * 3, 1, ctx, kind != "ngram", 2 * h * h)
        if kind != "ngram":
            for _ in range(1, D):
                total += forward(B * K, 1, ctx, True, 2 * h * h)
        if kind == "sampled":   # target logits and draft distributions of the visited nodes, read once by the acceptance
            total[0] += 2 * 4.0 * B * (D + 1) * V
        total *= steps
    return {"bytes": float(total[0]), "flops": float(total[1])}


def tolerance(case):
    # bf16: the same pass with the other attention kernel (wave per row, fp32 throughout) moves the emitted tokens' hidden
    # states by 5.5e-3 (28 blocks) to 7.9e-3 (the wide model) and the caches of a prefill by 4.5e-3, largest element 0.02-0.06
    # of the root mean square; the output projection rounded to bf16 moves them as far.  No token and no length moves.
    if case["model"] == "tiny":
        return {"rel": 2e-5, "max": 2e-4}
    return {"rel": 2.5e-2, "max": 0.2}
