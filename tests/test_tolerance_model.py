"""Where the bf16-mode tolerance comes from, rounding by rounding.

A bf16 decoder hands bf16 activations from one contraction to the next; the float64 oracle keeps them
exact.  The library rounds the operands of a block's five contractions: the normalised rows entering the q/k/v
projection (xn), the rotated queries (q), the attention output entering the output projection (att),
the normalised rows entering the MLP (xn2) and the gated product silu(gate)*up entering the down
projection (act; gate and up themselves stay fp32 inside the fused kernel); and the q/k/v product in front of
the bias and the rotation (qkv), so queries, keys and (with a bias) values are rounded twice.  Keys and values
as stored are cache state and rounded on both sides.  The residual stream and the output
projection's product stay fp32.

Rounding the ORACLE's own activations at those points, on the CPU, one point at a time and all
together, gives the per-rounding budget: each costs a relative rms error of a few 1e-3 of the
residual stream per block, they add in quadrature within a block, and the blocks' errors add in
quadrature along the stack (about per_block * sqrt(L)).  The GPU parity tests hold stacks of up to
four blocks to the flat 2e-2 and an L-block stack to max(2e-2, 1e-2 * sqrt(L)); this test keeps
those figures honest, with and without the rounding in front of the rotation, and shows what one more (the output
projection's product, which the library can be switched to round for measurements) would add.
"""
import dataclasses

import numpy as np
import torch

from oracle import decoder as dec
from synth import MID, make_decoder_weights

POINTS = ("xn", "q", "att", "xn2", "act")


def _block(cfg, lw, x0, K, V, pos, slots, vis, rounded=()):
    r = lambda name, a: dec.round_to_bf16(a) if name in rounded else a
    n = x0.shape[0]
    xn = r("xn", dec.rmsnorm(x0, lw["attn_norm"], cfg.rms_eps))
    qkv = r("qkv", xn @ lw["wqkv"].T)
    q = qkv[:, : cfg.q_dim].reshape(n, cfg.n_q_heads, cfg.head_dim)
    k = qkv[:, cfg.q_dim: cfg.q_dim + cfg.kv_dim].reshape(n, cfg.n_kv_heads, cfg.head_dim)
    v = qkv[:, cfg.q_dim + cfg.kv_dim:].reshape(n, cfg.n_kv_heads, cfg.head_dim)
    q = r("q", dec.rope(q, pos, cfg.rope_theta))
    Kc, Vc = K.copy(), V.copy()
    Kc[slots] = dec.round_to_bf16(dec.rope(k, pos, cfg.rope_theta))     # the cache is bf16 state on both sides
    Vc[slots] = dec.round_to_bf16(v)
    a = r("att", dec.attention(q, Kc, Vc, vis).reshape(n, cfg.q_dim))
    x = x0 + r("oproj", a @ lw["wo"].T)
    xn2 = r("xn2", dec.rmsnorm(x, lw["mlp_norm"], cfg.rms_eps))
    act = r("act", dec.silu(xn2 @ lw["wg"].T) * (xn2 @ lw["wu"].T))
    return x + act @ lw["wd"].T


def _setup(n_layers=4):
    cfg = dataclasses.replace(MID, n_layers=n_layers)
    tw = dec.weights_to_f64(make_decoder_weights(cfg, 3, device="cpu", dtype=torch.bfloat16))
    rng = np.random.default_rng(0)
    n, c = 24, 200
    x = dec.round_to_bf16(rng.normal(size=(n, cfg.hidden)) * 0.02)
    pos = c + np.arange(n)
    slots = c + np.arange(n)
    vis = np.zeros((n, c + n), bool)
    vis[:, :c] = True
    vis[:, c:] = np.tril(np.ones((n, n), bool))
    caches = [(dec.round_to_bf16(rng.normal(size=(c + n, cfg.n_kv_heads, cfg.head_dim))),
               dec.round_to_bf16(rng.normal(size=(c + n, cfg.n_kv_heads, cfg.head_dim)))) for _ in range(cfg.n_layers)]
    return cfg, tw, x, pos, slots, vis, caches


def _stack_errors(cfg, tw, x, pos, slots, vis, caches, rounded):
    exact, rnd, errs = x, x, []
    for l in range(cfg.n_layers):
        exact = _block(cfg, tw["layers"][l], exact, *caches[l], pos, slots, vis)
        rnd = _block(cfg, tw["layers"][l], rnd, *caches[l], pos, slots, vis, rounded)
        errs.append(np.sqrt(((rnd - exact) ** 2).mean()) / np.sqrt((exact ** 2).mean()))
    return errs, rnd, exact


def test_bf16_activation_rounding_costs_under_1e2_per_block_and_adds_in_quadrature():
    s = _setup()
    cfg = s[0]
    errs, rnd, exact = _stack_errors(*s, rounded=POINTS)
    print("relative rms error after 1..4 blocks, all five roundings:", errs)
    assert 1e-3 < errs[0] < 1e-2                       # one block: well inside 2e-2, not negligible
    assert errs[-1] < 2e-2                             # four blocks still inside the flat tolerance
    assert errs[-1] < 1.5 * errs[0] * np.sqrt(cfg.n_layers)   # no faster than ~sqrt(L)
    assert np.abs(rnd - exact).max() / np.abs(exact).max() < 2e-2


def test_per_rounding_budget_of_one_block():
    """Each of the five roundings alone, one block: a few 1e-3 each, adding in quadrature to the block's
    figure; the output projection's product, were it rounded too, would add one more of the same size."""
    s = _setup(n_layers=1)
    alone = {p: _stack_errors(*s, rounded=(p,))[0][0] for p in POINTS + ("oproj",)}
    together = _stack_errors(*s, rounded=POINTS)[0][0]
    with_oproj = _stack_errors(*s, rounded=POINTS + ("oproj",))[0][0]
    print("one block, relative rms error of the residual stream per rounding:", {k: round(v, 5) for k, v in alone.items()})
    print("all five:", round(together, 5), " quadrature sum:", round(float(np.sqrt(sum(alone[p] ** 2 for p in POINTS))), 5),
          " with the output projection rounded as well:", round(with_oproj, 5))
    for p in POINTS:
        assert 2e-4 < alone[p] < 6e-3, (p, alone[p])
    quad = np.sqrt(sum(alone[p] ** 2 for p in POINTS))
    assert 0.7 * quad < together < 1.3 * quad
    # a sixth rounding is not free, and not dominant either
    assert together < with_oproj < 1.5 * together


def test_rounding_in_front_of_the_rotation():
    """The q/k/v product rounded as well: as large alone as the others, in quadrature with them, and four blocks still inside 2e-2."""
    s = _setup(n_layers=4)
    alone = _stack_errors(*s, rounded=("qkv",))[0]
    five, six = (_stack_errors(*s, rounded=p)[0] for p in (POINTS, POINTS + ("qkv",)))
    print("qkv alone, after 1..4 blocks:", alone, " five:", five, " with it:", six)
    assert 2e-4 < alone[0] < 6e-3
    quad = np.sqrt(alone[0] ** 2 + five[0] ** 2)
    assert 0.7 * quad < six[0] < 1.3 * quad and six[0] < 1e-2 and six[-1] < 2e-2
