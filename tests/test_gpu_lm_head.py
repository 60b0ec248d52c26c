"""Wide products of up to 256 rows: tiles of 64 rows, launches cut into whole rounds and a rest, K shorter than the load ring."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2511_16665_amd import binding as tlt
from synth import TINY

from gpu_util import make_engine, make_models

pytestmark = pytest.mark.gpu


def _operands(M, N, K, seed, small_ints=False):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if small_ints:   # many equal sums, all exact
        A = torch.randint(-2, 3, (M, K), generator=g, device="cuda").bfloat16()
        W = torch.randint(-1, 2, (N, K), generator=g, device="cuda").bfloat16()
    else:
        A = torch.randn((M, K), generator=g, device="cuda").bfloat16()
        W = (torch.randn((N, K), generator=g, device="cuda") * 0.05).bfloat16()
    return A, W, A.double() @ W.double().t()


@pytest.mark.parametrize("M,N,K,mode", [
    (1, 38400, 192, 1),      # 300 tiles, two workgroups per CU, three K steps = the ring
    (33, 32896, 128, 0),     # 257 tiles, K shorter than the ring: no workgroup takes two
    (64, 384, 64, 0),        # three tiles, one K step in a ring of five
    (63, 32768, 576, 1),     # 256 tiles, one per CU, nine K steps
    (64, 70016, 1024, 1),    # several tiles per workgroup
    (48, 66304, 2048, 1),    # 128-row tiles: a whole round and a rest of three column tiles
    (33, 66304, 2048, 0),
    (200, 102400, 192, 1),   # a rest of 288 tiles whose K is shorter than its ring of weight slots
    (17, 128, 3584, 2),      # accumulating
])
def test_wide_products_of_few_rows(M, N, K, mode):
    A, W, want = _operands(M, N, K, M + N)
    print(f"product M={M} N={N} K={K} mode={mode}", flush=True)
    out = torch.full((M, N), 0.5 if mode == 2 else float("nan"), dtype=torch.float32 if mode else torch.bfloat16, device="cuda")
    tlt.gemm(tlt.TLT_BF16, mode, A, W, out)
    torch.cuda.synchronize()
    if mode == 2:
        want = want + 0.5
    # fp32 sums of K products of bf16 numbers: K * 2^-24 of the sum of magnitudes at most, far below; a bf16 result half a unit of 2^-8
    tol = 2.0 ** -8 if mode == 0 else 2.0 ** -24 * K
    assert float((out.double() - want).abs().max()) <= tol * float(want.abs().max())


@pytest.mark.parametrize("M,N,K,ties", [
    (65, 65792, 256, False), (128, 102400, 192, False), (100, 66304, 256, True), (128, 1024, 256, True),   # 128-row tiles (+ rest)
    (129, 66304, 192, False), (256, 102400, 192, True), (255, 2048, 512, True),                             # 256-row tiles (+ rest)
    (257, 66304, 192, True)])                                                                              # two rows of tiles
def test_row_argmax_over_whole_rounds_and_rest(M, N, K, ties):
    A, W, want = _operands(M, N, K, M + N + 1, ties)
    ws = torch.full((M * (N // 128) * 2 + 64,), float("nan"), dtype=torch.float32, device="cuda")
    out = torch.full((M,), -1, dtype=torch.int32, device="cuda")
    print(f"argmax M={M} N={N} K={K}", flush=True)
    assert tlt.gemm_argmax(A, W, ws[:-64], out) == 0
    torch.cuda.synchronize()
    assert torch.isnan(ws[-64:]).all()
    got, want = out.cpu().numpy(), want.cpu().numpy()
    if ties:
        np.testing.assert_array_equal(got, want.argmax(axis=1))   # the lowest column of the largest sum
    else:
        best = want.max(axis=1)
        assert np.all(want[np.arange(M), got] >= best - 2.0 ** -24 * K * np.abs(want).max())


@pytest.mark.parametrize("V", [63, 2047, 2048, 2049, 4095, 4096, 4097, 4100])   # one kernel up to 2048 logits, or 4096 in 16-byte pieces; two
def test_argmax_of_short_rows(V):
    """The first of the largest logits, with ties, at one row and at several."""
    cfg = dataclasses.replace(TINY, name=f"tiny-v{V}", n_layers=1, hidden=64, mlp=64, vocab=V)
    tw, dw, _, _ = make_models(cfg, 5, "fp32", std=0.2)
    rng = np.random.default_rng(V)
    for j in rng.permutation(V)[: 3 * V // 4]:                      # most rows twice or more
        tw["lm_head"][j] = tw["lm_head"][rng.integers(V)]
    for B, n in ((1, 1), (2, 5), (4, 16), (3, 64)):
        e, _, _ = make_engine(cfg, "fp32", tw, dw, B, 64, 2, 2, 128, seed=3, seq_len=np.full(B, 20, np.int32))
        t = e.tree(n)
        t.parent.copy_(torch.from_numpy(np.tile(np.arange(-1, n - 1, dtype=np.int32), (B, 1))))
        t.token.copy_(torch.from_numpy(rng.integers(V, size=(B, n)).astype(np.int32)))
        e.ctx.tree_finalize(B, t)
        logits, am = torch.empty((B, n, V), device="cuda"), torch.full((B, n), -7, dtype=torch.int32, device="cuda")
        print(f"argmax of short rows V={V} rows={B * n}", flush=True)
        e.ctx.verify_forward(B, t, e.kv, out_logits=logits, out_argmax=am)
        np.testing.assert_array_equal(am.cpu().numpy(), logits.cpu().numpy().argmax(-1))
        e.ctx.close()
