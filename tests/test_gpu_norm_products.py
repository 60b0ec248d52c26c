"""fp32 mode with few rows, whose products normalise their own rows, against more rows of the same sequences (norms of their own); and the
report that a step ends with."""
import ctypes
import dataclasses

import numpy as np
import pytest
import torch

from paper_2511_16665_amd import binding as tlt
from synth import TINY

from gpu_util import make_engine, make_models

pytestmark = pytest.mark.gpu


# rows: 16 and 12 (the last counts that are normalised in the products, up to 256 elements and above), 1, 5; widths at the limit, off the
# wave's 256 and 16, smaller than a wave's step
@pytest.mark.parametrize("hidden,mlp,vocab,B,n", [(256, 768, 1024, 2, 8), (1024, 512, 8192, 1, 16), (1020, 200, 300, 1, 5), (64, 36, 64, 1, 1),
                                                  (1024, 512, 8192, 3, 4), (260, 100, 300, 2, 6), (252, 100, 300, 3, 5)])
def test_products_that_normalise_their_rows(hidden, mlp, vocab, B, n):
    cfg = dataclasses.replace(TINY, hidden=hidden, mlp=mlp, vocab=vocab)
    tw, dw, _, _ = make_models(cfg, 7, "fp32", std=0.05)
    many = 17 // n + 1                                     # sequences of the other run: more than 16 rows
    lens = np.arange(3, 3 + many).astype(np.int32) * 5
    g = torch.Generator().manual_seed(1)
    token = torch.randint(0, vocab, (many, n), generator=g, dtype=torch.int32).cuda()
    out = []
    for count in (B, many):
        e, _, _ = make_engine(cfg, "fp32", tw, dw, many, max(n, 2), 2, 2, 128, seed=3, seq_len=lens)
        for pool in (e.kv.k_pool, e.kv.v_pool):
            pool.normal_(generator=torch.Generator(device="cuda").manual_seed(2))
        t = e.tree(n)
        t.token.copy_(token)
        t.parent.copy_(torch.arange(-1, n - 1, dtype=torch.int32, device="cuda").expand(many, n))
        e.ctx.tree_finalize(many, t)
        logits, hid = torch.zeros((many, n, vocab), device="cuda"), torch.zeros((many, n, hidden), device="cuda")
        print(f"verify hidden {hidden} rows {count * n}", flush=True)
        e.ctx.verify_forward(count, t, e.kv, out_logits=logits, out_hidden=hid)
        torch.cuda.synchronize()
        out.append((logits[:B].clone(), hid[:B].clone()))
    for a, b in zip(*out):
        # two orders of fp32 sums of up to 1024 products, through two blocks: a few 2^-24 of the largest value each
        assert float((a - b).abs().max()) <= 2.0 ** -18 * float(b.abs().max())


def test_step_report_returns_the_words_and_raises_what_kernels_saw():
    cfg = TINY
    tw, dw, _, _ = make_models(cfg, 7, "fp32", std=0.05)
    e, _, _ = make_engine(cfg, "fp32", tw, dw, 3, 8, 2, 2, 200, seed=3)
    words = torch.arange(1000, dtype=torch.int32, device="cuda") * 7 - 5
    pinned = torch.empty(1001, dtype=torch.int32, pin_memory=True)
    np.testing.assert_array_equal(e.ctx.step_report(words, pinned), words.cpu().numpy())
    np.testing.assert_array_equal(e.ctx.step_report(words[:1], pinned), [-5])
    bf = dataclasses.replace(TINY, head_dim=128)           # the MFMA attention checks the lengths against the caller's bound
    tw, dw, _, _ = make_models(bf, 7, "bf16", std=0.05)
    e, _, _ = make_engine(bf, "bf16", tw, dw, 2, 8, 2, 2, 200, seed=3, seq_len=np.array([40, 100], np.int32))
    t = e.tree(1)
    t.parent.fill_(-1)
    e.ctx.tree_finalize(2, t)
    am = e._buf("am", 1)
    e.kv.seq_len_bound = 50
    e.ctx.verify_forward(2, t, e.kv, out_argmax=am)
    with pytest.raises(tlt.TltError):
        e.ctx.step_report(am.view(-1), torch.empty(3, dtype=torch.int32, pin_memory=True))
    e.kv.seq_len_bound = 100                               # (raised once, then cleared)
    e.ctx.verify_forward(2, t, e.kv, out_argmax=am)
    pinned = torch.empty(3, dtype=torch.int32, pin_memory=True)
    np.testing.assert_array_equal(e.ctx.step_report(am.view(-1), pinned), am.view(-1).cpu().numpy())


def test_step_report_refuses_memory_that_kernels_cannot_reach():
    tw, dw, _, _ = make_models(TINY, 7, "fp32", std=0.05)
    e, _, _ = make_engine(TINY, "fp32", tw, dw, 3, 8, 2, 2, 200, seed=3)
    words = torch.arange(64, dtype=torch.int32, device="cuda")
    pageable, pinned = np.full(80, -9, np.int32), torch.full((80,), -9, dtype=torch.int32, pin_memory=True)
    stream, flags = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), ctypes.c_uint32(77)
    report = lambda out, n: e.ctx.lib.tlt_step_report(e.ctx.handle, stream, words.data_ptr(), n, ctypes.c_void_p(out), ctypes.byref(flags))
    for out in (pageable.ctypes.data, words.data_ptr()):            # ordinary host memory, device memory: refused on the host
        assert report(out, 64) == -1 and flags.value == 77
    torch.cuda.synchronize()                                         # (and no error is left behind)
    assert (pageable == -9).all() and words.tolist() == list(range(64))
    assert report(pinned.data_ptr() + 16, 64) == 0 and flags.value == 0   # from inside a pinned allocation
    assert pinned[4:69].tolist() == list(range(64)) + [0] and pinned[:4].tolist() == [-9] * 4 and (pinned[69:] == -9).all()
