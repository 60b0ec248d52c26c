"""The few-row kernels at the edges of their tiles: fp32 products (16 weight rows x 16, 32 or 64 activation rows per
workgroup, K in pieces of 16 dealt over four waves), bf16 gate/up products (tiles of 32 to 112 columns, K steps through a
ring of slots; from 33 rows on a wave per 32 rows), bf16 products kept as partial sums, and the paths of the decoder block that use them."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2511_16665_amd import binding as tlt
from synth import MID, TINY

from test_gpu_verify import test_verify_forward_matches_oracle as _verify_matches_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("out_mode", [1, 2])
@pytest.mark.parametrize("M,N,K", [
    (1, 1, 4), (1, 15, 12), (16, 16, 16), (17, 33, 60),       # one wave's piece, partial pieces, partial tiles
    (16, 1000, 68), (33, 256, 768), (32, 9000, 64),           # 16 rows per workgroup; 32 rows per workgroup
    (63, 9001, 132), (256, 9008, 64),                         # 64 rows per workgroup, ragged rows and columns
    (257, 48, 64), (8, 48, 66),                               # past the row limit, K not a multiple of 4: the tiled kernel
])
def test_fp32_product(M, N, K, out_mode):
    g = torch.Generator().manual_seed(M * 7 + K)
    A, W, C0 = (torch.randn(s, generator=g) for s in ((M, K), (N, K), (M, N)))
    want = A.double() @ W.double().T + (C0.double() if out_mode == 2 else 0)
    # a sum of K products and at most one addend in fp32, in any order
    bound = (K + 2) * 2.0 ** -24 * (A.double().abs() @ W.double().abs().T + C0.double().abs())
    out = C0.clone().cuda()
    print(f"fp32 product M={M} N={N} K={K} out_mode={out_mode}", flush=True)
    tlt.gemm(tlt.TLT_F32, out_mode, A.cuda(), W.cuda(), out)
    torch.cuda.synchronize()
    assert bool(((out.cpu().double() - want).abs() <= bound).all())


@pytest.mark.parametrize("M,N,K", [
    (97, 48000, 256), (193, 24000, 132),    # 1500 tiles of 64x64, the fewest that go there
    (33, 32768, 64), (160, 10881, 64),      # K of 64: 512 and 513 of them
])
def test_fp32_wide_product_takes_the_tiled_kernel(M, N, K):
    """Where the 64x64 tiles are the faster ones: the same bits as from operands that are not 16-byte aligned, which the few-row
    kernel never takes (it adds up K in another order)."""
    g = torch.Generator(device="cuda").manual_seed(M + K)
    A, W = (torch.randn(s, generator=g, device="cuda") for s in ((M, K), (N, K)))
    shifted = torch.empty(M * K + 1, device="cuda")[1:].view(M, K)
    shifted.copy_(A)
    out, want = (torch.empty((M, N), device="cuda") for _ in range(2))
    print(f"wide fp32 product M={M} N={N} K={K}", flush=True)
    tlt.gemm(tlt.TLT_F32, 1, A, W, out)
    tlt.gemm(tlt.TLT_F32, 1, shifted, W, want)
    torch.cuda.synchronize()
    assert torch.equal(out, want)


@pytest.mark.parametrize("n,ctxs,mlp", [
    (1, [0, 600], 84),          # one row; key tiles of a wave before and after the first round; a ragged MLP width
    (16, [63, 64, 257], 20),    # 48 rows
    (64, [1, 300, 5, 2, 9], 768),   # 320 rows: the tiled kernel and the separate gate, up and SiLU
])
def test_fp32_forward(n, ctxs, mlp):
    cfg = dataclasses.replace(TINY, name=f"tiny-mlp{mlp}", mlp=mlp)
    _verify_matches_oracle(cfg, "fp32", 1e-4, n, ctxs, 0.05, -1)


@pytest.mark.parametrize("M,N,K", [
    (1, 640, 256), (32, 8192, 64),              # 32 columns per workgroup; one K step, fewer than the ring has slots
    (17, 8320, 192), (33, 12288, 1088),         # 48 columns, partial last tile; K steps past one turn of the ring
    (32, 16512, 64), (64, 20480, 1024),         # 80 columns
    (5, 20608, 128), (40, 24576, 1024),         # 96 columns
    (31, 24704, 512), (64, 28672, 2560),        # 112 columns
    (65, 12416, 512), (128, 16384, 576),        # above 64 rows: three and four waves, 64 columns
    (97, 16512, 2560), (128, 20608, 2624),      # 80 and 96 columns, partial last tiles
    (33, 12288, 576), (64, 20480, 448), (40, 24576, 64), (31, 24704, 128), (64, 28672, 192),   # K too short for four sums: one chain, in the tiled
    (65, 12416, 384), (128, 16384, 64), (97, 16512, 320), (128, 20608, 128),                   # kernel or with a wave per 32 rows
    (64, 14336, 128), (66, 640, 128), (100, 24704, 64),       # beside the ranges: one chain
    (129, 16512, 64),                                         # five waves, the last one with a row
    (200, 12800, 448), (256, 20480, 192),                     # 256 rows x 80 columns, gate and up rows in turns of 16
    (250, 20608, 192),                                        # one more column tile: 256x256 tiles
])
def test_bf16_gate_up(M, N, K):
    g = torch.Generator().manual_seed(M + N + K)
    A = torch.randn((M, K), generator=g).bfloat16()
    W, U = ((torch.randn((N, K), generator=g) / K ** 0.5).bfloat16() for _ in range(2))
    act = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    print(f"gate/up M={M} N={N} K={K}", flush=True)
    tlt.gemm_glu(A.cuda(), W.cuda(), U.cuda(), act)
    torch.cuda.synchronize()
    Ad, Wd, Ud = A.cuda().double(), W.cuda().double(), U.cuda().double()
    gate, up = Ad @ Wd.T, Ad @ Ud.T
    want = torch.nn.functional.silu(gate) * up
    # fp32 sums of K products each, |silu'| < 1.1; exponential and reciprocal to a few units of 2^-23; one rounding to bf16
    sum_err = (K + 2) * 2.0 ** -24
    bound = (1.1 * sum_err * (Ad.abs() @ Wd.abs().T) * up.abs() + torch.nn.functional.silu(gate).abs() * sum_err * (Ad.abs() @ Ud.abs().T)
             + want.abs() * (2.0 ** -8 + (8 + gate.abs()) * 2.0 ** -22) + 1e-30)
    assert bool(((act.double() - want).abs() <= bound).all())


@pytest.mark.parametrize("M,N,K", [(33, 8320, 960), (64, 24576, 960), (32, 28672, 448), (64, 28672, 2496), (65, 13824, 448), (128, 18944, 2496)])
def test_bf16_gate_up_with_short_k_takes_one_chain(M, N, K):
    """One K step less than four sums over K ask for: the same bits as the first rows of a product of 300 rows (one chain over K, in the tiled kernels and
    with a wave per 32 rows)."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn((300, K), generator=g, device="cuda").bfloat16()
    W, U = ((torch.randn((N, K), generator=g, device="cuda") / K ** 0.5).bfloat16() for _ in range(2))
    act, want = (torch.empty((m, N), dtype=torch.bfloat16, device="cuda") for m in (M, 300))
    print(f"gate/up M={M} N={N} K={K} and 300 rows", flush=True)
    assert tlt.gemm_glu(A[:M].contiguous(), W, U, act) == 0
    assert tlt.gemm_glu(A, W, U, want) == 0
    torch.cuda.synchronize()
    assert torch.equal(act, want[:M])


@pytest.mark.parametrize("M,N,K,room,slices", [
    (1, 640, 1280, 12, 3), (17, 640, 1280, 2, 2),     # 64-column tiles, 20 K steps in three cuts; room for two slices only
    (32, 512, 8256, 12, 12),                          # the most cuts, 129 K steps
    (17, 14336, 1088, 12, 1),                         # no cut
    (31, 10240, 2624, 12, 2),                         # 96-column tiles, the last one partial, 41 K steps
    (32, 9216, 2624, 12, 3),                          # 128-column tiles
    (5, 512, 256, 12, 1),                             # K too short to cut: the general plan
    (16, 4096, 8192, 12, 8), (32, 10240, 8192, 12, 3), (1, 8192, 4096, 12, 4),   # cuts an odd multiple of 2048 apart: the general plan
    (1, 18432, 5184, 12, 7),                          # the general plan has more than four times the cuts
])
def test_bf16_partial_products(M, N, K, room, slices):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn((M, K), generator=g, device="cuda").bfloat16()
    W = (torch.randn((N, K), generator=g, device="cuda") / K ** 0.5).bfloat16()
    buf = torch.full((room * M * N,), float("nan"), device="cuda")
    print(f"partial products M={M} N={N} K={K}", flush=True)
    parts = tlt.gemm_parts(A, W, buf)
    torch.cuda.synchronize()
    assert parts.shape[0] == slices
    assert bool(torch.isnan(buf[parts.numel():]).all())   # nothing behind the last slice
    Ad, Wd = A.double(), W.double()
    # K products of bf16 values, exact in fp32, and their sums in fp32, in any order (the slices are added up in float64 here)
    bound = K * 2.0 ** -24 * (Ad.abs() @ Wd.abs().T)
    assert bool(((parts.double().sum(0) - Ad @ Wd.T).abs() <= bound).all())


@pytest.mark.parametrize("hidden,heads,n", [
    (512, 4, 5),       # 64 columns per workgroup, one cut
    (6144, 8, 32),     # output projection in two cuts, down in 96-column tiles
    (8704, 68, 9),     # output projection in 128-column tiles
])
def test_bf16_forward_few_rows(hidden, heads, n):
    cfg = dataclasses.replace(MID, name=f"mid-h{hidden}", hidden=hidden, n_q_heads=heads, n_kv_heads=4, mlp=3072, vocab=512, n_layers=1)
    _verify_matches_oracle(cfg, "bf16", 2e-2, n, [70], 0.02, -1)


def test_bf16_forward_of_576_rows_of_4608_elements():
    """More than 512 rows wider than 4096: the norms with 256 threads."""
    cfg = dataclasses.replace(MID, name="mid-h4608", hidden=4608, n_q_heads=36, n_kv_heads=4, mlp=1024, vocab=256, n_layers=1)
    _verify_matches_oracle(cfg, "bf16", 2e-2, 64, [3, 70, 0, 1, 16, 5, 9, 33, 2], 0.02, -1)


@pytest.mark.parametrize("dtype,d", [("fp32", 64), ("fp32", 192), ("fp32", 256), ("bf16", 64), ("bf16", 192)])
def test_row_attention_head_dims(dtype, d):
    """Value rows spread over the lanes: 4, 1 (with idle lanes), 1, 8 and 2 rows (with idle lanes) at a time."""
    cfg = dataclasses.replace(TINY, name=f"tiny-d{d}", head_dim=d, hidden=512, mlp=768)
    _verify_matches_oracle(cfg, dtype, 1e-4 if dtype == "fp32" else 2e-2, 7, [0, 61, 65, 330], 0.05, 0)
