"""The few-row kernels at the edges of their tiles: fp32 products (16 weight rows x 16, 32 or 64 activation rows per
workgroup, K in pieces of 16 dealt over four waves) and the paths of the decoder block that use them."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2511_16665_amd import binding as tlt
from synth import TINY

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


@pytest.mark.parametrize("n,ctxs,mlp", [
    (1, [0, 600], 84),          # one row; key tiles of a wave before and after the first round; a ragged MLP width
    (16, [63, 64, 257], 20),    # 48 rows
    (64, [1, 300, 5, 2, 9], 768),   # 320 rows: the tiled kernel and the separate gate, up and SiLU
])
def test_fp32_forward(n, ctxs, mlp):
    cfg = dataclasses.replace(TINY, name=f"tiny-mlp{mlp}", mlp=mlp)
    _verify_matches_oracle(cfg, "fp32", 1e-4, n, ctxs, 0.05, -1)
