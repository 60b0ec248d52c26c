"""Products of 33 to 256 activation rows at the edges of their tiles: 32 rows per wave, two to eight waves, tiles of every width, cuts along K."""
import pytest
import torch

from paper_2511_16665_amd import binding as tlt

pytestmark = pytest.mark.gpu


FOUR_SUMS = [(33, 8192, 64), (64, 640, 1024), (63, 8320, 1024), (96, 16384, 512), (96, 18944, 2560), (72, 24576, 2560)]   # of the cases below: not in one chain


@pytest.mark.parametrize("M,N,K", [
    (33, 8192, 64), (64, 640, 1024), (65, 8192, 1024), (128, 128, 1088),        # two blocks of 16 columns; one K step, fewer than the ring has slots
    (63, 8320, 1024), (97, 12288, 1088), (129, 8320, 512), (256, 12288, 576),   # three: partial and whole last tiles
    (40, 12416, 1024), (96, 16384, 512), (161, 16384, 640), (225, 12416, 512),  # four
    (34, 20480, 64), (66, 16512, 128), (160, 16512, 64), (193, 18944, 320),     # five
    (224, 20480, 192), (65, 20608, 64), (192, 24576, 128), (224, 20608, 448),   # five, six
    (64, 24704, 64), (127, 28672, 192), (130, 24704, 128), (192, 28672, 64),    # seven
    (257, 16512, 128), (225, 16512, 128), (193, 28672, 64), (32, 16512, 64),    # beside the ranges
    (66, 12288, 1088), (161, 11008, 576), (200, 12288, 576), (130, 16384, 576), (224, 13824, 576), (96, 18944, 2560),   # with these every pair of waves and blocks
    (66, 18944, 64), (192, 18944, 192), (64, 24576, 64), (96, 24576, 64), (72, 24576, 2560), (150, 22016, 128),
    (96, 27648, 192),
])
def test_bf16_gate_up(M, N, K):
    """The same bits as the first rows of a product of 300 rows (one chain over K in all tiles), but for long K up to 128 rows and for 32 rows, which
    take four sums and round differently."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn((300, K), generator=g, device="cuda").bfloat16()
    W, U = ((torch.randn((N, K), generator=g, device="cuda") / K ** 0.5).bfloat16() for _ in range(2))
    act = torch.full((M + 1, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    want = torch.empty((300, N), dtype=torch.bfloat16, device="cuda")
    print(f"gate/up M={M} N={N} K={K} and 300 rows", flush=True)
    assert tlt.gemm_glu(A[:M].contiguous(), W, U, act) == 0
    assert tlt.gemm_glu(A, W, U, want) == 0
    torch.cuda.synchronize()
    assert bool(torch.isnan(act[M]).all())   # nothing behind the last row
    if M > 32 and (M, N, K) not in FOUR_SUMS:
        assert torch.equal(act[:M], want[:M])
    else:   # sums of K products in fp32 in another order (2^-24 each), one rounding to bf16 (2^-8) of either result
        gate, up = (A[:M].double() @ x.double().T for x in (W, U))
        err = (K + 2) * 2.0 ** -24 * (A[:M].double().abs() @ (W.double().abs() + U.double().abs()).T) * (1.1 * up.abs() + gate.abs() + 1)
        assert bool(((act[:M].double() - want[:M].double()).abs() <= 2 * err + 2.0 ** -7 * want[:M].double().abs() + 1e-30).all())


@pytest.mark.parametrize("M,N,K", [
    (32, 8192, 1024),                                                  # the kernel of up to 32 rows: a sum per wave
    (33, 640, 512), (64, 8192, 2048),                                  # two blocks of 16 columns
    (48, 11008, 2048), (72, 13824, 1536), (66, 16384, 512), (128, 16384, 2560),   # three, four
    (33, 18944, 1024), (64, 18944, 3584), (96, 18944, 2560), (128, 18944, 3584), (64, 24576, 1536), (72, 24576, 2560), (100, 20608, 3008),   # five, six
    (64, 27648, 2560),                                                 # seven
])
def test_bf16_gate_up_sums_long_k_in_four(M, N, K):
    """The error of a gate/up product's fp32 sums, laid open: the gate is 32 exactly, which SiLU leaves as it is, and three blocks of identity columns take the
    up sum's value, rounded to 24 bits, off again, so the bf16 result is the error to three digits.  A chain of n additions of random terms errs by
    n / sqrt(2) roundings of a term's size, four of n / 4 each by half of that; the identity columns, which add nothing, take up to a third of K from the
    last quarters, which leaves 0.59 at most: below 0.7 of the same rows among 300, which run in one chain."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    Kx = (3 * M + 64) // 64 * 64                       # (at least one column more)
    A = torch.zeros((300, K + Kx), dtype=torch.bfloat16, device="cuda")
    A[:, :K] = torch.randn((300, K), generator=g, device="cuda")
    U, W = (torch.zeros((N, K + Kx), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    U[:, :K] = torch.randn((N, K), generator=g, device="cuda") / K ** 0.5
    A[:, -1], W[:, -1] = 1, 32
    rest = A[:M, :K].double() @ U[:, :K].double().T    # [M, N]
    for i in range(3):
        A[:M, K + i * M: K + (i + 1) * M] = torch.eye(M, device="cuda")
        U[:, K + i * M: K + (i + 1) * M] = -rest.T.float().bfloat16()
        rest += U[:, K + i * M: K + (i + 1) * M].double().T
    act, many = (torch.empty((m, N), dtype=torch.bfloat16, device="cuda") for m in (M, 300))
    print(f"gate/up sums M={M} N={N} K={K} and 300 rows", flush=True)
    assert tlt.gemm_glu(A[:M].contiguous(), W, U, act) == 0
    assert tlt.gemm_glu(A, W, U, many) == 0
    err, one = ((x[:M].double() / 32 - rest).pow(2).mean().sqrt().item() for x in (act, many))
    print(f"  error {err:.3e}, in one chain {one:.3e}: {err / one:.3f}", flush=True)
    assert err <= 0.7 * one


@pytest.mark.parametrize("M,N,K", [
    (33, 3584, 1536), (64, 4608, 2048), (65, 2560, 2112), (96, 3584, 3584), (97, 7168, 1024), (128, 4096, 4096), (127, 8192, 2048),   # 64 columns, even and uneven cuts
    (40, 1536, 4096), (128, 2048, 3072),                                                                                              # ... ten and eight of them
    (129, 5120, 8192), (160, 10240, 1536), (161, 8192, 5120), (192, 14336, 2048), (193, 6144, 3584), (224, 3584, 8192),               # 128 columns
    (225, 5120, 8192), (256, 10240, 2048),
    (80, 8192, 4096), (225, 3584, 18944), (129, 3584, 3584), (72, 14336, 1024),                                                       # beside the ranges
])
def test_bf16_parts(M, N, K):
    """The slices' sum against float64, bounded by one rounding of 2^-24 per product and slice; nothing behind the slices, the same bits again."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn((M, K), generator=g, device="cuda").bfloat16()
    W = (torch.randn((N, K), generator=g, device="cuda") / K ** 0.5).bfloat16()
    buf = torch.full((13 * M * N,), float("nan"), device="cuda")
    print(f"slices M={M} N={N} K={K}", flush=True)
    parts = tlt.gemm_parts(A, W, buf[:12 * M * N])
    torch.cuda.synchronize()
    n = parts.shape[0]
    assert 1 <= n <= 12 and bool(torch.isnan(buf[n * M * N:]).all())
    got = parts.double().sum(0)
    err = (K + 2) * 2.0 ** -24 * (A.double().abs() @ W.double().abs().T)
    assert bool(((got - A.double() @ W.double().T).abs() <= err).all())
    again = tlt.gemm_parts(A, W, torch.empty_like(buf))
    assert torch.equal(parts, again)


@pytest.mark.parametrize("M,N,K,slices,chains", [
    (33, 3584, 1536, 4, 4), (64, 4608, 2048, 3, 4), (65, 2560, 2112, 5, 4), (96, 3584, 3584, 4, 4), (97, 7168, 1024, 2, 4), (128, 4096, 4096, 4, 4),
    (127, 8192, 2048, 2, 4), (40, 1536, 4096, 10, 4), (128, 2048, 3072, 8, 4),
    (129, 5120, 8192, 6, 2), (160, 10240, 1536, 3, 2), (161, 8192, 5120, 4, 2), (192, 14336, 2048, 2, 2), (193, 6144, 3584, 5, 2), (224, 3584, 8192, 9, 2),
    (225, 5120, 8192, 6, 2), (256, 10240, 2048, 3, 2),
    (80, 8192, 4096, 4, 1), (225, 3584, 18944, 9, 1), (129, 3584, 3584, 4, 1), (72, 14336, 1024, 2, 1),          # beside the ranges: the tiled kernel's cuts, in one chain each
])
def test_bf16_parts_cuts_and_their_error(M, N, K, slices, chains):
    """How many slices, and their error to float64 in the root of the mean square, against that of a random walk.  A chain of m matrix instructions of 16
    products, m = K / 16 / (slices * chains), rounds its partial sum twice in each; a rounding errs by 0.43 * 2^-24 of the value in the mean (uniform within half a
    unit, mantissas spread over their logarithm), and the squares of the growing sums are m / 2 of a result's for all chains of an element together.
    The chains of a slice meet in at most as many additions; the slices are added in float64 here.  0.5 for 0.43: one chain in the place of several is outside."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn((M, K), generator=g, device="cuda").bfloat16()
    W = (torch.randn((N, K), generator=g, device="cuda") / K ** 0.5).bfloat16()
    print(f"slices M={M} N={N} K={K}", flush=True)
    parts = tlt.gemm_parts(A, W, torch.empty(12 * M * N, device="cuda"))
    want = A.double() @ W.double().T
    err, bound = float((parts.double().sum(0) - want).norm() / want.norm()), 0.5 * 2.0 ** -24 * (K / 16 / (slices * chains) + chains) ** 0.5
    print(f"  {parts.shape[0]} slices, error {err:.2e}, bound {bound:.2e}", flush=True)
    assert parts.shape[0] == slices and err <= bound


@pytest.mark.parametrize("M,N,K", [
    (33, 65792, 2048), (65, 81920, 192), (128, 81920, 128), (96, 82176, 64), (100, 90112, 320), (128, 90112, 512),   # 64 and 96 columns, partial last tiles
    (97, 90368, 64),                                                                                                # beside the range
])
def test_bf16_whole_rounds_and_rest(M, N, K):
    """The same bits as the first rows of a product of 300 rows (all tiles add up K in one order), nothing behind the last row."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn((300, K), generator=g, device="cuda").bfloat16()
    W = (torch.randn((N, K), generator=g, device="cuda") / K ** 0.5).bfloat16()
    out = torch.full((M + 1, N), float("nan"), device="cuda")
    want = torch.empty((300, N), device="cuda")
    print(f"stored M={M} N={N} K={K} and 300 rows", flush=True)
    tlt.gemm(tlt.TLT_BF16, 1, A[:M].contiguous(), W, out[:M])
    tlt.gemm(tlt.TLT_BF16, 1, A, W, want)
    torch.cuda.synchronize()
    assert bool(torch.isnan(out[M]).all()) and torch.equal(out[:M], want[:M])
