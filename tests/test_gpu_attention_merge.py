"""The merge of the chunks' partial results where rows are many (half a wave per row): row counts off the workgroup's eight, one to many
chunks per sequence, against the attention kernel that has no chunks."""
import numpy as np
import pytest
import torch

from paper_2511_16665_amd import binding as tlt
from synth import fill_kv_pool, random_block_table

from gpu_util import rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,n,Hq,Hkv,longest", [(24, 13, 28, 2, 9000), (3, 64, 28, 4, 20000), (41, 1, 104, 1, 700), (6, 50, 28, 4, 1)])
def test_merge_of_many_rows(B, n, Hq, Hkv, longest):
    d, page = 128, 16
    rng = np.random.default_rng(n)
    ctxs = np.sort(rng.integers(0, longest + 1, B)).astype(np.int32)
    ctxs[0], ctxs[-1] = 0, longest
    table, n_pages = random_block_table(ctxs + n + 8, page, seed=3, extra_pages=3)
    k, v = fill_kv_pool(1, n_pages, Hkv, page, d, seed=9, dtype=torch.bfloat16)
    qkv = torch.randn((B, n, (Hq + 2 * Hkv) * d), generator=torch.Generator().manual_seed(1)).bfloat16().cuda()
    mask = torch.tensor([[((2 << i) - 1) - (1 << 64 if i == 63 else 0) for i in range(n)]] * B, dtype=torch.int64).cuda()
    kv = tlt.KV(k[0].cuda(), v[0].cuda(), torch.from_numpy(table.astype(np.int32)).cuda(), torch.from_numpy(ctxs).cuda(), longest)
    assert n * (Hq // Hkv) * Hkv * B > 4096
    outs = []
    for impl in (0, 1):
        out = torch.full((B, n, Hq * d), 7.0, dtype=torch.bfloat16, device="cuda")
        ws = tlt.attention_workspace(B, n, Hq, Hkv, d, longest + n + 8)
        print(f"attention B={B} n={n} Hq={Hq} Hkv={Hkv} impl={impl}", flush=True)
        assert tlt.attention(tlt.TLT_BF16, Hq, page, qkv, mask, kv, out, ws, impl) == 0
        torch.cuda.synchronize()
        outs.append(out.float().cpu().numpy())
    for b in range(B):
        assert rel_err(outs[1][b], outs[0][b]) <= 2e-2, b
