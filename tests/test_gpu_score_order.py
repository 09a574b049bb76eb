"""The order in which a score adds the weights of its rows: lanes 16, 8, 4, 2 and 1 apart (rows of a tile lie in consecutive lanes),
in every form of the reduction.  A row scored alone gives its weights; added on the host in f32 in that order they are the same bits.
Which of two nearly equal states stays depends on these."""

import numpy as np
import pytest
import torch

import paper_2406_12018_amd as api

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dtype, head_dim, rows", [("bf16", 64, 32), ("bf16", 128, 32), ("f32", 64, 16), ("f32", 128, 16)])
def test_rows_are_added_in_one_order(dtype, head_dim, rows):
    print(f"score order {dtype, head_dim, rows}", flush=True)
    n, dt = 300, torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cpu").manual_seed(8)
    mk = lambda *shape: torch.randn(shape, generator=g).to(dt).to(DEV)
    q, k = mk(1, 1, 2, rows, head_dim), mk(1, 1, 2, n, head_dim)

    def score(q):
        cfg = api.Config(batch=1, layers=1, q_heads=2, kv_heads=2, head_dim=head_dim, chunk_len=n, budget=1, instr_len=q.shape[3],
                         dtype=api.F32 if dtype == "f32" else api.BF16)
        return api.citrus_instr_score(cfg, q, None, 0, k, workspace=api.alloc_workspace(cfg))[0, 0].cpu().numpy()

    sums = np.stack([score(q[:, :, :, r:r + 1].contiguous()) for r in range(rows)])
    apart = rows // 2
    while apart:
        sums = sums + sums[np.arange(rows) ^ apart]
        apart //= 2
    assert sums.dtype == np.float32 and np.array_equal(score(q), sums[0])
