"""The single-product instruction score at the edges of its instances: strips of 32 and 64 rows with a remainder, key tiles a wave
does not have, caches that end inside a tile, more rows than one head's; against f64.

Tolerance: a logit is a sum of D bf16 products in f32, off by at most D 2^-24 sum |q k|; with normal inputs sum |q k| is about
0.64 D, which times scale and log2 e makes D = 128: 8e-5, D = 64: 3e-5 of a weight, and the sums over rows and keys keep it."""

import pytest
import torch

import paper_2406_12018_amd as api

pytestmark = pytest.mark.gpu
DEV = "cuda"

# layers, query heads, KV heads, rows, cache, chunk; what runs at head dimension 64 and 128: strips or two passes
# (test_dispatch_cpu.py checks that it does)
CASES = [
    (1, 1, 1, 1, 0, 1, "SS"),
    (1, 2, 1, 16, 0, 33, "SS"),        # one strip, one wave with a second tile
    (1, 4, 2, 17, 31, 226, "SS"),      # 68 rows; 257 keys; a cache that ends inside a tile
    (1, 4, 1, 8, 1000, 280, "SS"),     # 1280 keys
    (1, 4, 1, 9, 1000, 281, "SS"),     # 1281: ten tiles per wave
    (1, 8, 2, 64, 2000, 560, "SS"),    # 2560
    (1, 8, 2, 64, 2000, 561, "TT"),
    (5, 32, 8, 51, 300, 213, "SS"),    # 204 rows: 32-row strips no longer fit side by side, 64-row strips with a rest of 12
    (1, 64, 2, 128, 475, 37, "SS"),    # 4096 rows per KV head, 512 keys: as many as the scratch holds
    (1, 64, 2, 128, 476, 37, "TT"),
    (1, 64, 2, 129, 400, 37, "TT"),    # 4128 rows
    (24, 32, 8, 64, 250, 60, "SS"),    # 192 KV heads of four strips of 64
    (25, 32, 8, 64, 250, 60, "ST"),    # 200: one round of the two-pass kernel at head_dim 128
    (32, 32, 8, 49, 100, 61, "ST"),    # 256 of 196 rows
    (40, 8, 8, 40, 100, 50, "TS"),     # one strip per KV head, 320 KV heads
    (16, 32, 8, 32, 1000, 281, "SS"), (17, 32, 8, 32, 1000, 281, "TT"),  # 128 rows, 1281 keys: two strips per compute unit
    (2, 8, 2, 256, 1000, 281, "SS"), (8, 8, 2, 256, 1000, 281, "TS"),    # 1024 rows of four heads
]


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(x) for x in c))
def test_scores_against_f64(case, head_dim):
    L, Hq, Hkv, rows, n_c, c, _ = case
    print(f"strip scores {case} head_dim {head_dim}", flush=True)
    g = torch.Generator(device="cpu").manual_seed(5)
    mk = lambda *shape: torch.randn(shape, generator=g).to(torch.bfloat16).to(DEV)
    q, kc, k = mk(1, L, Hq, rows, head_dim), mk(1, L, Hkv, n_c + 3, head_dim), mk(1, L, Hkv, c, head_dim)
    cfg = api.Config(batch=1, layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=head_dim, chunk_len=c, budget=n_c + 3, instr_len=rows)
    ws = api.alloc_workspace(cfg)
    score = api.citrus_instr_score(cfg, q, kc, n_c, k, workspace=ws)
    assert torch.equal(score, api.citrus_instr_score(cfg, q, kc, n_c, k, workspace=ws))
    keys = torch.cat([kc[:, :, :, :n_c], k], dim=3).double()
    qs = q.double().reshape(1, L, Hkv, Hq // Hkv * rows, head_dim)
    want = torch.softmax(torch.matmul(qs, keys.transpose(-1, -2).contiguous()) / head_dim ** 0.5, dim=-1).sum(dim=-2)
    torch.testing.assert_close(score.double(), want, rtol=8e-5 if head_dim == 128 else 3e-5, atol=1e-7)


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")], ids=str)
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("rows,n_c,c", [(8, 0, 33), (8, 160, 40), (64, 1200, 70), (16, 0, 1)], ids=str)
def test_logits_that_are_not_finite(rows, n_c, c, head_dim, bad):
    """The last key's logits are not finite; in the first case they are all its wave has.  A row whose logit is NaN or +inf there
    has no weight anywhere that is a number, as a softmax in f64 has it; -inf is a weight of 0 unless there is no other key."""
    print(f"strip scores, last key {bad}, {rows} rows, {n_c} + {c} head_dim {head_dim}", flush=True)
    g = torch.Generator(device="cpu").manual_seed(9)
    mk = lambda *shape: torch.randn(shape, generator=g).to(torch.bfloat16).to(DEV)
    q, kc, k = mk(1, 1, 4, rows, head_dim), mk(1, 1, 2, n_c + 1, head_dim), mk(1, 1, 2, c, head_dim)
    q[..., 3] = q[..., 3].abs() + 0.5  # one sign: the logits are `bad` for every row
    k[:, :, :, -1, 3] = bad
    cfg = api.Config(batch=1, layers=1, q_heads=4, kv_heads=2, head_dim=head_dim, chunk_len=c, budget=n_c + 1, instr_len=rows)
    score = api.citrus_instr_score(cfg, q, kc, n_c, k, workspace=api.alloc_workspace(cfg))
    if bad == float("-inf") and n_c + c > 1:
        assert (score[..., -1] == 0).all() and score.isfinite().all()
        torch.testing.assert_close(score.double().sum(-1), torch.full((1, 1, 2), 2.0 * rows, device=DEV, dtype=torch.double), rtol=1e-5, atol=0)
    else:
        assert score.isnan().all()
