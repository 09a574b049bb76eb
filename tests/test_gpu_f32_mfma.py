"""The f32 kernels at the edges of their tiles (sixteen rows, sixteen keys per wave, eight waves), on both sides of the
single-launch score, and with values that are not finite where some rows do not see them; against f64.

Tolerance of the mode: 1e-5.  Logits are exact to f64; a probability keeps the rounding of its f32 argument, 2^-24 of |s - max| in
the exponent, and of f32 sums."""

import dataclasses

import pytest
import torch

import paper_2406_12018_amd as api

pytestmark = pytest.mark.gpu
DEV = "cuda"

# layers, query heads, KV heads, chunk, cache, instruction rows
CASES = [
    (1, 1, 1, 1, 0, 1),
    (1, 2, 1, 16, 0, 16),
    (1, 4, 2, 17, 15, 16),      # 32 rows of a group: the last of the single-launch score at head_dim 128
    (1, 4, 2, 15, 112, 17),     # 34: two launches at 128
    (2, 4, 1, 33, 96, 16),      # 64 rows: the last at 64; 129 keys, a second tile for one wave
    (1, 4, 1, 1, 511, 17),      # 512 keys, 68 rows
    (1, 2, 2, 64, 449, 5),      # 513 keys
    (1, 3, 3, 31, 700, 40),
    # from 512 workgroups of sixteen rows on: fewer waves, by the number of keys, and more of them at 1024, 2048 and 4096
    (16, 32, 8, 1, 30, 2), (16, 32, 8, 1, 32, 2), (16, 16, 4, 17, 200, 3), (16, 32, 8, 1, 14, 2), (16, 32, 8, 1, 16, 2),
    (32, 32, 8, 1, 127, 2), (32, 32, 8, 1, 130, 2), (64, 16, 16, 20, 33, 1), (64, 32, 16, 33, 40, 1),
]


def reference(q, keys, values, n_c, qi):
    """Outputs, log-sum-exps, instruction scores in f64."""
    group, c, d = q.shape[2] // keys.shape[2], q.shape[3], q.shape[4]
    k, v = (x.double().repeat_interleave(group, dim=2) for x in (keys, values))
    s = torch.matmul(q.double(), k.transpose(-1, -2).contiguous()) / d ** 0.5
    hidden = torch.arange(k.shape[3], device=DEV)[None, :] > n_c + torch.arange(c, device=DEV)[:, None]
    s = s.masked_fill(hidden, float("-inf"))
    p = torch.matmul(qi.double(), k.transpose(-1, -2).contiguous()) / d ** 0.5
    score = torch.softmax(p, dim=-1).sum(dim=3).unflatten(2, (keys.shape[2], group)).sum(dim=3)
    return torch.softmax(s, dim=-1), v, torch.logsumexp(s, dim=-1), score


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(x) for x in c))
def test_step_against_f64(case, head_dim):
    L, Hq, Hkv, c, n_c, rows = case
    print(f"f32 step {case} head_dim {head_dim}", flush=True)
    g = torch.Generator(device="cpu").manual_seed(11)
    mk = lambda *shape: torch.randn(shape, generator=g).to(DEV)
    q, qi = mk(1, L, Hq, c, head_dim), mk(1, L, Hq, rows, head_dim)
    kc, vc, k, v = mk(1, L, Hkv, n_c + 1, head_dim), mk(1, L, Hkv, n_c + 1, head_dim), mk(1, L, Hkv, c, head_dim), mk(1, L, Hkv, c, head_dim)
    cfg = api.Config(batch=1, layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=head_dim, chunk_len=c, budget=n_c + 1, instr_len=rows,
                     dtype=api.F32)
    ws = api.alloc_workspace(cfg)
    lse = torch.empty((1, L, Hq, c), device=DEV)
    lm = torch.empty((1, L, Hkv, n_c + c), device=DEV)
    out = api.citrus_chunk_attn(cfg, q, kc, vc, n_c, k, v, lse=lse, lm_score=lm, workspace=ws)
    score = api.citrus_instr_score(cfg, qi, kc, n_c, k, workspace=ws)
    keys, values = torch.cat([kc[:, :, :, :n_c], k], dim=3), torch.cat([vc[:, :, :, :n_c], v], dim=3)
    p, v_all, want_lse, want_score = reference(q, keys, values, n_c, qi)
    close = lambda a, b: torch.testing.assert_close(a.double(), b, rtol=1e-5, atol=1e-5)
    close(out, torch.matmul(p, v_all))
    close(lse, want_lse)
    close(lm, p.sum(dim=3).unflatten(2, (Hkv, Hq // Hkv)).sum(dim=3))
    close(score, want_score)
    # one chunk of a document: attention and score in one launch where they can be, outputs and selection by the same bits
    out_doc = torch.empty_like(out)
    some = dataclasses.replace(cfg, budget=max(1, c // 2), cache_capacity=0)
    state = api.DocumentState.allocate(some)
    api.citrus_process_document(some, state, ws, doc=api.resident_doc(cfg, q, k, v, qi, out_doc))
    assert torch.equal(out_doc, api.citrus_chunk_attn(cfg, q, kc, vc, 0, k, v))
    kept = api.citrus_topk_select(cfg, api.citrus_instr_score(cfg, qi, kc, 0, k, workspace=ws), some.budget)
    rows_of = kept.long()[..., None].expand(-1, -1, -1, -1, head_dim)
    assert torch.equal(state.current()[0], torch.gather(k, 3, rows_of)) and torch.equal(state.current()[1], torch.gather(v, 3, rows_of))
    # a value that is not finite reaches the rows that see its key, and no other
    for bad in (float("inf"), float("nan")):
        v2 = v.clone()
        v2[:, :, :, c // 2, 3] = bad
        got = api.citrus_chunk_attn(cfg, q, kc, vc, n_c, k, v2)
        assert torch.equal(got[:, :, :, :c // 2], out[:, :, :, :c // 2])
        assert not got[:, :, :, c // 2:, 3].isfinite().any()
        others = [x for x in range(head_dim) if x != 3]
        close(got[:, :, :, c // 2:][..., others], torch.matmul(p, v_all)[:, :, :, c // 2:][..., others])


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("n_c,c", [(0, 33), (0, 17), (40, 1), (96, 33), (500, 40)], ids=str)
def test_a_key_that_is_nan_reaches_every_row_that_sees_it(n_c, c, head_dim):
    """The last key is the only one of its tile, and in the smaller cases of its wave: a maximum passes over NaN, the sums must
    not.  A row's softmax over a NaN logit is NaN throughout; the rows in front of the key do not see it."""
    print(f"f32 NaN key {n_c} + {c} head_dim {head_dim}", flush=True)
    g = torch.Generator(device="cpu").manual_seed(3)
    mk = lambda *shape: torch.randn(shape, generator=g).to(DEV)
    q, qi, k, v = mk(1, 1, 4, c, head_dim), mk(1, 1, 4, 8, head_dim), mk(1, 1, 2, c, head_dim), mk(1, 1, 2, c, head_dim)
    kc, vc = mk(1, 1, 2, n_c + 1, head_dim), mk(1, 1, 2, n_c + 1, head_dim)
    k[:, :, :, -1, 5] = float("nan")
    cfg = api.Config(batch=1, layers=1, q_heads=4, kv_heads=2, head_dim=head_dim, chunk_len=c, budget=n_c + 1, instr_len=8, dtype=api.F32)
    ws = api.alloc_workspace(cfg)
    lse = torch.empty((1, 1, 4, c), device=DEV)
    out = api.citrus_chunk_attn(cfg, q, kc, vc, n_c, k, v, lse=lse, workspace=ws)
    assert out[:, :, :, -1].isnan().all() and lse[:, :, :, -1].isnan().all()
    assert out[:, :, :, :-1].isfinite().all() and lse[:, :, :, :-1].isfinite().all()
    assert api.citrus_instr_score(cfg, qi, kc, n_c, k, workspace=ws).isnan().all()
