"""Chunk attention whose blocks mix heads (groups that 4 and 2 do not divide), and at head dimension 64 three workgroups to a
compute unit: remainders of tasks and of rows, with and without query rotation and log-sum-exps, against float64.  The launch
takes these forms beyond 256 workgroups (a 256-CU device)."""

import numpy as np
import pytest
import torch

import paper_2406_12018_amd as api
from oracle import citrus_oracle as orc

from helpers import assert_close, np64

pytestmark = pytest.mark.gpu
DEV = "cuda"

# L, Hq, Hkv, c, n_c, layers that are checked
SHAPES = [
    (40, 7, 1, 300, 70, [0, 39]),     # 70 tasks of a unit: nine blocks, the last of six
    (24, 12, 4, 97, 64, [0, 23]),     # groups of three: twelve tasks, a tile of one row
    (40, 10, 2, 40, 0, [39]),         # groups of five
    (20, 42, 6, 65, 130, [7]),        # groups of seven, a pair of blocks and a rest
    (12, 32, 8, 130, 100, [0, 11]),   # head_dim 64: three to a compute unit
    (70, 8, 8, 200, 63, [69]),        # one head per group
]


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(str(x) for x in s[:5]))
def test_blocks_of_tasks(shape, head_dim):
    L, Hq, Hkv, c, n_c, checked = shape
    print(f"attention tasks {shape} head_dim {head_dim}", flush=True)
    g = torch.Generator(device="cpu").manual_seed(5)
    rand = lambda *s: torch.randn(s, generator=g).to(torch.bfloat16).to(DEV)
    cfg = api.Config(batch=1, layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=head_dim, chunk_len=c, budget=n_c + 5, instr_len=4)
    q, k, v = rand(1, L, Hq, c, head_dim), rand(1, L, Hkv, c, head_dim), rand(1, L, Hkv, c, head_dim)
    kc, vc = rand(1, L, Hkv, n_c + 5, head_dim), rand(1, L, Hkv, n_c + 5, head_dim)
    guard = torch.full((1, L, Hq, c + 3, head_dim), 7.0, dtype=torch.bfloat16, device=DEV)  # rows behind the last are not written
    lse = torch.full((1, L, Hq, c), float("nan"), dtype=torch.float32, device=DEV)
    lse_cache = torch.full_like(lse, float("nan")) if n_c else None
    api.citrus_chunk_attn(cfg, q, kc, vc, n_c, k, v, out=guard[..., :c, :], lse=lse, lse_cache=lse_cache)
    assert (guard[..., c:, :] == 7.0).all()
    out = guard[..., :c, :]
    for l in checked:
        kcat = np.concatenate([np64(kc[0, l, :, :n_c]), np64(k[0, l])], axis=1)
        vcat = np.concatenate([np64(vc[0, l, :, :n_c]), np64(v[0, l])], axis=1)
        o_ref, lse_ref, _ = orc.chunk_attn(np64(q[0, l]), kcat, vcat, n_c)
        assert_close(np64(out[0, l]), o_ref, "bf16", f"out l{l}")
        assert_close(np64(lse[0, l]), lse_ref, "bf16", f"lse l{l}")
        if n_c:
            s = np.einsum("hqd,hkd->hqk", np64(q[0, l]), np.repeat(kcat[:, :n_c], Hq // Hkv, axis=0)) / np.sqrt(head_dim)
            m = s.max(-1)
            assert_close(np64(lse_cache[0, l]), m + np.log(np.exp(s - m[..., None]).sum(-1)), "bf16", f"lse_cache l{l}")
    # the same rows whatever the launch: one layer alone, in blocks of four waves
    one = api.Config(**{**cfg.__dict__, "layers": 1})
    alone = api.citrus_chunk_attn(one, *(t[:, -1:] for t in (q, kc, vc)), n_c, k[:, -1:], v[:, -1:])
    assert torch.equal(out[:, -1:], alone)


@pytest.mark.parametrize("head_dim", [64, 128])
def test_rotated_queries_of_mixed_heads(head_dim):
    L, Hq, Hkv, c, budget = 40, 7, 1, 100, 70
    cfg = api.Config(batch=1, layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=head_dim, chunk_len=c, budget=budget, instr_len=4, position_shift=1)
    g = torch.Generator(device="cpu").manual_seed(6)
    rand = lambda *s: torch.randn(s, generator=g).to(torch.bfloat16).to(DEV)
    q, k, v, qi = rand(1, L, Hq, 2 * c, head_dim), rand(1, L, Hkv, 2 * c, head_dim), rand(1, L, Hkv, 2 * c, head_dim), rand(2, 1, L, Hq, 4, head_dim)
    out, state, ws = torch.empty_like(q), api.DocumentState.allocate(cfg), api.alloc_workspace(cfg)
    doc = api.resident_doc(cfg, q, k, v, qi, out)
    api.citrus_process_document(cfg, state, ws, doc=doc, max_chunks=1)
    n_c, kc, vc = state.cache_len, state.k_cache[state.buffer_index].clone(), state.v_cache[state.buffer_index].clone()
    api.citrus_process_document(cfg, state, ws, doc=doc, first_chunk=1)
    plain = api.Config(**{**cfg.__dict__, "position_shift": 0})
    last = slice(c, None)
    rotate = lambda t, at: api.citrus_rope(cfg, t.contiguous(), at)
    ref = api.citrus_chunk_attn(plain, rotate(q[..., last, :], n_c), rotate(kc, 0), vc, n_c, rotate(k[..., last, :], n_c), v[..., last, :].contiguous())
    assert torch.equal(out[..., last, :], ref)
