"""Chunk attention of launches that leave compute units idle (four waves per workgroup, row blocks that are not paired)
and the cache-only normaliser at caches of every remainder.  Shapes sit on both sides of each line (a 256-CU device) and
at the edges of tiles and segments, against the CPU oracle; the split of a launch does not change a row's bits."""

import numpy as np
import pytest
import torch

import paper_2406_12018_amd as api
from oracle import citrus_oracle as orc

from helpers import assert_close, np64

pytestmark = pytest.mark.gpu
DEV = "cuda"


def rand(shape, seed):
    g = torch.Generator(device="cpu").manual_seed(seed)
    return torch.randn(shape, generator=g, dtype=torch.float32).to(torch.bfloat16).to(DEV)


# L, Hq, Hkv, c, n_c, layers that are checked
SHAPES = [
    (1, 1, 1, 1, 0, [0]),        # one key
    (1, 2, 1, 1, 64, [0]),       # one whole cache tile and one chunk state
    (1, 4, 2, 65, 64, [0]),      # the chunk begins with the second tile and ends behind it
    (1, 4, 1, 64, 128, [0]),     # tiles that end exactly
    (2, 3, 1, 33, 63, [1]),      # one row short of a cache tile
    (1, 8, 2, 130, 200, [0]),    # ragged end of the cache behind whole tiles
    (1, 7, 1, 97, 1, [0]),       # a cache of one state: a half tile without a key
    (1, 4, 1, 40, 96, [0]),      # the cache ends with half a tile
    (16, 32, 8, 33, 64, [0, 15]),   # 256 workgroups of four waves
    (17, 32, 8, 33, 70, [16]),      # 272, of eight waves 136: a row block each
    (11, 32, 8, 65, 128, [0, 10]),  # 264, 176
    (32, 32, 8, 65, 64, [31]),      # 512 row blocks of eight waves: in pairs
]


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(str(x) for x in s[:5]))
def test_small_launches(shape, head_dim):
    L, Hq, Hkv, c, n_c, checked = shape
    print(f"small attention launch {shape} head_dim {head_dim}", flush=True)
    cfg = api.Config(batch=1, layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=head_dim, chunk_len=c, budget=n_c + 5, instr_len=4)
    q = rand((1, L, Hq, c, head_dim), 1)
    kc, vc = rand((1, L, Hkv, n_c + 5, head_dim), 2), rand((1, L, Hkv, n_c + 5, head_dim), 3)
    k, v = rand((1, L, Hkv, c, head_dim), 4), rand((1, L, Hkv, c, head_dim), 5)
    lse = torch.full((1, L, Hq, c), float("nan"), dtype=torch.float32, device=DEV)
    lse_cache = torch.full_like(lse, float("nan")) if n_c else None
    out = api.citrus_chunk_attn(cfg, q, kc, vc, n_c, k, v, lse=lse, lse_cache=lse_cache)
    torch.cuda.synchronize()
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
    assert torch.equal(out, api.citrus_chunk_attn(cfg, q, kc, vc, n_c, k, v))
    one = api.Config(**{**cfg.__dict__, "layers": 1})
    alone = api.citrus_chunk_attn(one, *(t[:, -1:] for t in (q, kc, vc)), n_c, k[:, -1:], v[:, -1:])
    assert torch.equal(out[:, -1:], alone), "the last layer alone"


# layers, rows per step, budget: 33 and 65 rows make one and two row blocks of eight waves, 130 three (a pair and a rest);
# budgets are the second step's cached states, most of them no multiple of a 64-key tile
ROTATED = [(1, 33, 40), (11, 65, 40), (32, 65, 70), (16, 130, 100), (16, 130, 128)]


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("layers,c,budget", ROTATED, ids=["four_waves", "eight_waves", "pairs", "pairs_and_a_rest", "whole_tiles"])
def test_rotated_queries(layers, c, budget, head_dim):
    """Position shift: the kernels that rotate their query rows against the rotation as a call of its own."""
    print(f"rotated queries {layers} layers {c} rows budget {budget} head_dim {head_dim}", flush=True)
    cfg = api.Config(batch=1, layers=layers, q_heads=32, kv_heads=8, head_dim=head_dim, chunk_len=c, budget=budget, instr_len=4,
                     position_shift=1)
    rows = 3 * c
    q, k, v = rand((1, layers, 32, rows, head_dim), 1), rand((1, layers, 8, rows, head_dim), 2), rand((1, layers, 8, rows, head_dim), 3)
    qi, out, state = rand((3, 1, layers, 32, 4, head_dim), 4), torch.empty_like(q), api.DocumentState.allocate(cfg)
    ws = api.alloc_workspace(cfg)
    doc = api.resident_doc(cfg, q, k, v, qi, out)
    api.citrus_process_document(cfg, state, ws, doc=doc, max_chunks=2)
    n_c = state.cache_len
    assert n_c == budget
    kc, vc = state.k_cache[state.buffer_index].clone(), state.v_cache[state.buffer_index].clone()
    api.citrus_process_document(cfg, state, ws, doc=doc, first_chunk=2)
    plain = api.Config(**{**cfg.__dict__, "position_shift": 0})
    last = slice(2 * c, None)
    q_r = api.citrus_rope(cfg, q[..., last, :].contiguous(), n_c)
    k_r, kc_r = api.citrus_rope(cfg, k[..., last, :].contiguous(), n_c), api.citrus_rope(cfg, kc, 0)
    ref = api.citrus_chunk_attn(plain, q_r, kc_r, vc, n_c, k_r, v[..., last, :].contiguous())
    assert torch.equal(out[..., last, :], ref)
