"""bf16 with head dimension 64 on the matrix-core kernels: every kernel a step can reach, at the edges of tiles and row
blocks and on both sides of the scorer's and the decoding step's choices, against the CPU oracle."""

import numpy as np
import pytest
import torch

import paper_2406_12018_amd as api
from oracle import citrus_oracle as orc

from helpers import assert_close, np64

pytestmark = pytest.mark.gpu
DEV = "cuda"
D = 64


def rand(shape, seed, scale=1.0):
    g = torch.Generator(device="cpu").manual_seed(seed)
    return (torch.randn(shape, generator=g, dtype=torch.float32) * scale).to(torch.bfloat16).to(DEV)


# B, L, Hq, Hkv, c, n_c, n_i, spread of q and k
STEPS = [
    (1, 1, 1, 1, 1, 0, 1, 1.0),         # one key, one row
    (1, 2, 4, 4, 33, 31, 31, 1.0),      # one head per group: eight row tiles per workgroup, ragged everywhere
    (1, 1, 6, 2, 64, 64, 32, 1.0),      # three heads per group, tiles that end exactly
    (2, 1, 8, 2, 129, 127, 64, 1.0),    # a tile that holds the cache / chunk boundary and one past a row block
    (1, 1, 8, 4, 256, 960, 128, 1.0),   # 256 rows per KV group
    (1, 1, 8, 1, 128, 1000, 128, 0.5),  # 1024 rows per KV group: two launches, staged rows in whole chunks
    (1, 1, 7, 1, 95, 3000, 36, 0.5),    # seven heads per group, long ragged cache
]


@pytest.mark.parametrize("shape", STEPS, ids=lambda s: "-".join(str(x) for x in s[:7]))
def test_step_kernels(shape):
    B, L, Hq, Hkv, c, n_c, n_i, s = shape
    print(f"head_dim 64 step {shape}", flush=True)
    cfg = api.Config(batch=B, layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=D, chunk_len=c, budget=n_c + 3, instr_len=n_i)
    ws = api.alloc_workspace(cfg)
    q, qi = rand((B, L, Hq, c, D), 1, s), rand((B, L, Hq, n_i, D), 2, s)
    kc, vc = rand((B, L, Hkv, n_c + 3, D), 3, s), rand((B, L, Hkv, n_c + 3, D), 4)
    k, v = rand((B, L, Hkv, c, D), 5, s), rand((B, L, Hkv, c, D), 6)
    lse = torch.empty((B, L, Hq, c), dtype=torch.float32, device=DEV)
    lm = torch.empty((B, L, Hkv, n_c + c), dtype=torch.float32, device=DEV)
    out = api.citrus_chunk_attn(cfg, q, kc, vc, n_c, k, v, lse=lse, lm_score=lm, workspace=ws)
    score = api.citrus_instr_score(cfg, qi, kc, n_c, k, workspace=ws)
    torch.cuda.synchronize()
    for b in range(B):
        for l in range(L):
            kcat = np.concatenate([np64(kc[b, l, :, :n_c]), np64(k[b, l])], axis=1)
            vcat = np.concatenate([np64(vc[b, l, :, :n_c]), np64(v[b, l])], axis=1)
            o_ref, lse_ref, _ = orc.chunk_attn(np64(q[b, l]), kcat, vcat, n_c)
            assert_close(np64(out[b, l]), o_ref, "bf16", f"out b{b} l{l}")
            assert_close(np64(lse[b, l]), lse_ref, "bf16", f"lse b{b} l{l}")
            assert_close(np64(lm[b, l]), orc.lm_score(np64(q[b, l]), kcat, n_c), "bf16", f"lm_score b{b} l{l}")
            assert_close(np64(score[b, l]), orc.instr_score(np64(qi[b, l]), kcat), "bf16", f"score b{b} l{l}")
    assert torch.equal(out, api.citrus_chunk_attn(cfg, q, kc, vc, n_c, k, v, workspace=ws))
    assert torch.equal(score, api.citrus_instr_score(cfg, qi, kc, n_c, k, workspace=ws))


@pytest.mark.parametrize("G,n", [(1, 0), (4, 31), (8, 32), (7, 700), (4, 2500), (32, 65)])
def test_decode_step(G, n):
    """One token over n cached states, in one and in several key ranges."""
    print(f"head_dim 64 decode G={G} n={n}", flush=True)
    Hkv = 2
    cfg = api.Config(batch=1, layers=1, q_heads=G * Hkv, kv_heads=Hkv, head_dim=D, chunk_len=32, budget=n + 2, instr_len=8)
    ws = api.alloc_workspace(cfg)
    q, kn, vn = rand((1, 1, G * Hkv, 1, D), 1), rand((1, 1, Hkv, 1, D), 2), rand((1, 1, Hkv, 1, D), 3)
    kc, vc = rand((1, 1, Hkv, n + 2, D), 4), rand((1, 1, Hkv, n + 2, D), 5)
    ref, *_ = orc.chunk_attn(np64(q[0, 0]), np.concatenate([np64(kc[0, 0, :, :n]), np64(kn[0, 0])], axis=1),
                             np.concatenate([np64(vc[0, 0, :, :n]), np64(vn[0, 0])], axis=1), n)
    out = api.citrus_decode_step(cfg, q, kn, vn, kc, vc, n, workspace=ws)
    torch.cuda.synchronize()
    assert_close(np64(out[0, 0]), ref, "bf16", "out")
    assert torch.equal(kc[:, :, :, n:n + 1], kn) and torch.equal(vc[:, :, :, n:n + 1], vn)


@pytest.mark.parametrize("c,n_c", [(40, 0), (70, 90)])
def test_position_shift_rotates_queries_in_the_attention_kernel(c, n_c):
    """Two chunks with the position shift against rotated copies made by citrus_rope (itself checked against the oracle)."""
    base = dict(batch=1, layers=2, q_heads=4, kv_heads=2, head_dim=D, chunk_len=c, budget=max(n_c, 8), instr_len=8)
    shift, plain = api.Config(position_shift=1, **base), api.Config(cache_capacity=n_c + c, **base)
    q, k, v = rand((1, 2, 4, c, D), 1), rand((1, 2, 2, c, D), 2), rand((1, 2, 2, c, D), 3)
    qi, state = rand((1, 2, 4, 8, D), 4), api.DocumentState.allocate(shift)
    state.k_cache[0][:, :, :, :n_c], state.v_cache[0][:, :, :, :n_c] = rand((1, 2, 2, n_c, D), 5), rand((1, 2, 2, n_c, D), 6)
    state.cache_len = n_c
    kc, vc = state.k_cache[0].clone(), state.v_cache[0].clone()
    out = torch.empty_like(q)
    api.citrus_process_document(shift, state, api.alloc_workspace(shift), doc=api.resident_doc(shift, q, k, v, qi, out))
    want = api.citrus_chunk_attn(plain, api.citrus_rope(plain, q, n_c), api.citrus_rope(plain, kc, 0), vc, n_c,
                                 api.citrus_rope(plain, k, n_c), v)
    torch.cuda.synchronize()
    assert torch.equal(out, want)


def f64_attention(q, k, v, cached):
    """causal outputs over [cached states ; chunk] of one layer, log-sum-exps and column sums, in f64"""
    q, k, v = q.double(), k.double(), v.double()
    group = q.shape[0] // k.shape[0]
    logits = q @ k.repeat_interleave(group, 0).transpose(-1, -2).contiguous() / D ** 0.5
    seen = torch.arange(k.shape[1])[None, :] <= cached + torch.arange(q.shape[1])[:, None]
    logits = logits.masked_fill(~seen, -torch.inf)
    p = torch.softmax(logits, -1)
    return p @ v.repeat_interleave(group, 0), torch.logsumexp(logits, -1), p.reshape(k.shape[0], -1, k.shape[1]).sum(1)


def relative(x, ref):
    return float((x.double() - ref).norm() / ref.norm())


@pytest.mark.parametrize("layers", [1, 24])  # four waves per workgroup, eight in pairs of row blocks
@pytest.mark.parametrize("c,n_c,scale", [(64, 0, 2.0), (129, 100, 1.0), (300, 700, 0.5)])
def test_probabilities_keep_f32_accuracy(c, n_c, scale, layers):
    """Probabilities and row sums are f32 numbers, so the outputs are off by little more than their own rounding to bf16
    (the two bf16 parts of a probability leave 2^-18 of it against the rounding's 2^-9; 1 % allows for 2^-9 / 100) and
    the f32 results by f32's: with |logit| < 40, an exponent in log2 units carries 40 * 1.44 * 2^-24 = 3.4e-6 of rounding,
    once in the sum and once in the normaliser.  Probabilities rounded to bf16 leave 1.1 to 1.4 times the rounding in the
    outputs and 2e-4 or more in the log-sum-exps."""
    print(f"head_dim 64 accuracy c={c} n_c={n_c} layers={layers}", flush=True)
    Hq, Hkv = 8, 2
    cfg = api.Config(batch=1, layers=layers, q_heads=Hq, kv_heads=Hkv, head_dim=D, chunk_len=c, budget=max(n_c, 1), instr_len=8,
                     cache_capacity=n_c + 2)
    ws = api.alloc_workspace(cfg)
    q, k, v = rand((1, layers, Hq, c, D), 1), rand((1, layers, Hkv, c, D), 2, scale), rand((1, layers, Hkv, c, D), 3)
    kc, vc = rand((1, layers, Hkv, n_c + 2, D), 4, scale), rand((1, layers, Hkv, n_c + 2, D), 5)
    q[..., D // 2 - 1] = 4.0  # importance that all queries share: rows with a few heavy states
    lse = torch.empty((1, layers, Hq, c), dtype=torch.float32, device=DEV)
    lm = torch.empty((1, layers, Hkv, n_c + c), dtype=torch.float32, device=DEV)
    lse_cache = torch.empty_like(lse) if n_c else None
    out = api.citrus_chunk_attn(cfg, q, kc, vc, n_c, k, v, lse=lse, lm_score=lm, lse_cache=lse_cache, workspace=ws)
    one = api.citrus_decode_step(cfg, q[:, :, :, :1].contiguous(), k[:, :, :, :1].contiguous(), v[:, :, :, :1].contiguous(),
                                 kc, vc, n_c, workspace=ws)
    torch.cuda.synchronize()
    host = lambda x: x[0].cpu()
    for l in {0, layers - 1}:
        kcat = torch.cat([host(kc)[l, :, :n_c], host(k)[l]], 1)
        vcat = torch.cat([host(vc)[l, :, :n_c], host(v)[l]], 1)
        want, want_lse, want_lm = f64_attention(host(q)[l], kcat, vcat, n_c)
        rounding = relative(want.bfloat16(), want)
        assert relative(host(out)[l], want) < 1.01 * rounding
        assert float((host(lse)[l].double() - want_lse).abs().max()) < 7e-6
        assert relative(host(lm)[l], want_lm) < 7e-6
        first = want[:, :1]
        assert relative(host(one)[l], first) < 1.01 * relative(first.bfloat16(), first) + 1e-5
        if n_c:
            cached = torch.logsumexp(host(q)[l].double() @ kcat[:, :n_c].double().repeat_interleave(Hq // Hkv, 0)
                                     .transpose(-1, -2).contiguous() / D ** 0.5, -1)
            assert float((host(lse_cache)[l].double() - cached).abs().max()) < 7e-6


@pytest.mark.parametrize("layers", [1, 24])  # four waves per workgroup, eight in pairs of row blocks
@pytest.mark.parametrize("c,n_c", [(33, 0), (129, 100), (300, 65)])
def test_infinite_values_reach_only_rows_that_see_them(c, n_c, layers):
    """An infinite value (one in the cache, one in the chunk, one in the last state) makes the element infinite in the rows
    that see it and nothing else; rows that do not see a NaN key are untouched by it.  Finite elements keep the bound of
    the accuracy test."""
    print(f"head_dim 64 infinities c={c} n_c={n_c} layers={layers}", flush=True)
    Hq, Hkv, mid = 8, 2, c // 2
    cfg = api.Config(batch=1, layers=layers, q_heads=Hq, kv_heads=Hkv, head_dim=D, chunk_len=c, budget=max(n_c, 1), instr_len=8,
                     cache_capacity=n_c + 2)
    q, k, v = rand((1, layers, Hq, c, D), 1), rand((1, layers, Hkv, c, D), 2), rand((1, layers, Hkv, c, D), 3)
    kc, vc = rand((1, layers, Hkv, n_c + 2, D), 4), rand((1, layers, Hkv, n_c + 2, D), 5)
    host = lambda x: x[0].cpu()
    cat = lambda old, new: torch.cat([host(old)[-1, :, :n_c], host(new)[-1]], 1)
    want, want_lse, _ = f64_attention(host(q)[-1], cat(kc, k), cat(vc, v), n_c)
    clean = api.citrus_chunk_attn(cfg, q, kc, vc, n_c, k, v)
    v[..., mid, 5], v[..., c - 1, 63] = torch.inf, torch.nan
    if n_c:
        vc[..., n_c - 1, 0] = -torch.inf
        want[..., 0] = -torch.inf
    want[:, mid:, 5], want[:, c - 1:, 63] = torch.inf, torch.nan
    lse = torch.empty((1, layers, Hq, c), dtype=torch.float32, device=DEV)
    out = api.citrus_chunk_attn(cfg, q, kc, vc, n_c, k, v, lse=lse)
    k[..., c - 1, 7] = torch.nan
    hidden = api.citrus_chunk_attn(cfg, q, kc, vc, n_c, k, v)
    torch.cuda.synchronize()
    got, finite = host(out)[-1].double(), want.isfinite()
    assert torch.equal(got.isposinf(), want.isposinf()) and torch.equal(got.isneginf(), want.isneginf())
    assert torch.equal(got.isnan(), want.isnan())
    assert relative(got[finite], want[finite]) < 1.01 * relative(want[finite].bfloat16(), want[finite])
    assert float((host(lse)[-1].double() - want_lse).abs().max()) < 7e-6
    assert torch.equal(hidden[:, :, :, :c - 1].nan_to_num(7.0), out[:, :, :, :c - 1].nan_to_num(7.0))
    assert bool(hidden[:, :, :, c - 1].isnan().all())
    again = api.citrus_chunk_attn(cfg, q, kc, rand(vc.shape, 5), n_c, rand(k.shape, 2), rand(v.shape, 3))
    assert torch.equal(again, clean)


@pytest.mark.parametrize("G,n", [(4, 31), (7, 700), (4, 2500)])  # one key range, several
def test_infinite_values_in_a_decoding_step(G, n):
    print(f"head_dim 64 decode, infinities G={G} n={n}", flush=True)
    Hkv = 2
    cfg = api.Config(batch=1, layers=1, q_heads=G * Hkv, kv_heads=Hkv, head_dim=D, chunk_len=32, budget=n + 2, instr_len=8)
    q, kn, vn = rand((1, 1, G * Hkv, 1, D), 1), rand((1, 1, Hkv, 1, D), 2), rand((1, 1, Hkv, 1, D), 3)
    kc, vc = rand((1, 1, Hkv, n + 2, D), 4), rand((1, 1, Hkv, n + 2, D), 5)
    cat = lambda old, new: torch.cat([old[0, 0, :, :n], new[0, 0]], 1).cpu()
    want, *_ = f64_attention(q[0, 0].cpu(), cat(kc, kn), cat(vc, vn), n)
    vc[0, 0, 0, n // 2, 9], vn[0, 0, 0, 0, 60] = torch.inf, -torch.inf
    want[:G, :, 9], want[:G, :, 60] = torch.inf, -torch.inf
    out = api.citrus_decode_step(cfg, q, kn, vn, kc, vc, n, workspace=api.alloc_workspace(cfg))
    got, finite = out[0, 0].cpu().double(), want.isfinite()
    assert torch.equal(got.isposinf(), want.isposinf()) and torch.equal(got.isneginf(), want.isneginf())
    assert not bool(got.isnan().any())
    assert relative(got[finite], want[finite]) < 1.01 * relative(want[finite].bfloat16(), want[finite])
