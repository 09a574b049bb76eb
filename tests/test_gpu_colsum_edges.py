"""Column sums with known normalisers at the edges of their tiles: rows of several heads in one tile, ragged chunks of rows,
blocks of 128 and of 256 keys, the causal mask; against float64.

Tolerance: a weight is exp2 of a difference of two numbers below 64 that carry rounding errors of a few 2^-24 each (and a
product sum of at most 128 exact bf16 products): below 5e-5 relative; a sum of positive weights keeps that."""

import numpy as np
import pytest
import torch

import paper_2406_12018_amd as api

from helpers import np64

pytestmark = pytest.mark.gpu
DEV = "cuda"


def rand(shape, seed):
    g = torch.Generator(device="cpu").manual_seed(seed)
    return torch.randn(shape, generator=g, dtype=torch.float32).to(torch.bfloat16).to(DEV)


def logits(q, k, G, d):
    return np.einsum("hqd,hkd->hqk", np64(q), np.repeat(np64(k), G, axis=0)) / np.sqrt(d)


def by_group(w, Hkv):  # [Hq, rows, keys] -> [Hkv, keys]
    return w.reshape(Hkv, -1, w.shape[-1]).sum(1)


# L, Hq, Hkv, rows, keys; 128 keys per workgroup while that is the shorter sum of turns
SHAPES = [(1, 1, 1, 1, 1), (1, 3, 1, 31, 63), (2, 8, 2, 33, 65), (1, 7, 1, 5, 129), (1, 4, 2, 257, 127), (3, 14, 2, 100, 300),
          (1, 8, 1, 512, 257), (40, 8, 8, 64, 256), (64, 8, 8, 40, 200), (60, 4, 4, 256, 300)]


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
def test_cache_score_with_given_normalisers(shape, head_dim):
    L, Hq, Hkv, rows, n = shape
    print(f"column sums {shape} head_dim {head_dim}", flush=True)
    cfg = api.Config(batch=1, layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=head_dim, chunk_len=rows, budget=n, instr_len=4)
    q, k = rand((1, L, Hq, rows, head_dim), 1), rand((1, L, Hkv, n, head_dim), 2)
    lse = torch.empty((1, L, Hq, rows), dtype=torch.float32, device=DEV)
    want = np.empty((L, Hkv, n))
    for l in range(L):
        s = logits(q[0, l], k[0, l], Hq // Hkv, head_dim)
        m = s.max(-1, keepdims=True)
        norm = (m + np.log(np.exp(s - m).sum(-1, keepdims=True))).astype(np.float32)
        lse[0, l] = torch.from_numpy(norm[..., 0])
        want[l] = by_group(np.exp(s - norm.astype(np.float64)), Hkv)
    score = api.citrus_cache_score(cfg, q, k, n, lse_cache=lse)
    np.testing.assert_allclose(np64(score[0]), want, rtol=5e-5, atol=1e-9)
    assert torch.equal(score, api.citrus_cache_score(cfg, q, k, n, lse_cache=lse))


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("shape", [(64, 8, 8, 40, 200), (16, 32, 8, 500, 1000)], ids=lambda s: "-".join(map(str, s)))
def test_a_units_bits_do_not_depend_on_the_launch(shape, head_dim):
    """One layer alone, in blocks of 128 keys, and in a launch that fills the chip with blocks of 256."""
    L, Hq, Hkv, rows, n = shape
    print(f"column sums alone {shape} head_dim {head_dim}", flush=True)
    make = lambda layers: api.Config(batch=1, layers=layers, q_heads=Hq, kv_heads=Hkv, head_dim=head_dim, chunk_len=rows, budget=n, instr_len=4)
    q, k = rand((1, L, Hq, rows, head_dim), 1), rand((1, L, Hkv, n, head_dim), 2)
    lse = 6 + torch.rand((1, L, Hq, rows), device=DEV)
    score = api.citrus_cache_score(make(L), q, k, n, lse_cache=lse)
    for l in (0, L - 1):
        assert torch.equal(score[:, l:l + 1], api.citrus_cache_score(make(1), q[:, l:l + 1], k[:, l:l + 1], n, lse_cache=lse[:, l:l + 1].contiguous()))


# L, Hq, Hkv, rows, cached states: chunks of rows none of which sees a key of the block, tiles that wrap, blocks of both sizes
CAUSAL = [(1, 2, 1, 1, 0), (1, 4, 1, 33, 0), (1, 3, 1, 97, 31), (2, 8, 2, 300, 70), (1, 4, 2, 600, 0), (1, 8, 1, 640, 130),
          (64, 8, 8, 130, 100), (40, 8, 8, 300, 0)]


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("shape", CAUSAL, ids=lambda s: "-".join(map(str, s)))
def test_importance_of_the_chunk(shape, head_dim):
    """Also with a row that sees a NaN: its normaliser is NaN, and so is what it gives to the keys that it sees; the keys
    behind it are seen by rows that see the NaN as well, and those in front of it get nothing from its row alone."""
    L, Hq, Hkv, c, n_c = shape
    print(f"causal column sums {shape} head_dim {head_dim}", flush=True)
    cfg = api.Config(batch=1, layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=head_dim, chunk_len=c, budget=n_c + 1, instr_len=4)
    q, k, v = rand((1, L, Hq, c, head_dim), 1), rand((1, L, Hkv, c, head_dim), 2), rand((1, L, Hkv, c, head_dim), 3)
    kc, vc = rand((1, L, Hkv, n_c + 1, head_dim), 4), rand((1, L, Hkv, n_c + 1, head_dim), 5)

    def run(q):
        lse, score = torch.empty((1, L, Hq, c), dtype=torch.float32, device=DEV), torch.empty((1, L, Hkv, n_c + c), dtype=torch.float32, device=DEV)
        api.citrus_chunk_attn(cfg, q, kc, vc, n_c, k, v, lse=lse, lm_score=score)
        return lse, score

    lse, score = run(q)
    visible = np.arange(n_c + c)[None, None, :] <= n_c + np.arange(c)[None, :, None]
    for l in sorted({0, L - 1}):
        s = logits(q[0, l], torch.cat([kc[0, l, :, :n_c], k[0, l]], dim=1), Hq // Hkv, head_dim)
        w = np.where(visible, np.exp(s - np64(lse[0, l])[..., None]), 0.0)
        np.testing.assert_allclose(np64(score[0, l]), by_group(w, Hkv), rtol=5e-5, atol=1e-9)
    bad = c // 2  # one query row of head 0 is NaN: so is its normaliser
    q_bad = q.clone()
    q_bad[0, 0, 0, bad] = float("nan")
    _, score_bad = run(q_bad)
    assert score_bad[0, 0, 0, :n_c + bad + 1].isnan().all()
    assert not score_bad[0, 0, 0, n_c + bad + 1:].isnan().any() and torch.equal(score_bad[0, :, 1:], score[0, :, 1:])


@pytest.mark.parametrize("L, Hq, Hkv, c, n_c, head_dim", [(129, 32, 8, 128, 70, 128), (70, 32, 4, 256, 100, 128), (130, 32, 8, 256, 33, 64)])
def test_importance_in_a_long_launch(L, Hq, Hkv, c, n_c, head_dim):
    """More than 393216 query rows, 128 at a time within a head, take the kernel of short waves: the bits of a layer alone."""
    print(f"long causal launch {L, Hq, Hkv, c, n_c, head_dim}", flush=True)
    assert L * Hq * c > 3 << 17
    g = torch.Generator(device=DEV).manual_seed(5)
    make = lambda h, rows: torch.randn((1, L, h, rows, head_dim), generator=g, device=DEV).to(torch.bfloat16)
    q, k, v, kc, vc = make(Hq, c), make(Hkv, c), make(Hkv, c), make(Hkv, n_c), make(Hkv, n_c)

    def run(l0, l1):
        cfg = api.Config(batch=1, layers=l1 - l0, q_heads=Hq, kv_heads=Hkv, head_dim=head_dim, chunk_len=c, budget=n_c, instr_len=4)
        lse, score = torch.empty((1, l1 - l0, Hq, c), device=DEV), torch.empty((1, l1 - l0, Hkv, n_c + c), device=DEV)
        api.citrus_chunk_attn(cfg, q[:, l0:l1], kc[:, l0:l1], vc[:, l0:l1], n_c, k[:, l0:l1], v[:, l0:l1], lse=lse, lm_score=score)
        return lse, score

    lse, score = run(0, L)
    for l in (0, L - 1):
        lse_alone, alone = run(l, l + 1)
        assert torch.equal(lse[:, l:l + 1], lse_alone) and torch.equal(score[:, l:l + 1], alone)


@pytest.mark.parametrize("shape", [(256, 8, 8, 300, 500), (96, 16, 16, 211, 900)], ids=lambda s: "-".join(map(str, s)))
@pytest.mark.parametrize("head_dim", [64, 128])
def test_a_units_bits_in_short_waves(shape, head_dim):
    """Few rows per KV head in a launch of several turns, which takes the kernel of short waves, and one layer alone, which does not
    (test_dispatch_cpu.py has the rule)."""
    test_a_units_bits_do_not_depend_on_the_launch(shape, head_dim)


@pytest.mark.parametrize("L, Hq, Hkv, c, n_c, head_dim", [(128, 24, 8, 250, 300, 128), (128, 64, 16, 200, 300, 64), (96, 28, 4, 131, 1000, 64),
                                                          (40, 8, 8, 1000, 500, 64), (150, 12, 12, 333, 97, 128)])
def test_importance_of_ragged_rows_in_short_waves(L, Hq, Hkv, c, n_c, head_dim):
    """The same under the mask, with rows of several heads in a tile and a rest behind the last."""
    print(f"ragged causal launch {L, Hq, Hkv, c, n_c, head_dim}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(6)
    make = lambda h, rows: torch.randn((1, L, h, rows, head_dim), generator=g, device=DEV).to(torch.bfloat16)
    q, k, v, kc, vc = make(Hq, c), make(Hkv, c), make(Hkv, c), make(Hkv, n_c), make(Hkv, n_c)

    def run(l0, l1):
        cfg = api.Config(batch=1, layers=l1 - l0, q_heads=Hq, kv_heads=Hkv, head_dim=head_dim, chunk_len=c, budget=n_c, instr_len=4)
        score = torch.empty((1, l1 - l0, Hkv, n_c + c), device=DEV)
        api.citrus_chunk_attn(cfg, q[:, l0:l1], kc[:, l0:l1], vc[:, l0:l1], n_c, k[:, l0:l1], v[:, l0:l1], lm_score=score,
                              workspace=api.alloc_workspace(cfg))
        return score

    score = run(0, L)
    for l in (0, L - 1):
        assert torch.equal(score[:, l:l + 1], run(l, l + 1))
    s = logits(q[0, 0], torch.cat([kc[0, 0], k[0, 0]], dim=1), Hq // Hkv, head_dim)
    s = np.where(np.arange(n_c + c)[None, None, :] <= n_c + np.arange(c)[None, :, None], s, -np.inf)
    w = np.exp(s - s.max(-1, keepdims=True))
    # normalisers from the attention's log-sum-exps: bf16's tolerance of 1e-2 for their rounded probabilities
    np.testing.assert_allclose(np64(score[0, 0]), by_group(w / w.sum(-1, keepdims=True), Hkv), rtol=1e-2, atol=1e-6)
