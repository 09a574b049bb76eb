"""The eviction of one cache: every instance of the kernel that selects and gathers in one launch at the edges of its range
(candidates per thread, parts of a unit with a remainder, one and several partial sums), and what lies beyond it, against the same
steps issued one by one, bit for bit.  What is compared with is itself compared with the oracle in test_gpu_parity.py.  Two
caches, appended rows and carried sums: test_gpu_fused_launches.py."""

import pytest
import torch

import paper_2406_12018_amd as api

pytestmark = pytest.mark.gpu
DEV = "cuda"


def rand(shape, seed, dtype=torch.bfloat16):
    g = torch.Generator(device="cpu").manual_seed(seed)
    return torch.randn(shape, generator=g, dtype=torch.float32).to(dtype).to(DEV)


# layers, query heads, KV heads, head_dim, instruction rows, states, kept, start size, type
CASES = [
    (1, 1, 1, 64, 1, 2, 1, 0, "f32"),          # the smallest
    (1, 4, 1, 64, 8, 96, 64, 0, "f32"),
    (1, 4, 2, 128, 3, 511, 500, 4, "bf16"),    # two candidates per thread, the last thread's one
    (1, 4, 2, 64, 3, 512, 17, 0, "bf16"),
    (1, 4, 2, 128, 17, 512, 300, 0, "bf16"), (2, 8, 2, 64, 64, 257, 200, 3, "bf16"),  # two per thread; partial sums
    (1, 8, 2, 128, 64, 513, 512, 0, "bf16"),   # five per thread; partial sums
    (1, 32, 8, 128, 64, 1280, 768, 2, "bf16"),
    (2, 32, 8, 128, 64, 1281, 1280, 0, "bf16"),  # eight per thread; one state leaves
    (1, 4, 4, 128, 16, 2048, 1000, 0, "bf16"),
    (1, 4, 1, 128, 16, 2049, 1999, 0, "bf16"),  # 1024 threads
    (1, 8, 2, 128, 64, 2560, 31, 5, "bf16"),
    (3, 4, 2, 128, 16, 6144, 4096, 0, "bf16"),
    (32, 8, 8, 64, 2, 6144, 6100, 0, "bf16"),  # two launches: more rows than one is worth
    (32, 8, 8, 64, 2, 6144, 1400, 0, "bf16"),  # one part of a unit, 1024 threads
    (32, 8, 8, 128, 2, 1280, 765, 0, "bf16"), (32, 8, 8, 128, 2, 1280, 768, 0, "bf16"),  # the sides of 96 MB
    (1, 2, 1, 128, 16, 6145, 777, 0, "bf16"),   # too many for one launch
    (40, 16, 8, 128, 8, 90, 33, 0, "bf16"),     # more units than workgroups wanted
    (1, 4, 2, 128, 3, 100, 100, 0, "bf16"),     # nothing leaves
]


@pytest.mark.parametrize("per_layer", [0, 1], ids=["per_head", "per_layer"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(x) for x in c))
def test_eviction_against_its_steps(case, per_layer):
    L, Hq, Hkv, d, rows, n, k, start, dtype = case
    print(f"eviction {case} per_layer {per_layer}", flush=True)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    cfg = api.Config(batch=1, layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=d, chunk_len=16, budget=max(k, start + 1), instr_len=rows,
                     dtype=api.F32 if dtype == "f32" else api.BF16, cache_capacity=n, start_size=start, select_mode=per_layer)
    q, kc, vc = rand((1, L, Hq, rows, d), 1, dt), rand((1, L, Hkv, n, d), 2, dt), rand((1, L, Hkv, n, d), 3, dt)
    ws = api.alloc_workspace(cfg)
    k_new, v_new = torch.zeros((1, L, Hkv, k, d), dtype=dt, device=DEV), torch.zeros((1, L, Hkv, k, d), dtype=dt, device=DEV)
    idx = torch.full((1, L, cfg.sel_heads, k), -1, dtype=torch.int32, device=DEV)
    assert api.citrus_evict_cache(cfg, q, kc, vc, n, k, k_new, v_new, idx=idx, workspace=ws) == min(k, n)
    score = api.citrus_cache_score(cfg, q, kc, n, workspace=ws)
    want = api.citrus_topk_select(cfg, score, k)
    assert torch.equal(idx, want)
    rows_of = want.long().expand(1, L, Hkv, k)[..., None].expand(-1, -1, -1, -1, d)
    assert torch.equal(k_new, torch.gather(kc, 3, rows_of)) and torch.equal(v_new, torch.gather(vc, 3, rows_of))
    k_new.zero_()
    assert api.citrus_evict_cache(cfg, q, kc, vc, n, k, k_new, v_new, workspace=ws) == min(k, n)  # no positions asked for
    assert torch.equal(k_new, torch.gather(kc, 3, rows_of))
