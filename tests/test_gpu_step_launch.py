"""A step in one launch (attention, instruction score and the eviction by it) at the edges of its forms: one strip of instruction rows
and several, both numbers of key tiles, the most candidates, first steps that keep everything and first steps that evict.  The same
bits as the launches apart, twice over one workspace; a second document of another size on it finds its counters as it needs them."""

import pytest
import torch

import paper_2406_12018_amd as api
from test_gpu_fused_launches import test_merged_launches_give_the_bits_of_the_launches_apart as same_bits

pytestmark = pytest.mark.gpu

# dtype, L, Hq, Hkv, d, chunk, T, budget, instruction rows, options
CASES = [
    ("bf16", 1, 4, 4, 128, 64, 300, 100, 32, {}),               # one strip of 32 rows per head
    ("bf16", 1, 8, 4, 64, 130, 700, 129, 17, {}),               # two strips, the second of two rows; the first step evicts
    ("bf16", 1, 32, 8, 128, 100, 500, 37, 64, {}),              # eight strips
    ("bf16", 2, 16, 2, 128, 33, 200, 400, 70, {}),              # nothing is evicted
    ("bf16", 1, 8, 2, 128, 500, 2100, 780, 40, {}),             # 1280 candidates
    ("bf16", 1, 8, 2, 64, 500, 2100, 781, 40, {}),              # 1281
    ("bf16", 1, 4, 1, 64, 700, 4000, 1860, 30, dict(start_size=3)),  # 2560, the most
    ("bf16", 1, 8, 1, 128, 200, 1100, 300, 21, dict(score_mode=api.SCORE_ACCUMULATED)),  # sums of the first step are carried on
    ("bf16", 3, 8, 2, 128, 96, 500, 150, 16, dict(position_shift=1)),
    ("bf16", 1, 21, 3, 128, 150, 900, 200, 33, {}),             # eight strips of each of three units: over all XCDs
    ("bf16", 5, 20, 5, 64, 100, 700, 130, 40, {}),
    ("bf16", 16, 8, 4, 64, 98, 500, 65, 40, {}),                # 256 workgroups of the attention behind 192 of the score
    ("bf16", 1, 128, 32, 128, 64, 300, 70, 96, {}),             # 384 strips of 32 rows would be more than the compute units: 64 rows each
    ("bf16", 1, 64, 8, 128, 512, 2000, 768, 192, {}),           # the same, 1280 candidates
    ("bf16", 33, 16, 4, 64, 32, 150, 60, 12, {}),               # one strip of 64 rows per unit, 48 of them there
    ("bf16", 1, 48, 6, 64, 256, 1100, 700, 256, dict(position_shift=1)),
    ("f32", 1, 4, 1, 64, 32, 300, 64, 8, {}),
    ("f32", 2, 4, 2, 128, 60, 300, 125, 9, dict(start_size=2)),
    ("f32", 1, 2, 2, 64, 212, 900, 300, 30, dict(score_mode=api.SCORE_ACCUMULATED)),  # 512 candidates, 150 KB kept: gather apart
    ("f32", 1, 2, 1, 128, 20, 90, 200, 16, dict(position_shift=1)),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(x) for x in c[:9]))
def test_step_in_one_launch(case):
    same_bits(case)
    same_bits(case)


def test_a_provider_that_uses_the_workspace():
    """Behind the provider's own calls on the call's workspace a step finds its counters as it needs them."""
    print("provider on the workspace", flush=True)
    H, Hkv, d, c, budget, rows, steps = 16, 4, 128, 64, 100, 40, 5
    cfg = api.Config(batch=1, layers=2, q_heads=H, kv_heads=Hkv, head_dim=d, chunk_len=c, budget=budget, instr_len=rows)
    g = torch.Generator(device="cpu").manual_seed(4)
    mk = lambda *shape: torch.randn(shape, generator=g).to(torch.bfloat16).to("cuda")
    q, k, v, qi = mk(1, 2, H, steps * c, d), mk(1, 2, Hkv, steps * c, d), mk(1, 2, Hkv, steps * c, d), mk(steps, 1, 2, H, rows, d)
    ws, runs = api.alloc_workspace(cfg), []
    lm_score = torch.empty((1, 2, Hkv, c), dtype=torch.float32, device="cuda")
    for used in (False, True):
        out, state = torch.empty_like(q), api.DocumentState.allocate(cfg)
        for t in (*state.k_cache, *state.v_cache):
            t.zero_()

        def provider(i, io):
            if i == steps:
                return 1
            qc, kc, vc, oc = (t[:, :, :, i * c:(i + 1) * c] for t in (q, k, v, out))
            if used:
                api.citrus_chunk_attn(cfg, qc, None, None, 0, kc, vc, lm_score=lm_score, workspace=ws)
            io.q, io.k, io.v, io.out = (api.binding.tensor(t) for t in (qc, kc, vc, oc))
            io.q_instr, io.chunk_len = api.binding.tensor(qi[i]), c
            return 0
        assert api.citrus_process_document(cfg, state, ws, provider=provider) == steps
        torch.cuda.synchronize()
        runs.append([out, *(t.clone() for t in state.current())])
    for a, b in zip(*runs):
        assert torch.equal(a, b)
