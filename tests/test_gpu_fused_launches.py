"""Launches that a step merges while nobody asks for the events between them: attention and instruction score, selection and
gather, the evictions of two caches.  A document with every event runs them apart; outputs, positions, caches and carried sums
are the same bits, with a second stream too.  (The steps apart are compared with the oracle in test_gpu_parity.py.)"""

import ctypes as C

import pytest
import torch

import paper_2406_12018_amd as api

pytestmark = pytest.mark.gpu
DEV = "cuda"
INSTR, SHARED, DUAL, STANDARD = api.CACHE_INSTR, api.CACHE_SHARED, api.CACHE_DUAL, api.CACHE_STANDARD

# type, layers, query heads, KV heads, head_dim, chunk, document, budget, instruction, options
CASES = [
    ("f32", 1, 4, 1, 64, 32, 200, 64, 8, {}),                     # attention and score in one launch from the first chunk on
    ("f32", 2, 4, 2, 128, 48, 300, 100, 16, dict(start_size=4)),
    ("f32", 16, 32, 8, 64, 17, 100, 40, 2, {}),                   # too many workgroups for it
    ("f32", 1, 4, 2, 64, 40, 250, 70, 40, dict(position_shift=1)),
    ("bf16", 1, 32, 8, 128, 128, 1000, 300, 64, {}),              # the score's strips are added up by the eviction
    ("bf16", 1, 8, 2, 64, 100, 777, 150, 64, dict(start_size=3)),
    ("bf16", 1, 8, 2, 128, 64, 400, 128, 8, dict(position_shift=1)),
    ("bf16", 2, 32, 8, 64, 512, 2100, 768, 64, {}),
    ("bf16", 1, 16, 4, 128, 600, 3000, 1400, 40, {}),             # more than 1280 keys
    ("bf16", 2, 16, 4, 128, 96, 700, 200, 64, dict(score_mode=api.SCORE_ACCUMULATED)),          # carried sums
    ("f32", 1, 8, 2, 64, 30, 250, 64, 8, dict(score_mode=api.SCORE_ACCUMULATED, cache_mode=SHARED)),
    ("bf16", 1, 8, 4, 64, 64, 500, 128, 20, dict(score_mode=api.SCORE_ACCUMULATED, select_mode=api.SELECT_PER_LAYER)),
    ("bf16", 2, 16, 4, 128, 128, 900, 300, 64, dict(cache_mode=DUAL, budget_lm=100)),           # two jobs of different sizes
    ("bf16", 1, 8, 2, 64, 64, 500, 40, 16, dict(cache_mode=DUAL, budget_lm=200, start_size=2)),
    ("bf16", 2, 16, 4, 128, 128, 900, 200, 64, dict(cache_mode=DUAL, budget_lm=300, lm_ordering=api.LM_EVICT_THEN_APPEND)),
    ("f32", 1, 4, 2, 64, 32, 200, 64, 8, dict(cache_mode=DUAL, budget_lm=48, lm_ordering=api.LM_EVICT_THEN_APPEND)),
    ("bf16", 1, 16, 4, 128, 128, 900, 200, 16, dict(cache_mode=STANDARD, lm_ordering=api.LM_EVICT_THEN_APPEND)),  # appended rows
    ("f32", 1, 4, 2, 64, 32, 200, 64, 8, dict(cache_mode=STANDARD)),
]


def events(steps):
    made = [torch.cuda.Event(enable_timing=True) for _ in range(steps * api.binding.EVENTS_PER_STEP)]
    for e in made:
        e.record()  # the handle exists from the first record on
    return made, (C.c_void_p * len(made))(*(e.cuda_event for e in made))


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(x) for x in c[:9]) + "".join(f"-{k}{v}" for k, v in c[9].items()))
def test_merged_launches_give_the_bits_of_the_launches_apart(case):
    dtype, L, Hq, Hkv, d, chunk, T, budget, rows, options = case
    print(f"fused launches {case}", flush=True)
    g = torch.Generator(device="cpu").manual_seed(21)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    mk = lambda *shape: torch.randn(shape, generator=g).to(dt).to(DEV)
    cfg = api.Config(batch=1, layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=d, chunk_len=chunk, budget=budget, instr_len=rows,
                     dtype=api.F32 if dtype == "f32" else api.BF16, **options)
    steps = (T + chunk - 1) // chunk
    q, k, v, qi = mk(1, L, Hq, T, d), mk(1, L, Hkv, T, d), mk(1, L, Hkv, T, d), mk(steps, 1, L, Hq, rows, d)
    ws = api.alloc_workspace(cfg)
    runs = []
    for form in ("merged", "apart", "side stream"):
        out = torch.empty_like(q)
        kept = torch.full((steps, 1, L, cfg.sel_heads, budget), -1, dtype=torch.int32, device=DEV)
        kept_lm = torch.full((steps, 1, L, cfg.sel_heads, max(cfg.budget_lm, 1)), -1, dtype=torch.int32, device=DEV)
        state = api.DocumentState.allocate(cfg)
        made, handles = events(steps) if form == "apart" else (None, None)
        side = api.SideStream() if form == "side stream" else None
        done = api.citrus_process_document(cfg, state, ws, doc=api.resident_doc(cfg, q, k, v, qi, out), idx_history=kept,
                                           idx_history_lm=kept_lm if cfg.cache_mode == DUAL else None, phase_events=handles, side=side)
        torch.cuda.synchronize()
        assert done == steps
        result = [out, kept, kept_lm, *state.current()]
        if cfg.cache_mode == DUAL:
            result += state.current_lm()
        if state.acc_score is not None:
            result.append(state.acc_score[state.buffer_index][..., :state.cache_len])
        runs.append((state.cache_len, state.buffer_index, state.cache_len_lm, state.buffer_index_lm, [t.clone() for t in result]))
        del made
    for other in runs[1:]:
        assert other[:4] == runs[0][:4]
        for a, b in zip(runs[0][4], other[4]):
            assert torch.equal(a, b)
