"""The work a user of this library has it do, as cases that can be measured and compared.

A case is a dict of plain values.  `kind` says what one pass is:

  document  a whole document through citrus_process_document, then the first answer token
            (citrus_decode_step) over the states the loop retained; a cache that the document's own chunks
            evict (Standard CSE) is evicted once more by the instruction in between (citrus_evict_cache).
  layer     the same work as a model with its own layers issues it: the four entry points of a step
            (citrus_chunk_attn, citrus_instr_score, citrus_topk_select, citrus_kv_compact) chunk by chunk for
            the layers that run at the same time, outputs allocated by the calls.
  decode    `tokens` generated tokens (citrus_decode_step) over a retained cache that grows by one per token.

Inputs follow what attention meets: q, k, v are normal, every key carries an importance of its own that all
queries share (one channel with an offset in q: attention's heavy hitters, log-normal weights), the first four
states are attention sinks and one state in fifty is heavier still.  All from the seed.

What comes back is what a user reads: the attention output of every chunk, the scores while candidates still
have their document order, the tokens' outputs and the cache a token was appended to.  The retained states come
back through the attention over them: two states of nearly the same score may trade places, and then all rows
behind them move by one.
"""

from __future__ import annotations

import math

import torch

import paper_2406_12018_amd as api

_MODES = {"instr": api.CACHE_INSTR, "shared": api.CACHE_SHARED, "dual": api.CACHE_DUAL, "standard": api.CACHE_STANDARD}
ANSWER_ROWS = 64  # room behind the budget for the instruction's and the answer's states


def _case(kind, name=None, *, dtype="bf16", batch=1, layers=1, q_heads=32, kv_heads=8, head_dim=128, chunk=512, doc=4096,
          budget=768, instr=64, mode="instr", paper_order=False, per_layer=False, accumulated=False, shift=False,
          states=0, tokens=0):
    case = {"kind": kind, "dtype": dtype, "batch": batch, "layers": layers, "q_heads": q_heads, "kv_heads": kv_heads,
            "head_dim": head_dim}
    if kind == "decode":
        case.update(states=states, tokens=tokens)
    else:
        case.update(chunk=chunk, doc=doc, budget=budget, instr=instr)
    if kind == "document":
        case.update(mode=mode, paper_order=paper_order, per_layer=per_layer, accumulated=accumulated, shift=shift)
    if name is not None:
        case["name"] = name
    return case


def listed():
    return [
        # the tiny f32 configuration: a correctness run, sixteen steps of a few microseconds of work each
        _case("document", "tiny_f32", dtype="f32", q_heads=4, kv_heads=1, head_dim=64, chunk=32, doc=512, budget=64, instr=8),
        # one layer of the Mistral-7B shape inside a model that calls its layers one after the other
        _case("layer", "one_layer_steps", chunk=512, doc=2048),
        # the same layer, the whole chunk loop in one call; the document ends inside a chunk
        _case("document", "one_layer_document", doc=7941),
        # the headline workload: all 32 layers of the Mistral-7B shape, a document of 16384 tokens
        _case("document", "mistral7b_document", layers=32, doc=16384),
        # position shift (rotary embedding at cache slots), two short ragged documents
        _case("document", "position_shift", batch=2, layers=16, doc=4000, shift=True),
        # the Llama-2-7B shape: multi-head attention, long chunks and instruction, shared cache with
        # accumulated scores and layer-wise selection
        _case("document", "mha_shared_accumulated", batch=2, layers=8, q_heads=32, kv_heads=32, chunk=1024, doc=8192,
              budget=1024, instr=128, mode="shared", per_layer=True, accumulated=True),
        # individual caches: a language-modelling cache next to the instruction's
        _case("document", "dual_cache", batch=2, layers=8, doc=8192, mode="dual"),
        # Standard CSE in the printed order, final eviction by the instruction
        _case("document", "standard_paper_order", layers=16, doc=6000, mode="standard", paper_order=True),
        # the largest layers: 64 query heads, chunks of 2048, budget 4096, instruction of 256 tokens
        _case("document", "large_layers", layers=4, q_heads=64, chunk=2048, doc=16384, budget=4096, instr=256),
        # head dimension 64
        _case("document", "head_dim_64", layers=8, head_dim=64, doc=4096),
        # generation: one request, all layers in one call
        _case("decode", "decode_one_request", layers=32, states=832, tokens=4),
        # generation: four requests over long caches of the large layers
        _case("decode", "decode_batch_long", batch=4, layers=20, q_heads=64, states=4352, tokens=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: kinds, types and options in the proportions they are used in, sizes spread over their ranges.
    A case that would cost more than the largest listed one is made smaller."""
    kind = rng.choice(["document", "document", "document", "layer", "decode"])
    dtype = "f32" if rng.random() < 0.12 else "bf16"
    head_dim = 64 if rng.random() < 0.25 else 128
    group = rng.choice([1, 2, 3, 4, 4, 7, 8])
    kv_heads = rng.choice([1, 2, 4, 8, 8, 16, 32])
    while kv_heads * group > 64:
        kv_heads //= 2
    # f32 and head dimension 64 are taken in runs of modest size
    most = {("f32", 64): 2e10, ("f32", 128): 2e10, ("bf16", 64): 4e11, ("bf16", 128): 8e12}[dtype, head_dim]
    batch, layers = rng.choice([1, 1, 1, 2, 3, 4, 8]), 1 if kind == "layer" else _log(rng, 1, 40)
    common = dict(dtype=dtype, batch=batch, layers=layers, q_heads=kv_heads * group, kv_heads=kv_heads, head_dim=head_dim)
    if kind == "decode":
        case = _case("decode", states=_log(rng, 64, 6000), tokens=rng.choice([1, 2, 4, 8]), **common)
        most_bytes = 3e8 if dtype == "f32" or head_dim == 64 else 4e9
        while work(case)["bytes"] > most_bytes:
            case["layers" if case["layers"] > 1 else "states"] //= 2
        return case
    chunk = _log(rng, 32, 2048)
    budget = max(32, int(chunk * rng.uniform(0.5, 2.5)))
    case = _case(kind, chunk=chunk, doc=int(chunk * rng.uniform(2.2, 4.2 if kind == "layer" else 16.0)), budget=budget,
                 instr=_log(rng, 6, 256), **common)
    if kind == "document":
        mode = rng.choice(["instr", "instr", "shared", "dual", "standard"])
        case.update(mode=mode, per_layer=rng.random() < 0.25)
        if mode in ("dual", "standard"):
            case["paper_order"] = rng.random() < 0.5
        else:
            case["accumulated"] = rng.random() < 0.25
        if mode != "standard":
            case["shift"] = rng.random() < 0.25
    while work(case)["flops"] > most or work(case)["bytes"] > 8e9:
        if case["layers"] > 1:
            case["layers"] = case["layers"] * 2 // 3
        elif case["batch"] > 1:
            case["batch"] -= 1
        elif case["doc"] > 3 * case["chunk"]:
            case["doc"] = case["doc"] * 3 // 4
        else:
            case["chunk"] = case["chunk"] * 3 // 4
            case["budget"] = max(32, case["budget"] * 3 // 4)
            case["doc"] = case["doc"] * 3 // 4
    return case


def _chunks(case):
    return [(lo, min(case["doc"], lo + case["chunk"])) for lo in range(0, case["doc"], case["chunk"])]


def _config(case):
    dtype = api.F32 if case["dtype"] == "f32" else api.BF16
    shape = dict(batch=case["batch"], layers=case["layers"], q_heads=case["q_heads"], kv_heads=case["kv_heads"],
                 head_dim=case["head_dim"], dtype=dtype)
    if case["kind"] == "decode":
        return api.Config(chunk_len=32, budget=case["states"], instr_len=32,
                          cache_capacity=case["states"] + ANSWER_ROWS, **shape)
    shape.update(chunk_len=case["chunk"], budget=case["budget"], instr_len=case["instr"])
    if case["kind"] == "layer":
        return api.Config(**shape)
    held = case["chunk"] if case["paper_order"] else 0
    return api.Config(cache_mode=_MODES[case["mode"]], budget_lm=case["budget"] if case["mode"] == "dual" else 0,
                      select_mode=api.SELECT_PER_LAYER if case["per_layer"] else api.SELECT_PER_KV_HEAD,
                      lm_ordering=api.LM_EVICT_THEN_APPEND if case["paper_order"] else api.LM_SCORE_AFTER_APPEND,
                      score_mode=api.SCORE_ACCUMULATED if case["accumulated"] else api.SCORE_PER_STEP,
                      position_shift=int(case["shift"]), cache_capacity=case["budget"] + held + ANSWER_ROWS, **shape)


class _Inputs:
    """Seeded tensors of one case on the GPU."""

    def __init__(self, cfg, seed):
        self.cfg, self.gen = cfg, torch.Generator(device="cuda").manual_seed(seed)
        self.channel = cfg.head_dim // 2 - 1  # the lowest rotary frequency: importance hardly moves with position

    def _normal(self, *shape):
        return torch.randn(shape, generator=self.gen, dtype=self.cfg.torch_dtype, device="cuda")

    def queries(self, heads, rows, *lead):
        q = self._normal(*lead, self.cfg.batch, self.cfg.layers, heads, rows, self.cfg.head_dim)
        q[..., self.channel] = 4.0
        return q

    def keys(self, rows):
        k = self._normal(self.cfg.batch, self.cfg.layers, self.cfg.kv_heads, rows, self.cfg.head_dim)
        importance = k[..., self.channel] * (self.cfg.head_dim ** 0.5 / 4.0)  # logit part ~ N(0, 1) for every query
        k *= 0.35                                                            # the part that depends on the query
        boost = torch.rand((self.cfg.batch, 1, 1, rows), generator=self.gen, device="cuda") < 0.02
        boost[..., :4] = True
        k[..., self.channel] = importance + boost * (2.0 * self.cfg.head_dim ** 0.5 / 4.0)
        return k

    def values(self, rows):
        return self._normal(self.cfg.batch, self.cfg.layers, self.cfg.kv_heads, rows, self.cfg.head_dim)

    def token(self):
        return self.queries(self.cfg.q_heads, 1), self.keys(1), self.values(1)


def prepare(case, seed):
    cfg = _config(case)
    make = _Inputs(cfg, seed)
    state = {"kind": case["kind"], "cfg": cfg, "workspace": api.alloc_workspace(cfg)}
    if case["kind"] == "decode":
        rows = cfg.cache_capacity
        state.update(k_cache=make.keys(rows), v_cache=make.values(rows), states=case["states"],
                     tokens=[make.token() for _ in range(case["tokens"])])
        return state
    chunks = _chunks(case)
    if case["kind"] == "layer":
        state["chunks"] = [(make.queries(cfg.q_heads, hi - lo), make.keys(hi - lo), make.values(hi - lo),
                            make.queries(cfg.q_heads, cfg.instr_len)) for lo, hi in chunks]
        cache = (cfg.batch, cfg.layers, cfg.kv_heads, cfg.cache_capacity, cfg.head_dim)
        state["caches"] = [[torch.zeros(cache, dtype=cfg.torch_dtype, device="cuda") for _ in range(2)] for _ in range(2)]
        return state
    q, k, v = make.queries(cfg.q_heads, case["doc"]), make.keys(case["doc"]), make.values(case["doc"])
    qi = make.queries(cfg.q_heads, cfg.instr_len, len(chunks))
    out = torch.empty_like(q)
    state.update(tensors=(q, k, v, qi), out=out, doc=api.resident_doc(cfg, q, k, v, qi, out), q_final=qi[-1],
                 caches=api.DocumentState.allocate(cfg), token=make.token())
    return state


def _run_document(s):
    cfg, caches = s["cfg"], s["caches"]
    caches.cache_len = caches.cache_len_lm = caches.buffer_index = caches.buffer_index_lm = 0
    api.citrus_process_document(cfg, caches, s["workspace"], doc=s["doc"])
    now, kept = caches.buffer_index, caches.cache_len
    if cfg.cache_mode == api.CACHE_STANDARD:  # the instruction evicts once more before the answer
        kept = api.citrus_evict_cache(cfg, s["q_final"], caches.k_cache[now], caches.v_cache[now], kept, cfg.budget,
                                      caches.k_cache[now ^ 1], caches.v_cache[now ^ 1], workspace=s["workspace"])
        now ^= 1
    q, k, v = s["token"]
    first = api.citrus_decode_step(cfg, q, k, v, caches.k_cache[now], caches.v_cache[now], kept, workspace=s["workspace"])
    return {"out": s["out"], "first_token": first}


def _run_layer(s):
    cfg, ws, kept, now = s["cfg"], s["workspace"], 0, 0
    outs, scores = [], []
    for i, (q, k, v, qi) in enumerate(s["chunks"]):
        (kc, vc), (k_new, v_new) = s["caches"][now], s["caches"][now ^ 1]
        outs.append(api.citrus_chunk_attn(cfg, q, kc, vc, kept, k, v, workspace=ws))
        score = api.citrus_instr_score(cfg, qi, kc, kept, k, workspace=ws)
        if i == 0:  # later candidates are the survivors of a selection
            scores.append(score)
        idx = api.citrus_topk_select(cfg, score, cfg.budget)
        m = min(cfg.budget, kept + k.shape[3])
        api.citrus_kv_compact(cfg, kc, vc, kept, k, v, idx, m, k_new, v_new)
        kept, now = m, now ^ 1
    return {"out": outs, "score": scores}


def _run_decode(s):
    outs = [api.citrus_decode_step(s["cfg"], q, k, v, s["k_cache"], s["v_cache"], s["states"] + i, workspace=s["workspace"])
            for i, (q, k, v) in enumerate(s["tokens"])]
    return {"out": outs, "k_cache": s["k_cache"], "v_cache": s["v_cache"]}


def run(state):
    return {"document": _run_document, "layer": _run_layer, "decode": _run_decode}[state["kind"]](state)


def work(case):
    """Every input read once and every output written once; causal attention over [cache ; chunk] (two products), the
    instruction's scores (one product per instruction row and candidate), one token."""
    d, esize = case["head_dim"], 4 if case["dtype"] == "f32" else 2
    units, hq, hkv = case["batch"] * case["layers"], case["q_heads"], case["kv_heads"]
    if case["kind"] == "decode":
        rows = sum(case["states"] + i + 1 for i in range(case["tokens"]))
        return {"bytes": units * d * esize * (2 * hkv * rows + case["tokens"] * (2 * hq + 2 * hkv)),
                "flops": 4.0 * units * d * hq * rows}
    chunks = _chunks(case)
    standard = case.get("mode") == "standard"
    instr_rows = case["instr"] * (1 if standard else len(chunks))
    flops, cached, scored = 0.0, 0, 0  # states the chunk attends over; states the instruction's cache holds
    for lo, hi in chunks:
        c = hi - lo
        flops += 4.0 * d * hq * (c * cached + c * (c + 1) / 2)
        if not standard:
            flops += 2.0 * d * hq * case["instr"] * (scored + c)
        scored = min(case["budget"], scored + c)
        cached = min(cached, case["budget"]) + c if case.get("paper_order") else min(case["budget"], cached + c)
    return {"bytes": units * d * esize * (2 * hq * case["doc"] + 2 * hkv * case["doc"] + hq * instr_rows),
            "flops": units * flops}


def tolerance(case):
    """bf16 results carry bf16's rounding; where a selection lies in between, two states whose scores differ by less
    than the scores' own rounding may trade places, which moves an output by about one state's weight.  f32: the
    rounding of 32-bit sums."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 1e-2} if case["kind"] == "decode" else {"rel": 2e-2, "max": 0.5}
