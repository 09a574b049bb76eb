"""Host side of the library without a GPU: which kernels a call launches, with which grids and LDS, and what is left when a
launch fails.  The calls run in a child process in which fake_hip.cpp stands in front of the HIP runtime; nothing reaches a
device.  This file is the child's program too."""

import ctypes as C
import inspect
import json
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


# ---- in the child ----
class Fake:
    """What the binding reads of a tensor: an address and strides (those of a dense one)."""

    def __init__(self, *shape, at=1 << 20, strides=None):
        self.shape, self.at = shape, at
        self.strides = strides or tuple(_product(shape[i + 1:]) for i in range(len(shape)))

    def stride(self, i=None):
        return self.strides if i is None else self.strides[i]

    def dim(self):
        return len(self.shape)

    def __getitem__(self, i):  # of the first axis
        return Fake(*self.shape[1:], at=self.at + i * self.strides[0] * 4, strides=self.strides[1:])

    def data_ptr(self):
        return self.at

    def numel(self):
        return _product(self.shape)


def _product(xs):
    p = 1
    for x in xs:
        p *= x
    return p


class Recorder:
    def __init__(self, lib, lib_under_test=None):
        self.lib, self.lib_under_test = lib, lib_under_test
        lib.fake_log.restype = C.c_char_p

    def __call__(self, call, fail_at=-1):
        """The launches of a call: [kernel, grid, workgroup, dynamic LDS], and ["lds", bytes, kernel] for a raised limit."""
        self.lib.fake_reset(fail_at)
        call()
        out = []
        for line in self.lib.fake_log().decode().splitlines():
            if line.startswith("lds "):
                _, size, name = line.split(" ", 2)
                out.append(["lds", int(size), short(name)])
            else:
                grid, block, shared, name = re.fullmatch(r"launch \[(.*?)\] \[(.*?)\] (\d+) (.*)", line).groups()
                out.append([short(name), [int(x) for x in grid.split()], [int(x) for x in block.split()], int(shared)])
        return out


def short(name):
    """`evict_kernel<6, 1024, ...>` of a demangled signature."""
    name = re.sub(r"^void ", "", name).replace("citrus::(anonymous namespace)::", "")
    return name[:name.rindex("(")] if name.endswith(")") else name


def workspace(api, cfg, spare=0):
    return Fake(api.workspace_bytes(cfg) + spare, at=1 << 30)


# ---- in the test ----
def in_child(body, tmp_path, **kw):
    """Runs `body(api, launches, **kw)` of this file in a child and returns what it returns."""
    shim = str(tmp_path / "fake_hip.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", shim, os.path.join(ROOT, "tests", "fake_hip.cpp")])
    done = subprocess.run([sys.executable, os.path.abspath(__file__), shim, body.__name__, json.dumps(kw)], cwd=ROOT,
                          stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=300)
    assert done.returncode == 0, done.stderr[-3000:]
    return json.loads(done.stdout.splitlines()[-1])


def f32_of_many_heads(api, launches):
    """The most heads a configuration may have: 65535 layers of 129 heads, one query row each."""
    L, H = 65535, 129
    cfg = api.Config(batch=1, layers=L, q_heads=H, kv_heads=H, head_dim=64, chunk_len=1, budget=4, instr_len=1, dtype=api.F32)
    q, cache, ws = Fake(1, L, H, 1, 64), Fake(1, L, H, 4, 64, at=1 << 21), workspace(api, cfg)
    state = api.DocumentState([cache, Fake(1, L, H, 4, 64, at=1 << 22)], [cache, Fake(1, L, H, 4, 64, at=1 << 22)])
    doc = api.resident_doc(cfg, q, q, q, Fake(1, 1, L, H, 1, 64), q)
    return [launches(lambda: api.citrus_chunk_attn(cfg, q, cache, cache, 3, q, q, out=q, stream=0)),
            launches(lambda: api.citrus_decode_step(cfg, q, q, q, cache, cache, 3, out=q, workspace=ws, stream=0)),
            launches(lambda: api.citrus_instr_score(cfg, q, cache, 3, q, score=q, workspace=ws, stream=0)),
            launches(lambda: api.citrus_process_document(cfg, state, ws, doc=doc, stream=0))]


def test_f32_launches_of_many_heads_stay_within_a_grid(tmp_path):
    """8.45 million heads of a row each: more than 2^32 work-items if the grid were one-dimensional."""
    attn, decode, score, document = in_child(f32_of_many_heads, tmp_path)
    names = lambda launches: [x[0] for x in launches if x[0] != "lds"]
    assert names(attn) == ["attn_f32_kernel<64, 1>"] and names(decode) == ["attn_f32_kernel<64, 1>", "compact_kernel"]
    assert names(score) == ["score_f32_kernel<64>"] and names(document)[:2] == ["attn_f32_kernel<64, 1>", "score_f32_kernel<64>"]
    for launch in attn + decode + score + document:
        if launch[0] in ("attn_f32_kernel<64, 1>", "score_f32_kernel<64>"):
            assert _product(launch[1]) == 65535 * 129


def evictions_of_large_budgets(api, launches, budgets):
    launches.lib.fake_compute_units(32)  # a part of the chip: one workgroup holds all that a unit keeps
    out = []
    for k in budgets:
        L, H, n, d = 5, 8, 6144, 64
        cfg = api.Config(batch=1, layers=L, q_heads=H, kv_heads=H, head_dim=d, chunk_len=8, budget=k, instr_len=2, cache_capacity=n)
        q, cache, new, ws = Fake(1, L, H, 2, d), Fake(1, L, H, n, d), Fake(1, L, H, k, d, at=1 << 22), workspace(api, cfg)
        out += launches(lambda: api.citrus_evict_cache(cfg, q, cache, cache, n, k, new, new, workspace=ws, stream=0))
    return out


def test_a_kernel_asks_for_one_lds_limit_whatever_the_budget(tmp_path):
    """Two threads that ask for different limits could lower each other's: the smaller may arrive last."""
    calls = in_child(evictions_of_large_budgets, tmp_path, budgets=[5400, 5700, 6100])
    asked = [x for x in calls if x[0] == "lds" and "evict_kernel" in x[2]]
    used = [x[3] for x in calls if "evict_kernel" in x[0]]
    assert sorted(set(used)) == [4 * k for k in (5400, 5700, 6100)]
    assert len({x[1] for x in asked}) == 1 and asked[0][1] >= max(used)
    assert len({x[2] for x in asked}) == len(asked)  # once per kernel


def two_caches_with_a_failing_launch(api, launches):
    """A document of two chunks; the launch that fails, and what the call then leaves."""
    H, d, c, k = 4, 64, 32, 48
    cfg = api.Config(batch=1, layers=1, q_heads=H, kv_heads=H, head_dim=d, chunk_len=c, budget=k, budget_lm=k, instr_len=8,
                     cache_mode=api.CACHE_DUAL)
    q, cache, ws = Fake(1, 1, H, 2 * c, d), lambda i: Fake(1, 1, H, k, d, at=(4 + i) << 20), workspace(api, cfg)
    doc = api.resident_doc(cfg, q, q, q, Fake(2, 1, 1, H, 8, d), q)
    out = []
    for fail_at in range(-1, 8):
        state = api.DocumentState([cache(0), cache(1)], [cache(2), cache(3)], k_cache_lm=[cache(4), cache(5)], v_cache_lm=[cache(6), cache(7)])

        def call():
            try:
                api.citrus_process_document(cfg, state, ws, doc=doc, stream=0)
            except api.CitrusError as e:
                assert e.status == 5
        names = [x[0] for x in launches(call, fail_at) if x[0] != "lds"]
        out.append([names, state.cache_len, state.buffer_index, state.cache_len_lm, state.buffer_index_lm])
    return out


def test_a_failed_step_leaves_both_caches_in_front_of_it(tmp_path):
    """The caches' evictions share the step's last launch.  A cache whose eviction was not launched has not moved on: its other
    buffer holds nothing."""
    whole, *failing = in_child(two_caches_with_a_failing_launch, tmp_path)
    per_step = len(whole[0]) // 2
    assert whole[0][per_step - 1].startswith("evict_kernel") and whole[1:] == [48, 0, 48, 0]
    assert len(failing) == 2 * per_step
    for fail_at, (names, *state) in enumerate(failing):
        assert names == whole[0][:fail_at]
        assert state == ([0, 0, 0, 0] if fail_at < per_step else [32, 1, 32, 1]), fail_at


def scores(api, launches, shapes):
    return [scores_of_one_shape(api, launches, *shape) for shape in shapes]


def scores_of_one_shape(api, launches, L, Hq, Hkv, rows, n, head_dim):
    """The same scores through every entry point that computes them, with workspaces of several sizes."""
    q, cache, new = Fake(1, L, Hq, rows, head_dim), Fake(1, L, Hkv, n, head_dim), Fake(1, L, Hkv, 1, head_dim, at=1 << 22)
    chunk = Fake(1, L, Hkv, n - 1, head_dim)
    out = []
    for capacity, instr_len in ((n, rows), (4 * n, rows), (n, 3 * rows), (n, rows + 700)):
        cfg = api.Config(batch=1, layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=head_dim, chunk_len=n, budget=1, instr_len=instr_len,
                         cache_capacity=capacity)
        ws = workspace(api, cfg)
        out += [launches(lambda: api.citrus_cache_score(cfg, q, cache, n, score=q, workspace=ws, stream=0)),
                launches(lambda: api.citrus_evict_cache(cfg, q, cache, cache, n, 1, new, new, workspace=ws, stream=0))]
        if instr_len == rows:
            out.append(launches(lambda: api.citrus_instr_score(cfg, q, cache, 1, chunk, score=q, workspace=ws, stream=0)))
        try:
            out.append(launches(lambda: api.citrus_evict_cache_static(cfg, q, cache, cache, n, 1, new, new, stream=0)))
        except api.CitrusError as e:
            assert e.status == 4  # more than the static array
    return [[x for x in calls if x[0] != "lds" and not x[0].startswith(("evict_kernel", "strip_sum_kernel"))] for calls in out]


SHAPES = [  # layers, query heads, KV heads, rows, candidates
    (1, 64, 2, 128, 512), (1, 64, 2, 128, 513), (1, 64, 2, 128, 640),  # 4096 rows per KV head: 16 floats of scratch a row hold 512 keys
    (4, 32, 2, 128, 1024), (4, 32, 2, 128, 1025), (4, 32, 2, 128, 1280),  # 2048 rows, strips of 64
    (32, 32, 32, 64, 1280), (32, 32, 8, 64, 1280), (80, 8, 8, 40, 90), (1, 32, 8, 64, 2560), (16, 32, 8, 128, 2000)]


@pytest.mark.parametrize("head_dim", [64, 128])
def test_the_scorer_follows_from_the_call_alone(head_dim, tmp_path):
    """Not from the size of the scratch behind it: the entry points promise the same bits."""
    shapes = [[*shape, head_dim] for shape in SHAPES]
    for shape, (first, *others) in zip(shapes, in_child(scores, tmp_path, shapes=shapes)):
        assert len(first) >= 1 and len(others) >= 9
        for calls in others:
            assert calls == first, shape


def evictions(api, launches, shapes):
    out = []
    for L, head_dim, n, k in shapes:
        H = 8
        cfg = api.Config(batch=1, layers=L, q_heads=H, kv_heads=H, head_dim=head_dim, chunk_len=8, budget=k, instr_len=1, cache_capacity=n)
        q, cache, new, ws = Fake(1, L, H, 1, head_dim), Fake(1, L, H, n, head_dim), Fake(1, L, H, k, head_dim, at=1 << 22), workspace(api, cfg)
        calls = launches(lambda: api.citrus_evict_cache(cfg, q, cache, cache, n, k, new, new, workspace=ws, stream=0))
        out.append([x[0].split("<")[0] for x in calls if x[0] != "lds"])
    return out


def test_evictions_that_memory_bounds_are_two_launches(tmp_path):
    shapes = {(32, 128, 1280, 765): 1, (32, 128, 1280, 768): 2,    # 96 MB of keys and values
              (32, 64, 2048, 1536): 1, (32, 64, 2049, 1536): 2,    # rows of 128 bytes: only with 1024 threads
              (128, 64, 2560, 31): 1, (129, 64, 2560, 31): 2,      # four units per compute unit
              (1, 128, 6144, 4096): 1, (1, 128, 6145, 4096): 2}
    for (shape, count), names in zip(shapes.items(), in_child(evictions, tmp_path, shapes=[list(x) for x in shapes])):
        assert names[-count:] == (["evict_kernel"] if count == 1 else ["topk_regs_kernel" if shape[2] <= 6144 else "topk_kernel",
                                                                       "compact_kernel"]), shape


def strip_cases(api, launches, cases):
    out = []
    for L, Hq, Hkv, rows, n_c, c, head_dim in cases:
        cfg = api.Config(batch=1, layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=head_dim, chunk_len=c, budget=n_c + 3, instr_len=rows)
        q, k, ws = Fake(1, L, Hq, rows, head_dim), Fake(1, L, Hkv, n_c + 3, head_dim), workspace(api, cfg)
        calls = launches(lambda: api.citrus_instr_score(cfg, q, k, n_c, Fake(1, L, Hkv, c, head_dim), score=q, workspace=ws, stream=0))
        out.append("S" if any("instr_strip_kernel" in x[0] for x in calls) else "T")
    return out


def test_the_strip_tests_run_the_kernel_they_name(tmp_path):
    from test_gpu_strips import CASES
    cases = [[*case[:6], head_dim] for case in CASES for head_dim in (64, 128)]
    ran = in_child(strip_cases, tmp_path, cases=cases)
    assert [a + b for a, b in zip(ran[::2], ran[1::2])] == [case[6] for case in CASES]


def one_launch_steps(api, launches, cases):
    """Documents of three chunks: the launches behind which a step ends."""
    out = []
    for f32, G, Hkv, d, c, k, rows in cases:
        cfg = api.Config(batch=1, layers=1, q_heads=G * Hkv, kv_heads=Hkv, head_dim=d, chunk_len=c, budget=k, instr_len=rows,
                         dtype=api.F32 if f32 else api.BF16)
        q, cache = Fake(1, 1, G * Hkv, 3 * c, d), lambda i: Fake(1, 1, Hkv, k, d, at=(4 + i) << 20)
        doc = api.resident_doc(cfg, q, Fake(1, 1, Hkv, 3 * c, d), Fake(1, 1, Hkv, 3 * c, d), Fake(3, 1, 1, G * Hkv, rows, d), q)
        state = api.DocumentState([cache(0), cache(1)], [cache(2), cache(3)])
        calls = launches(lambda: api.citrus_process_document(cfg, state, workspace(api, cfg), doc=doc, stream=0))
        out.append([x[0].split("<")[0] for x in calls if x[0] != "lds"])
    return out


def test_steps_that_are_one_launch(tmp_path):
    """The counters of a unit's workgroups are cleared once per call, in front of the first step that counts."""
    bf16, f32, clear, evict = "attn_score_kernel", "attn_score_f32_kernel", "clear_tickets_kernel", "evict_kernel"
    attn, strips = "attn_pipe_kernel", "instr_strip_kernel"
    cases = {(0, 4, 8, 128, 512, 768, 64): [bf16, clear, bf16, bf16],       # the first step keeps all of its states
             (0, 4, 8, 128, 512, 400, 64): [clear, bf16, bf16, bf16],
             (0, 4, 8, 128, 512, 2048, 64): [bf16, bf16, bf16],
             (0, 1, 8, 128, 32, 30, 32): [bf16, bf16, bf16],                # one strip per unit: nothing to count
             (0, 4, 8, 128, 32, 40, 64): [bf16, clear, bf16, bf16],
             (0, 4, 32, 128, 64, 70, 96): [bf16, clear, bf16, bf16],        # 384 strips
             (0, 4, 33, 128, 64, 70, 96): [attn, evict] + [attn, strips, evict] * 2,  # 396
             (0, 4, 8, 128, 1024, 800, 8): [bf16, bf16, bf16],              # 256 workgroups of the attention
             (0, 4, 8, 128, 1025, 800, 8): [attn, strips, evict] * 3,
             (1, 4, 1, 64, 32, 64, 8): [f32, f32, f32],
             (1, 2, 1, 128, 100, 128, 8): [f32, f32, f32],                  # 128 KB of a unit stay
             (1, 2, 1, 128, 100, 129, 8): [f32, f32, evict, f32, evict]}
    for (case, want), got in zip(cases.items(), in_child(one_launch_steps, tmp_path, cases=[list(c) for c in cases])):
        assert got == want, case


def merged_steps(api, launches, shapes):
    """Documents of three chunks whose last step evicts, as they run and with every event asked for (launches apart): grids of the
    step's attention and score launches, what the score's columns need and what the block behind them holds, in floats."""
    class Dims(C.Structure):
        _fields_ = [(x, C.c_int) for x in ("B", "L", "Hq", "Hkv", "G", "D")] + [("scale", C.c_float)]

    block = launches.lib_under_test._ZN6citrus33instr_score_mfma_workspace_floatsERKNS_4DimsEii
    block.restype, block.argtypes = C.c_size_t, [C.POINTER(Dims), C.c_int, C.c_int]
    out = []
    for L, Hq, Hkv, d, c, k, rows in shapes:
        cfg = api.Config(batch=1, layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=d, chunk_len=c, budget=k, instr_len=rows)
        q, kv = Fake(1, L, Hq, 3 * c, d), Fake(1, L, Hkv, 3 * c, d)
        cache = lambda i: Fake(1, L, Hkv, k, d, at=(4 + i) << 20)
        doc = api.resident_doc(cfg, q, kv, kv, Fake(3, 1, L, Hq, rows, d), q)

        def last_step(events):
            state = api.DocumentState([cache(0), cache(1)], [cache(2), cache(3)])
            api.citrus_process_document(cfg, state, workspace(api, cfg), doc=doc, max_chunks=2, stream=0)
            calls = launches(lambda: api.citrus_process_document(cfg, state, workspace(api, cfg), doc=doc, first_chunk=2, stream=0,
                                                                 phase_events=events))
            grids = lambda name: [_product(x[1]) for x in calls if x[0].startswith(name)]
            return grids("attn_score_kernel<"), grids("attn_pipe_kernel<"), grids("instr_strip_kernel<")

        merged = last_step(None)[0]
        if not merged:
            continue
        _, attn, strips = last_step((C.c_void_p * (3 * api.binding.EVENTS_PER_STEP))(*[1] * (3 * api.binding.EVENTS_PER_STEP)))
        held = block(Dims(1, L, Hq, Hkv, Hq // Hkv, d, 1.0), rows, cfg.cache_capacity + c)
        out.append([[L, Hq, Hkv, d, c, k, rows], merged, attn, strips, min(2 * c, k) + c, held])
    return out


def test_a_merged_step_takes_the_strips_of_the_score_alone(tmp_path):
    """As many, so of the same height (the same bits), and their columns fit the scratch block, which is checked for those."""
    import random
    rng = random.Random(3)
    shapes = [(1, 64, 8, 128, 512, 768, rows) for rows in (128, 160, 192)]
    shapes += [(1, 40, 5, 128, 512, 768, 256), (1, 32, 8, 128, 512, 768, 320), (1, 56, 8, 128, 300, 700, 200),
               (1, 48, 6, 64, 256, 700, 256), (5, 8, 1, 128, 500, 500, 256), (1, 128, 32, 128, 64, 70, 96)]
    crowded = len(shapes)
    while len(shapes) < 300:
        L, G, Hkv, d = rng.choice([1, 2, 5, 16]), rng.choice([1, 2, 3, 4, 7, 8]), rng.choice([1, 2, 4, 8, 16, 32]), rng.choice([64, 128])
        c, rows = rng.randint(16, 600), rng.randint(1, 320)
        shapes.append((L, G * Hkv, Hkv, d, c, rng.randint(c // 2, 2 * c), rows))
    steps = in_child(merged_steps, tmp_path, shapes=shapes)
    assert len(steps) >= 60 and all(list(shape) in [x[0] for x in steps] for shape in shapes[:crowded])
    for shape, merged, attn, strips, n, held in steps:
        L, Hkv = shape[0], shape[2]
        assert merged == [attn[0] + strips[0]], shape
        assert strips[0] == L * Hkv or strips[0] * n <= held, shape


def one_launch_steps_of_a_provider(api, launches):
    G, Hkv, d, c, k, rows = 4, 8, 128, 32, 40, 64
    cfg = api.Config(batch=1, layers=1, q_heads=G * Hkv, kv_heads=Hkv, head_dim=d, chunk_len=c, budget=k, instr_len=rows)
    q, kv, qi, cache = Fake(1, 1, G * Hkv, c, d), Fake(1, 1, Hkv, c, d), Fake(1, 1, G * Hkv, rows, d), lambda i: Fake(1, 1, Hkv, k, d, at=(4 + i) << 20)
    state = api.DocumentState([cache(0), cache(1)], [cache(2), cache(3)])

    def provider(i, io):
        if i == 4:
            return 1
        io.q, io.out, io.q_instr, io.chunk_len = api.binding.tensor(q), api.binding.tensor(q), api.binding.tensor(qi), c
        io.k, io.v = api.binding.tensor(kv), api.binding.tensor(kv)
        return 0
    calls = launches(lambda: api.citrus_process_document(cfg, state, workspace(api, cfg), provider=provider, stream=0))
    return [x[0].split("<")[0] for x in calls if x[0] != "lds"]


def test_counters_are_cleared_behind_a_provider(tmp_path):
    """What a provider enqueues may use the call's workspace: the counters of a step are cleared behind it."""
    step = ["clear_tickets_kernel", "attn_score_kernel"]
    assert in_child(one_launch_steps_of_a_provider, tmp_path) == step[1:] + step * 3  # the first step keeps all: nothing is counted


def attention_grids(api, launches, shapes, head_dim):
    out = []
    for L, Hq, Hkv, c in shapes:
        cfg = api.Config(batch=1, layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=head_dim, chunk_len=c, budget=c, instr_len=4)
        q, kv = Fake(1, L, Hq, c, head_dim), Fake(1, L, Hkv, c, head_dim)
        calls = launches(lambda: api.citrus_chunk_attn(cfg, q, kv, kv, c, kv, kv, out=q, stream=0))
        out += [[x[0], _product(x[1])] for x in calls if x[0].startswith("attn_pipe_kernel")]
    return out


def test_row_blocks_are_paired_where_pairs_take_no_more_turns(tmp_path):
    """Pairs are formed within a group of heads: with an odd number of row blocks there, one is left over in each."""
    grids = {(8, 32, 8, 512): 256,   # 8 row blocks a head group, 512 in all: pairs fill the chip once
             (9, 32, 8, 512): 576,   # 288 pairs would take two turns of two, single blocks take three
             (6, 64, 8, 300): 480,   # 5 row blocks of each of two head groups: 288 workgroups if they were paired
             (17, 64, 8, 576): 2448, # 9 of two
             (20, 64, 4, 161): 960,  # 3 of four
             (3, 48, 4, 598): 180,   # 29 row blocks that mix heads: 14 pairs and one fit the chip side by side
             (32, 8, 2, 312): 192,   # 5 row blocks
             (2, 32, 8, 1063): 272,  # 17: 144 workgroups would leave too much of the chip idle
             (2, 64, 8, 1063): 544}  # 17 of two head groups: 288
    got = in_child(attention_grids, tmp_path, shapes=[list(s) for s in grids], head_dim=128)
    assert [grid for _, grid in got] == list(grids.values())


def test_single_row_blocks_of_head_dim_64_are_three_to_a_compute_unit(tmp_path):
    """Beyond the compute units pairs of eight waves, or single blocks of four; never single blocks of eight."""
    pairs, three = "attn_pipe_kernel<64, 8, false, 2>", "attn_pipe_kernel<64, 4, false, 3>"
    launches = {(8, 32, 8, 512): [pairs, 256], (9, 32, 8, 512): [three, 1152],
                (48, 16, 8, 641): [three, 4224],  # 2304 blocks of eight waves take nine turns, their pairs ten
                (11, 16, 8, 567): [three, 792], (32, 8, 8, 256): [pairs, 256]}
    assert in_child(attention_grids, tmp_path, shapes=[list(s) for s in launches], head_dim=64) == list(launches.values())


def column_sums(api, launches, shapes):
    out = []
    for causal, L, Hq, Hkv, c, n_c, d in shapes:
        cfg = api.Config(batch=1, layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=d, chunk_len=c, budget=n_c, instr_len=4)
        q, kv, cache, ws = Fake(1, L, Hq, c, d), Fake(1, L, Hkv, c, d), Fake(1, L, Hkv, n_c, d), workspace(api, cfg)
        if causal:
            calls = launches(lambda: api.citrus_chunk_attn(cfg, q, cache, cache, n_c, kv, kv, out=q, lm_score=q, workspace=ws, stream=0))
        else:
            calls = launches(lambda: api.citrus_cache_score(cfg, q, cache, n_c, lse_cache=q, score=q, workspace=ws, stream=0))
        out += [x[0] for x in calls if x[0].startswith("colsum")]
    return out


def test_column_sums_kernels(tmp_path):
    """Where the one of 64 keys a wave is slower, that of 32 keys is taken, whatever the number of rows."""
    many, whole, pipelined = "colsum_many_kernel<%d, false", "colsum_many_kernel<%d, true", "colsum_mfma_kernel<%d"
    kernels = {(0, 3, 8, 8, 29, 59, 128): many % 128, (0, 1, 1, 1, 96, 2000, 128): many % 128, (0, 1, 1, 1, 97, 200, 128): pipelined % 128,
               (0, 1, 1, 1, 192, 128, 64): many % 64, (0, 1, 1, 1, 192, 129, 64): pipelined % 64,
               (1, 128, 64, 16, 200, 300, 64): many % 64, (1, 64, 32, 8, 384, 300, 64): whole % 64, (1, 1, 32, 8, 200, 1100, 64): pipelined % 64,
               (1, 96, 32, 8, 1400, 400, 64): many % 64, (1, 24, 32, 8, 1500, 500, 64): pipelined % 64, (1, 64, 4, 2, 275, 535, 64): many % 64,
               (1, 96, 32, 8, 400, 768, 128): many % 128, (1, 64, 56, 8, 400, 1500, 128): pipelined % 128, (1, 64, 24, 8, 200, 40, 128): many % 128,
               (1, 24, 64, 8, 250, 300, 128): pipelined % 128, (1, 64, 32, 8, 512, 768, 128): whole % 128,
               (0, 96, 16, 8, 300, 768, 64): many % 64, (0, 128, 16, 8, 250, 300, 64): pipelined % 64, (0, 96, 32, 8, 512, 200, 128): whole % 128,
               (0, 128, 8, 8, 512, 1024, 128): whole % 128, (0, 64, 24, 8, 700, 700, 128): pipelined % 128,
               (1, 24, 16, 8, 211, 2500, 64): many % 64, (0, 48, 4, 4, 546, 2000, 64): many % 64, (1, 1, 16, 8, 211, 2500, 64): pipelined % 64,
               (1, 48, 4, 4, 148, 2500, 128): many % 128, (0, 48, 8, 4, 600, 2000, 128): pipelined % 128}
    got = in_child(column_sums, tmp_path, shapes=[list(s) for s in kernels])
    assert len(got) == len(kernels)
    for (shape, want), kernel in zip(kernels.items(), got):
        assert kernel.startswith(want) and (kernel.endswith("true>" if shape[0] else "false>") or want == pipelined % shape[-1]), shape


def f32_attention(api, launches, shapes):
    out = []
    for H, c, n_c, d in shapes:
        cfg = api.Config(batch=1, layers=1, q_heads=H, kv_heads=H, head_dim=d, chunk_len=c, budget=n_c, instr_len=4, dtype=api.F32)
        q, cache = Fake(1, 1, H, c, d), Fake(1, 1, H, n_c, d)
        calls = launches(lambda: api.citrus_chunk_attn(cfg, q, cache, cache, n_c, q, q, out=q, stream=0))
        out += [x[0] for x in calls if x[0] != "lds"]
    return out


def test_f32_waves_that_have_a_simd_each_keep_it(tmp_path):
    """512 workgroups of two waves: as many waves as the chip has SIMDs."""
    got = in_child(f32_attention, tmp_path, shapes=[[128, 55, 93, 128], [512, 10, 26, 128], [129, 55, 93, 128], [127, 55, 93, 128]])
    assert got == ["attn_f32_apart_kernel<128, 2>"] * 2 + ["attn_f32_kernel<128, 2>", "attn_f32_kernel<128, 8>"]


if __name__ == "__main__":
    fake = C.CDLL(sys.argv[1], C.RTLD_GLOBAL)  # before anything that loads the real runtime
    sys.path.insert(0, ROOT)
    import paper_2406_12018_amd as api_

    body_ = globals()[sys.argv[2]]
    assert inspect.isfunction(body_)
    print(json.dumps(body_(api_, Recorder(fake, api_.binding._lib()), **json.loads(sys.argv[3]))))
