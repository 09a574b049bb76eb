"""Selection at the sizes where the kernel instance changes (2048, 3072 and 6144 candidates, more units than compute units
or than two rounds of them) and around one row of 256 candidates, on scores that end the radix passes early, late and on ties: exactly the top k under (score descending,
position ascending), in ascending position."""

import pytest
import torch

import paper_2406_12018_amd as api

pytestmark = pytest.mark.gpu
DEV = "cuda"


def scores(kind, units, n):
    g = torch.Generator().manual_seed(n)
    x = torch.randn((units, n), generator=g)
    if kind == "spread":       # differing values over many octaves
        return torch.exp(3.0 * x)
    if kind == "close":        # differ in the lowest bits only: all four passes
        return 1.0 + torch.randperm(n, generator=g).float().expand(units, n) * 2.0 ** -23
    if kind == "ties":         # few values, both zeros among them
        return torch.round(x) * torch.where(x < 0.2, -1.0, 1.0)
    if kind == "equal":
        return torch.full((units, n), -0.75)
    return torch.where(x > 1.0, torch.inf, torch.where(x < -1.0, -torch.inf, x))  # "infinite"


def check(layers, heads, n, kind, per_layer):
    cfg = api.Config(batch=1, layers=layers, q_heads=heads, kv_heads=heads, head_dim=64, chunk_len=n, budget=n, instr_len=1,
                     select_mode=api.SELECT_PER_LAYER if per_layer else api.SELECT_PER_KV_HEAD)
    x = scores(kind, layers * heads, n).reshape(1, layers, heads, n)
    ranked = x
    if per_layer:  # the heads' scores in head order, in 32 bits
        ranked = x[:, :, 0]
        for g in range(1, heads):
            ranked = ranked + x[:, :, g]
        ranked = ranked.unsqueeze(2)
    order = torch.sort(ranked, dim=-1, descending=True, stable=True).indices
    for k in sorted({1, (n + 1) // 2, n - 1}):
        print(f"select {layers} layers {heads} heads n {n} k {k} {kind} per_layer {per_layer}", flush=True)
        want = torch.sort(order[..., :k], dim=-1).values.to(torch.int32)
        got = api.citrus_topk_select(cfg, x.to(DEV), k).cpu()
        assert torch.equal(got.reshape(want.shape), want)


@pytest.mark.parametrize("kind", ["spread", "close", "ties", "equal", "infinite"])
@pytest.mark.parametrize("n", [2, 63, 65, 255, 256, 257, 1280, 2047, 2048, 2049, 3072, 3073, 6144, 6145])
def test_selection(n, kind):
    check(2, 3, n, kind, per_layer=False)
    if kind != "infinite":  # inf - inf has no rank
        check(2, 3, n, kind, per_layer=True)


@pytest.mark.parametrize("kind", ["spread", "close", "ties", "equal"])
@pytest.mark.parametrize("layers,heads,n,per_layer", [
    (88, 3, 2049, False), (88, 3, 6144, False),                  # more units than compute units
    (520, 2, 2, True), (520, 3, 257, True), (520, 4, 2048, True),  # more than two rounds of them, short sums
    (520, 5, 2048, True), (520, 3, 2049, True), (520, 2, 2049, True), (520, 2, 3072, True), (1300, 2, 6144, True),  # longer ones
])
def test_selection_of_many_units(layers, heads, n, per_layer, kind):
    check(layers, heads, n, kind, per_layer)


@pytest.mark.parametrize("kind", ["spread", "close", "ties", "equal"])
@pytest.mark.parametrize("layers,heads,n,per_layer", [
    (1, 2, 511, False), (1, 2, 512, False), (1, 2, 513, False), (2, 1, 768, False), (2, 1, 769, False), (2, 1, 1281, False),
    (3, 2, 1023, True), (3, 2, 1024, True), (3, 2, 1025, True), (3, 2, 1536, True), (3, 2, 1537, True),
    (520, 2, 512, True), (520, 2, 513, True), (520, 3, 1281, True),    # short sums
    (1300, 2, 512, True), (1300, 2, 513, True), (1300, 3, 1280, True),  # of more than five units per compute unit
])
def test_selection_where_the_candidates_per_thread_and_the_radix_change(layers, heads, n, per_layer, kind):
    check(layers, heads, n, kind, per_layer)
