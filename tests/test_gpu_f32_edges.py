"""The f32 kernels at the edges of their tiles (64 keys, 16 value rows, 32 query rows of a KV group, four rows per
workgroup), both head dimensions, against the same definitions in f64.  Bound 1e-5 relative: f32 sums over at most
300 states leave about sqrt(300) * 2^-24 = 1e-6, the exponential's f32 argument (|logit| < 30) 30 * 2^-24 = 2e-6."""

import pytest
import torch

import paper_2406_12018_amd as api

pytestmark = pytest.mark.gpu
DEV = "cuda"


def reference(q, k, v, cached):
    """causal outputs over [cached states ; chunk] of one layer, and the probabilities, in f64"""
    k, v, q = k.double(), v.double(), q.double()
    group, rows, n = q.shape[0] // k.shape[0], q.shape[1], k.shape[1]
    logits = q @ k.repeat_interleave(group, 0).transpose(-1, -2).contiguous() / q.shape[-1] ** 0.5
    seen = torch.arange(n)[None, :] <= cached + torch.arange(rows)[:, None]
    return torch.softmax(logits.masked_fill(~seen, -torch.inf), -1) @ v.repeat_interleave(group, 0)


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("cached,chunk,instr,group", [(0, 1, 1, 1), (15, 2, 3, 1), (16, 16, 11, 3), (47, 17, 32, 1),
                                                     (63, 65, 33, 1), (64, 66, 8, 4), (200, 100, 31, 7)])
def test_steps(cached, chunk, instr, group, head_dim):
    heads = 2
    cfg = api.Config(batch=1, layers=1, q_heads=heads * group, kv_heads=heads, head_dim=head_dim, dtype=api.F32,
                     chunk_len=chunk, budget=max(cached, 1), instr_len=instr, cache_capacity=max(cached, 1) + 1)
    g = torch.Generator().manual_seed(1000 * cached + chunk)
    rand = lambda h, rows: 1.5 * torch.randn((1, 1, h, rows, head_dim), generator=g)
    q, qi = rand(heads * group, chunk), rand(heads * group, instr)
    k_new, v_new = rand(heads, chunk), rand(heads, chunk)
    kc, vc = rand(heads, max(cached, 1) + 1), rand(heads, max(cached, 1) + 1)
    # an infinite value behind the last state a row sees must not reach the row
    last_v = v_new.clone()
    if chunk > 1:
        last_v[..., -1, :] = torch.inf
    ws = api.alloc_workspace(cfg)
    dev = lambda x: x.to(DEV)
    print(f"f32 cached {cached} chunk {chunk} instr {instr} group {group} d {head_dim}", flush=True)
    k_all = torch.cat([kc[0, 0, :, :cached], k_new[0, 0]], 1)
    v_all = torch.cat([vc[0, 0, :, :cached], v_new[0, 0]], 1)
    want = reference(q[0, 0], k_all, v_all, cached)
    for values, rows in ((v_new, chunk), (last_v, chunk - 1)):
        got = api.citrus_chunk_attn(cfg, dev(q), dev(kc), dev(vc), cached, dev(k_new), dev(values), workspace=ws)
        diff = (got[0, 0].cpu().double() - want)[:, :rows]
        assert rows == 0 or float(diff.norm() / want[:, :rows].norm()) < 1e-5

    score = api.citrus_instr_score(cfg, dev(qi), dev(kc), cached, dev(k_new), workspace=ws)
    logits = (qi[0, 0].double() @ k_all.double().repeat_interleave(group, 0).transpose(-1, -2).contiguous()
              / head_dim ** 0.5)
    want_score = torch.softmax(logits, -1).reshape(heads, group * instr, -1).sum(1)
    assert float((score[0, 0].cpu().double() - want_score).norm() / want_score.norm()) < 1e-5

    if cached:
        dk, dv = dev(kc), dev(vc)
        one = api.citrus_decode_step(cfg, dev(q[..., :1, :].contiguous()), dev(k_new[..., :1, :].contiguous()),
                                     dev(v_new[..., :1, :].contiguous()), dk, dv, cached, workspace=ws)
        diff = one[0, 0].cpu().double() - want[:, :1]
        assert float(diff.norm() / want[:, :1].norm()) < 1e-5
