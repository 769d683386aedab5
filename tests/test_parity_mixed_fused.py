"""GPU: the decode step over the mixed cache takes the newest token's rows from its
arguments while the same launch writes them to the segment store.  With a store whose
unwritten slots hold NaN, for a newest token in the sink, in the window before and
after it wraps, in no segment (W = 0), and alone: the step's output has the bits of
decode_attn_mixed on the cache that it leaves behind, repeated steps agree, and the
written rows are the arguments'.  The same where the bf16 tokens have a launch of their
own (more than 8 query heads per KV head, S0 + W <= 256, more pairs than CUs)."""
import math

import numpy as np
import pytest
import torch

import paper_2605_17757_amd as ok
import workloads as W

pytestmark = pytest.mark.gpu

D = 128


@pytest.mark.parametrize("Hq,Hkv", [(3, 3), (12, 2), (24, 2)])
@pytest.mark.parametrize("S0,win", [(64, 256), (0, 64), (48, 0), (5, 3), (20, 600)])
def test_step_equals_attention_on_its_cache(Hq, Hkv, S0, win):
    _check(Hq, Hkv, S0, win, sorted({1, max(1, S0), S0 + 1, S0 + max(1, win), S0 + win + 1, S0 + win + 70, 65, 700}))


@pytest.mark.parametrize("Hq", [18, 32])
@pytest.mark.parametrize("S0,win", [(0, 0), (0, 64), (48, 0), (5, 3), (64, 192), (64, 193)])
def test_many_sequences(Hq, S0, win):
    Hkv, lens = 2, sorted({1, max(1, S0), S0 + max(1, win), S0 + win + 70, 131})
    B = torch.cuda.get_device_properties(0).multi_processor_count // Hkv + 2
    _check(Hq, Hkv, S0, win, [lens[b % len(lens)] for b in range(B)])


def _check(Hq, Hkv, S0, win, lens):
    B, mp = len(lens), -(-max(lens) // 64) + 1
    g = torch.Generator().manual_seed(S0 * 1000 + win + Hq)
    lay = ok.Layout(Hkv, B * mp)
    table = torch.randperm(B * mp, generator=g).to(torch.int32).reshape(B, mp).cuda()
    Rk, Rv = (torch.from_numpy(W.rotation(s)).cuda() for s in (Hq, Hq + 1))
    pool = ok.alloc_pool(lay)
    seg = torch.full((B, Hkv, 2, S0 + win, D), math.nan, dtype=torch.bfloat16, device="cuda")
    n = torch.tensor(lens, dtype=torch.int32, device="cuda")
    rows = [torch.randn(2, ln, Hkv, D, generator=g).to(torch.bfloat16).cuda() for ln in lens]
    seq = torch.cat([torch.full((ln - 1,), b, dtype=torch.int32) for b, ln in enumerate(lens)]).cuda()
    pos = torch.cat([torch.arange(ln - 1) for ln in lens]).cuda()
    ok.mixed_append(lay, pool, seg, S0, win, *(torch.cat([r[i, :-1] for r in rows]) for i in (0, 1)), seq, pos,
                    table, n - 1, Rk, Rv, 0.9, 0.9)
    k_new, v_new = (torch.stack([r[i, -1] for r in rows]).contiguous() for i in (0, 1))
    q = torch.randn(B, Hq, D, generator=g).to(torch.bfloat16).cuda()
    S = ok.default_num_splits(lay, B, Hq, mp * 64)
    ws = ok.alloc_mixed_workspace(lay, B, Hq, S)
    ws.fill_(0xff)  # NaN in every slot that is read without having been written
    outs = [torch.empty(B, Hq, D, device="cuda") for _ in range(2)]
    ok.decode_step_mixed(lay, pool, seg, S0, win, k_new, v_new, 0.9, 0.9, q, table, n, Rk, Rv, D ** -0.5, S,
                         ws, outs[0])
    ok.decode_attn_mixed(lay, pool, seg, S0, win, q, table, n, Rk, Rv, D ** -0.5, S, ws, outs[1])
    torch.cuda.synchronize()
    assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1])
    for b, ln in enumerate(lens):
        p = ln - 1
        if p < S0 or win > 0:
            s = p if p < S0 else S0 + (p - S0) % win
            assert torch.equal(seg[b, :, 0, s], k_new[b]) and torch.equal(seg[b, :, 1, s], v_new[b])
    assert np.isfinite(outs[0].cpu().numpy()).all()
