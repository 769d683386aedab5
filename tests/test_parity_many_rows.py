"""GPU parity of calls whose (sequence, head) rows exceed what one launch takes (2^20;
a grid of 2^32 threads or more is cut without an error): the sequences are dealt to
several launches.  65535 sequences, the most a call accepts, that share one page; rows
at the start, the end and on both sides of a launch's last sequence against the oracle
(2e-4 of the largest output: sums of three terms), and every other row against the
same query's first row."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_17757_amd as ok
import workloads as W
from helpers import bits, log

pytestmark = pytest.mark.gpu

D, B, HQ, HKV = 128, 65535, 20, 4
CUT = (1 << 20) // HQ  # sequences of the first launch
PAIRS = [(b, h) for b in (0, 1, CUT - 1, CUT, CUT + 1, B - 1) for h in (0, 4, HQ - 1)]


def _inputs(n, rph):
    g = torch.Generator().manual_seed(n + rph)
    q = torch.randn(7, HQ, D, generator=g).to(torch.bfloat16)[torch.arange(B) % 7].contiguous().cuda()
    k, v = (torch.randn(n, HKV, D, generator=g).to(torch.bfloat16).cuda() for _ in range(2))
    R = [np.stack([W.rotation(s + h) for h in range(HKV)]) if rph else W.rotation(s) for s in (3, 30)]
    table = torch.zeros(B, 1, dtype=torch.int32, device="cuda")
    lens = torch.full((B,), n, dtype=torch.int32, device="cuda")
    return q, k, v, R, [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in R], table, lens


def _check(out, q, want, what):
    got = out.reshape(B, HQ, D)
    for b0 in range(7):  # equal queries have equal rows
        assert torch.equal(got[b0::7], got[b0].expand_as(got[b0::7])), (what, b0)
    err = float(np.max(np.abs(np.stack([got[b, h].cpu().numpy() for b, h in PAIRS]) - want)))
    log(what, "max |err|", err)
    assert err <= 2e-4 * max(1.0, float(np.max(np.abs(want))))


@pytest.mark.parametrize("rph", [0, 1])
def test_plain_cache(rph):
    q, k, v, R, Rd, table, lens = _inputs(3, rph)
    lay = ok.Layout(HKV, 1, rot_per_head=rph)
    pool = ok.alloc_pool(lay)
    ok.kv_append(lay, pool, k[:2], v[:2], torch.arange(2).cuda(), *Rd, 0.9, 0.9)
    out = torch.empty(B, HQ, D, device="cuda")
    for S in (1, 2):
        ws = ok.alloc_workspace(lay, B, HQ, S).fill_(0xff)
        ok.decode_step(lay, pool, k[2:], v[2:], torch.full((1,), 2).cuda(), 0.9, 0.9, q, table, lens, *Rd,
                       D ** -0.5, S, ws, out)
        torch.cuda.synchronize()
        want = oracle.decode(pool.cpu().numpy(), d=D, Hkv=HKV, P=64, G=32, q=bits(q), block_table=table.cpu().numpy(),
                             seq_lens=lens.cpu().numpy(), Rk=R[0], Rv=R[1], sm_scale=D ** -0.5, pairs=PAIRS)
        _check(out, q, want, "step rph %d splits %d" % (rph, S))
        out.fill_(float("nan"))
        ok.decode_attn(lay, pool, q, table, lens, *Rd, D ** -0.5, S, ws.fill_(0xff), out)
        torch.cuda.synchronize()
        _check(out, q, want, "attn rph %d splits %d" % (rph, S))


def test_mixed_cache():
    S0, WIN = 1, 1
    q, k, v, R, Rd, table, lens = _inputs(3, 0)
    lay = ok.Layout(HKV, 1)
    pool, seg = ok.alloc_pool(lay), ok.alloc_seg(lay, B, S0, WIN)
    seg[:, :, 0] = k[:2].transpose(0, 1)  # token 0 in the sink, token 1 in the window
    seg[:, :, 1] = v[:2].transpose(0, 1)
    kn, vn = (x[2].expand(B, HKV, D).contiguous() for x in (k, v))
    out = torch.empty(B, HQ, D, device="cuda")
    ws = ok.alloc_mixed_workspace(lay, B, HQ, 1).fill_(0xff)
    ok.decode_step_mixed(lay, pool, seg, S0, WIN, kn, vn, 0.9, 0.9, q, table, lens, *Rd, D ** -0.5, 1, ws, out)
    torch.cuda.synchronize()
    assert torch.equal(seg[:, :, :, 0], torch.stack([k[0], v[0]], 1).expand(B, HKV, 2, D))
    assert torch.equal(seg[:, :, :, 1], torch.stack([kn, vn], 2))
    want = oracle.decode_mixed(pool.cpu().numpy(), bits(seg).reshape(-1), d=D, Hkv=HKV, P=64, G=32, S0=S0, W=WIN,
                               q=bits(q), block_table=table.cpu().numpy(), seq_lens=lens.cpu().numpy(), Rk=R[0],
                               Rv=R[1], sm_scale=D ** -0.5, pairs=PAIRS)
    _check(out, q, want, "mixed step")
    out.fill_(float("nan"))
    ok.decode_attn_mixed(lay, pool, seg, S0, WIN, q, table, lens, *Rd, D ** -0.5, 1, ws.fill_(0xff), out)
    torch.cuda.synchronize()
    _check(out, q, want, "mixed attention")


def test_mixed_step_past_the_grid_limit():
    """65535 sequences of 130 KV heads: 2^32 threads and more in blocks of 512 (26 GB).
    Of one bf16 token the output is its value row."""
    H = 130
    lay = ok.Layout(H, 1)
    q, k, v = (torch.randn(B, H, D, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    out = torch.zeros_like(v)
    ok.decode_step_mixed(lay, ok.alloc_pool(lay), ok.alloc_seg(lay, B, 0, 1), 0, 1, k, v, 0.9, 0.9, q,
                         torch.zeros(B, 1, dtype=torch.int32, device="cuda"),
                         torch.ones(B, dtype=torch.int32, device="cuda"), None, None, D ** -0.5, 1,
                         ok.alloc_mixed_workspace(lay, B, H, 1), out)
    torch.cuda.synchronize()
    assert torch.equal(out, v)
