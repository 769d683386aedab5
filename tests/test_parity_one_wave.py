"""GPU parity of the split kernel with one wave per page range, in every instance: up
to 4, 8, 12 and 16 query heads per KV head (with padding heads), groups of 32, 64 and
128 channels, both metadata formats, the plain and the mixed cache, one split and
three.  Calls with enough ranges that teams of waves do not fit the GPU: short ragged
sequences of 16 KV heads, zero-length ones among them, and ranges that cross
sequences.  The oracle decodes sampled rows from the same page bytes; outputs within
2e-4 of the largest: operands of 21 bits, fp32 sums of some hundred terms.  The bf16
output is the rounded fp32 output."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_17757_amd as ok
import workloads as W
from helpers import bits, log

pytestmark = pytest.mark.gpu

D, HKV, S0, WIN = 128, 16, 8, 16


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("g", [3, 7, 11, 14])
@pytest.mark.parametrize("meta", [ok.META_F16, ok.META_BF16])
@pytest.mark.parametrize("G", [32, 64, 128])
def test_one_wave_instances(G, meta, g, mixed):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    B, Hq, mp = 4 * cus // HKV + 6, HKV * g, 4  # a range per sequence: more blocks than any team rule admits
    seed = 1000 + G + meta * 7 + g
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, mp * 64 + 1, size=B).astype(np.int32)
    lens[:8] = 0, 1, 64, 65, 0, mp * 64, 128, 0
    lens[-1] = 0
    gen = torch.Generator().manual_seed(seed)
    n = int(lens.sum())
    k, v = (torch.randn(n, HKV, D, generator=gen) for _ in range(2))
    k[..., (5, 90)] *= 15.0
    k, v = k.to(torch.bfloat16).cuda(), v.to(torch.bfloat16).cuda()
    q = torch.randn(B, Hq, D, generator=gen).to(torch.bfloat16)
    table = rng.permutation(B * mp).astype(np.int32).reshape(B, mp)
    lay = ok.Layout(HKV, B * mp, group_size=G, meta_dtype=meta)
    Rk, Rv = W.rotation(seed), W.rotation(seed + 1)
    Rk_d, Rv_d, table_d, lens_d = (torch.from_numpy(x).cuda() for x in (Rk, Rv, table, lens))
    pool = ok.alloc_pool(lay)
    seq = np.repeat(np.arange(B, dtype=np.int32), lens)
    pos = np.concatenate([np.arange(m, dtype=np.int64) for m in lens])
    if mixed:
        seg = ok.alloc_seg(lay, B, S0, WIN)
        ok.mixed_append(lay, pool, seg, S0, WIN, k, v, torch.from_numpy(seq).cuda(), torch.from_numpy(pos).cuda(),
                        table_d, lens_d, Rk_d, Rv_d, 0.9, 0.9)
    else:
        slots = table[seq, pos // 64].astype(np.int64) * 64 + pos % 64
        ok.kv_append(lay, pool, k, v, torch.from_numpy(slots).cuda(), Rk_d, Rv_d, 0.9, 0.9)
    out = torch.empty(B, Hq, D, device="cuda")
    live = [b for b in list(range(8)) + [B - 2] + list(rng.integers(8, B - 1, size=3)) if lens[b]]
    pairs = [(int(b), int(h)) for b in live for h in (0, g - 1, int(rng.integers(Hq)), Hq - 1)]
    common = dict(d=D, Hkv=HKV, P=64, G=G, q=bits(q), block_table=table, seq_lens=np.maximum(lens, 1), Rk=Rk, Rv=Rv,
                  sm_scale=D ** -0.5, pairs=pairs, meta=meta)
    if mixed:
        want = oracle.decode_mixed(pool.cpu().numpy(), bits(seg).reshape(-1), S0=S0, W=WIN, **common)
    else:
        want = oracle.decode(pool.cpu().numpy(), **common)
    tol = 2e-4 * max(1.0, float(np.max(np.abs(want))))
    for S in (1, 3):
        if mixed:
            ok.decode_attn_mixed(lay, pool, seg, S0, WIN, q.cuda(), table_d, lens_d, Rk_d, Rv_d, D ** -0.5, S,
                                 ok.alloc_mixed_workspace(lay, B, Hq, S).fill_(0xff), out)
        else:
            ok.decode_attn(lay, pool, q.cuda(), table_d, lens_d, Rk_d, Rv_d, D ** -0.5, S,
                           ok.alloc_workspace(lay, B, Hq, S).fill_(0xff), out)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert not got[lens == 0].any()
        err = float(np.max(np.abs(np.stack([got[b, h] for b, h in pairs]) - want)))
        log("G", G, "meta", meta, "g", g, "mixed", mixed, "splits", S, "max |err|", err)
        assert np.isfinite(got).all() and err <= tol
        out16 = torch.empty(B, Hq, D, device="cuda", dtype=torch.bfloat16)
        args = (q.cuda(), table_d, lens_d, Rk_d, Rv_d, D ** -0.5, S)
        if mixed:
            ok.decode_attn_mixed(lay, pool, seg, S0, WIN, *args, ok.alloc_mixed_workspace(lay, B, Hq, S), out16)
        else:
            ok.decode_attn(lay, pool, *args, ok.alloc_workspace(lay, B, Hq, S), out16)
        torch.cuda.synchronize()
        assert torch.equal(out16, out.to(torch.bfloat16))
