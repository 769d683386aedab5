"""GPU parity of the cache update where its kernels and their dispatch can go wrong:
one token, a remainder of 16 tokens, the last size of the one-item-per-block kernel
(256 items of 16 tokens of a head per tensor on a 256-CU GPU) and the first of the
bulk kernel, one and several KV heads, every quantizer format, tokens that are
skipped (negative slots), and rows whose quantile, scale or division is degenerate:
zero, constant, equal magnitudes, one outlier, tiny and huge values (saturated scales),
and finite rows that rotate to an fp32 infinity.  Page bytes are those of the oracle,
without exception."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_17757_amd as ok
import workloads as W
from helpers import bits, log

pytestmark = pytest.mark.gpu

# name -> (group size, meta, clip mode, rotate K, rotate V, one rotation per KV head)
FORMATS = {
    "default": (32, 0, 0, True, True, 0),
    "paper": (128, 1, 1, True, True, 0),
    "g64_quantile_identity_v": (64, 0, 1, True, False, 0),
    "bf16_per_head": (32, 1, 0, True, True, 1),
    "identity": (32, 1, 1, False, False, 0),
}


def _rows(n, Hkv, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(n, Hkv, 128, generator=g)
    x[..., (5, 90)] *= 15.0
    kind = torch.randint(0, 12, (n, Hkv), generator=g)
    x[kind == 0] = 0.0
    x[kind == 1] = -3.0
    x[kind == 2] = x[kind == 2].sign() * 0.5                 # equal magnitudes
    x[kind == 3] *= 1e-30                                    # bf16 scales below 2^-60
    x[kind == 4] *= 1e25                                     # and above 2^60
    x[kind == 5, 64:] = 0.0
    x[(kind == 6).nonzero(as_tuple=True) + (torch.full(((kind == 6).sum(),), 7),)] = 3e4
    return x.to(torch.bfloat16)


@pytest.mark.parametrize("fmt", list(FORMATS))
@pytest.mark.parametrize("n_tok,Hkv", [(1, 1), (17, 3), (512, 8), (513, 8), (4111, 1)])
def test_append_edges(fmt, n_tok, Hkv):
    G, meta, clip_mode, rk, rv, rph = FORMATS[fmt]
    seed = 31 * n_tok + Hkv
    n_pages = (n_tok + 63) // 64 + 2
    lay = ok.Layout(Hkv, n_pages, group_size=G, clip_mode=clip_mode, meta_dtype=meta, rot_per_head=rph)
    R = np.stack([W.rotation(seed + h) for h in range(Hkv if rph else 1)])
    R = np.ascontiguousarray(R if rph else R[0])
    Rk, Rv = (R if rk else None), (np.ascontiguousarray(np.swapaxes(R, -1, -2)) if rv else None)
    k, v = _rows(n_tok, Hkv, seed), _rows(n_tok, Hkv, seed + 1)
    rng = np.random.default_rng(seed)
    slots = rng.permutation(n_pages * 64)[:n_tok].astype(np.int64)
    slots[rng.random(n_tok) < 0.05] = -1
    keep = slots >= 0
    pool = torch.full((ok.pool_bytes(lay),), 0x5a, dtype=torch.uint8, device="cuda")
    dev = [None if m is None else torch.from_numpy(m).cuda() for m in (Rk, Rv)]
    for rho in (0.9, 1.0):
        ok.kv_append(lay, pool, k.cuda(), v.cuda(), torch.from_numpy(slots).cuda(), dev[0], dev[1], rho, rho)
        torch.cuda.synchronize()
        want = np.full(ok.pool_bytes(lay), 0x5a, np.uint8)
        oracle.kv_append(want, d=128, Hkv=Hkv, P=64, G=G, k=bits(k[torch.from_numpy(keep)]),
                         v=bits(v[torch.from_numpy(keep)]), slot_mapping=slots[keep], Rk=Rk, Rv=Rv,
                         clip_k=rho, clip_v=rho, meta=meta, clip=clip_mode)
        diff = int((pool.cpu().numpy() != want).sum())
        log(fmt, n_tok, Hkv, rho, "differing bytes", diff)
        assert diff == 0


@pytest.mark.parametrize("fmt", list(FORMATS))
@pytest.mark.parametrize("n_tok,Hkv", [(40, 3), (700, 8)])
def test_append_overflowing_rows(fmt, n_tok, Hkv):
    """Finite bf16 rows up to 3.3e38, of which some rotate to infinities of one or both
    signs (both update kernels): the oracle's page bytes, and its clip errors (finite
    ones within 1e-9: terms of one sign, some 1e4 of them)."""
    G, meta, clip_mode, rk, rv, rph = FORMATS[fmt]
    g = torch.Generator().manual_seed(n_tok)
    size = torch.tensor([1.0, 1e4, 1e20, 1e36, 1e37, 3e37, 8e37])
    k, v = (torch.randn(n_tok, Hkv, 128, generator=g).clamp(-4, 4)
            * size[torch.randint(0, 7, (n_tok, Hkv), generator=g)][..., None] for _ in range(2))
    k[::9] = k[::9].sign() * 3.3e38
    v[::9] = 0.0
    v[::9, :, 7] = 3.3e38
    k, v = k.to(torch.bfloat16), v.to(torch.bfloat16)
    assert torch.isfinite(k).all() and torch.isfinite(v).all()
    R = np.stack([W.rotation(5 + h) for h in range(Hkv if rph else 1)])
    R = np.ascontiguousarray(R if rph else R[0])
    Rk, Rv = (R if rk else None), (np.ascontiguousarray(np.swapaxes(R, -1, -2)) if rv else None)
    dev = [None if m is None else torch.from_numpy(m).cuda() for m in (Rk, Rv)]
    lay = ok.Layout(Hkv, n_tok // 64 + 1, group_size=G, clip_mode=clip_mode, meta_dtype=meta, rot_per_head=rph)
    slots = np.arange(n_tok, dtype=np.int64)
    for rho in (0.5, 0.9, 1.0):
        pool = torch.full((ok.pool_bytes(lay),), 0x5a, dtype=torch.uint8, device="cuda")
        ok.kv_append(lay, pool, k.cuda(), v.cuda(), torch.from_numpy(slots).cuda(), dev[0], dev[1], rho, rho)
        torch.cuda.synchronize()
        want = np.full(ok.pool_bytes(lay), 0x5a, np.uint8)
        oracle.kv_append(want, d=128, Hkv=Hkv, P=64, G=G, k=bits(k), v=bits(v), slot_mapping=slots, Rk=Rk,
                         Rv=Rv, clip_k=rho, clip_v=rho, meta=meta, clip=clip_mode)
        diff = int((pool.cpu().numpy() != want).sum())
        log(fmt, n_tok, Hkv, rho, "differing bytes", diff)
        assert diff == 0
    cands = np.array([0.31, 0.9, 1.0], np.float32)
    for x, m, Rx in ((k, dev[0], Rk), (v[:8], dev[1], Rv)):
        err = ok.calib_clip(lay, x.cuda(), m, torch.from_numpy(cands).cuda())[0].cpu().numpy()
        ref = oracle.clip_errors(bits(x), Rx, G=G, cands=cands, meta=meta, clip=clip_mode)
        log(fmt, n_tok, Hkv, "clip errors", err, ref)
        assert np.array_equal(np.isfinite(err), np.isfinite(ref)) and not np.isnan(err).any()
        fin = np.isfinite(ref)
        assert np.all(np.abs(err[fin] - ref[fin]) <= 1e-9 * np.abs(ref[fin]))


@pytest.mark.parametrize("fmt", list(FORMATS))
@pytest.mark.parametrize("n_tok,Hkv,n_cands", [(1, 1, 1), (17, 3, 32), (47, 2, 9)])
def test_clip_errors_edges(fmt, n_tok, Hkv, n_cands):
    """calib_clip at the edges of its 16-token items and of the candidate count, on
    the same degenerate rows.  Error sums: the same fp64 terms in another order, the
    term (x~ - s (code - z))^2 with one rounding fewer, so within the few roundings of
    the cancellation in x~ - s (code - z), at most |x~| 2^-52 each: relative to the
    rows' mean square, 1e-12 covers them with room."""
    G, meta, clip_mode, rk, _, rph = FORMATS[fmt]
    seed = 77 * n_tok + Hkv
    lay = ok.Layout(Hkv, 1, group_size=G, clip_mode=clip_mode, meta_dtype=meta, rot_per_head=rph)
    R = np.stack([W.rotation(seed + h) for h in range(Hkv if rph else 1)])
    R = np.ascontiguousarray(R if rph else R[0]) if rk else None
    x = _rows(n_tok, Hkv, seed)
    x = x.float().clamp(-1e3, 1e3).to(torch.bfloat16)  # errors of one size
    cands = np.linspace(0.31, 1.0, n_cands).astype(np.float32)
    err, best = ok.calib_clip(lay, x.cuda(), None if R is None else torch.from_numpy(R).cuda(),
                              torch.from_numpy(cands).cuda())
    torch.cuda.synchronize()
    want = oracle.clip_errors(bits(x), R, G=G, cands=cands, meta=meta, clip=clip_mode)
    got, ms = err.cpu().numpy(), float(x.double().square().mean())
    log(fmt, n_tok, Hkv, "max error over mean square", float(np.max(np.abs(got - want))) / max(ms, 1e-300))
    assert np.all(np.abs(got - want) <= 1e-12 * ms)
    assert float(best.cpu()[0]) == float(cands[int(np.argmin(got))])


@pytest.mark.parametrize("fmt", ["paper", "g64_quantile_identity_v"])
def test_clip_ratios_outside_the_unit_interval(fmt):
    """Candidate ratios are not validated: one below 0 gives the error of 0, one above 1
    that of 1, and the others are not affected."""
    G, meta, clip_mode, _, _, rph = FORMATS[fmt]
    lay = ok.Layout(2, 1, group_size=G, clip_mode=clip_mode, meta_dtype=meta, rot_per_head=rph)
    x = torch.randn(40, 2, 128, generator=torch.Generator().manual_seed(9)).to(torch.bfloat16).cuda()
    R = torch.from_numpy(W.rotation(9)).cuda()
    err = [ok.calib_clip(lay, x, R, torch.tensor(c, device="cuda"))[0].cpu().tolist()
           for c in ([0.0, 0.5, 1.0], [-0.01, 0.5, 1.5], [-3.0, 0.5, 2.0])]
    log(fmt, err)
    assert err[0] == err[1] == err[2]


@pytest.mark.parametrize("fmt,Hkv", [("default", 8), ("paper", 8), ("bf16_per_head", 6)])
def test_step_with_more_items_than_blocks(fmt, Hkv):
    """A decode step's update takes its items of 16 tokens of a head on at most one block
    per CU and tensor (per-head rotations: a multiple of the heads); with more items a
    block takes several in turn.  Page bytes: the oracle's for decode_step; for
    decode_step_mixed those of kv_append of the rows that leave the window, and the
    segment store changes in the new tokens' rows only."""
    G, meta, clip_mode, rk, rv, rph = FORMATS[fmt]
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    B = 16 * (cus // Hkv) + 16 * 2 + 5
    assert -(-B // 16) * Hkv > cus
    lay = ok.Layout(Hkv, B, group_size=G, clip_mode=clip_mode, meta_dtype=meta, rot_per_head=rph)
    R = np.stack([W.rotation(70 + h) for h in range(Hkv if rph else 1)])
    R = np.ascontiguousarray(R if rph else R[0])
    Rd = torch.from_numpy(R).cuda()
    rng = np.random.default_rng(B)
    k, v = _rows(B, Hkv, 71), _rows(B, Hkv, 72)
    q = torch.randn(B, Hkv, 128, generator=torch.Generator().manual_seed(73)).to(torch.bfloat16).cuda()
    table = torch.from_numpy(rng.permutation(B).astype(np.int32)).reshape(B, 1).cuda()
    lens = torch.from_numpy(rng.integers(1, 65, size=B).astype(np.int32)).cuda()
    out = torch.empty(B, Hkv, 128, device="cuda")
    slots = table[:, 0].long() * 64 + lens.long() - 1
    slots[5::17] = -1  # skipped tokens
    pool = ok.alloc_pool(lay)
    ok.decode_step(lay, pool, k.cuda(), v.cuda(), slots, 0.9, 0.9, q, table, lens, Rd, Rd, 128 ** -0.5, 1,
                   ok.alloc_workspace(lay, B, Hkv, 1), out)
    torch.cuda.synchronize()
    want, keep = np.zeros(ok.pool_bytes(lay), np.uint8), (slots >= 0).cpu()
    oracle.kv_append(want, d=128, Hkv=Hkv, P=64, G=G, k=bits(k[keep]), v=bits(v[keep]),
                     slot_mapping=slots.cpu().numpy()[keep.numpy()], Rk=R, Rv=R, clip_k=0.9, clip_v=0.9, meta=meta,
                     clip=clip_mode)
    diff = int((pool.cpu().numpy() != want).sum())
    log(fmt, "step: differing bytes", diff)
    assert diff == 0

    S0, win = 2, 3
    lens = lens % 9 + 1
    store = torch.stack([_rows(B * (S0 + win), Hkv, s).reshape(B, S0 + win, Hkv, 128).transpose(1, 2) for s in (74, 75)], 2)
    seg = store.contiguous().cuda()
    pool.zero_()
    ok.decode_step_mixed(lay, pool, seg, S0, win, k.cuda(), v.cuda(), 0.9, 0.9, q, table, lens, Rd, Rd, 128 ** -0.5, 1,
                         ok.alloc_mixed_workspace(lay, B, Hkv, 1), out)
    p = lens.long().cpu() - 1
    slot = torch.where(p < S0, p, S0 + (p - S0) % win)
    b = torch.arange(B)
    left = store[b, :, :, slot]  # [B, Hkv, 2, 128]: what the new rows displaced
    demoted = p - win >= S0
    ref = ok.alloc_pool(lay)
    to = table[:, 0].long() * 64 + (lens.long() - 1 - win)
    ok.kv_append(lay, ref, *(left[demoted][:, :, i].contiguous().cuda() for i in (0, 1)), to[demoted.cuda()].contiguous(),
                 Rd, Rd, 0.9, 0.9)
    torch.cuda.synchronize()
    store = store.clone()
    store[b, :, 0, slot], store[b, :, 1, slot] = k, v
    same = bool((pool == ref).all()), bool((seg.cpu().view(torch.int16) == store.contiguous().view(torch.int16)).all())
    log(fmt, "mixed step: demoted", int(demoted.sum()), "pages, segments as expected", same)
    assert demoted.any() and same == (True, True)
