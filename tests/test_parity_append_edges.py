"""GPU parity of the cache update where its kernels and their dispatch can go wrong:
one token, a remainder of 16 tokens, the last size of the one-item-per-block kernel
(256 items of 16 tokens of a head per tensor on a 256-CU GPU) and the first of the
bulk kernel, one and several KV heads, every quantizer format, tokens that are
skipped (negative slots), and rows whose quantile, scale or division is degenerate:
zero, constant, equal magnitudes, one outlier, tiny and huge values.  Page bytes are
those of the oracle, without exception."""
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
    if not meta:  # binary16 scales saturate there: covered by the bf16 formats
        k, v = k.clamp(-6e4, 6e4), v.clamp(-6e4, 6e4)
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
