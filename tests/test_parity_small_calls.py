"""GPU parity of decode calls around the rules that choose the split kernel's and the
reduce kernel's instances: a team of waves per page range (calls that leave the GPU
mostly idle) or one wave, pieces shorter than a team, ranges that cross sequences,
empty sequences, one split; and 2, 4, 8 or 16 rows per reduce block, at the row counts
where the choice changes and one row off them.  Outputs against the oracle within
2e-4 of the largest output: the score and weight operands carry at least 21 bits and
sums are fp32, of at most a few thousand terms (observed: 4e-5 at most)."""
import numpy as np
import pytest

import workloads as W
from helpers import gpu_append, gpu_decode, log, make_case, max_abs, oracle_append, oracle_decode
from test_parity_mixed import Mixed

pytestmark = pytest.mark.gpu


def _check(cfg, splits, pairs=None):
    case = make_case(cfg)
    pool, want_pool = gpu_append(case), oracle_append(case)
    if pairs is None:
        pairs = [(b, h) for b in range(cfg.B) for h in range(cfg.Hq) if cfg.lens[b]]
    want = oracle_decode(case, want_pool, lens=np.maximum(cfg.lens, 1), pairs=pairs)
    for S in splits:
        out = gpu_decode(case, pool, S)
        got = out.cpu().numpy()
        assert not got[np.asarray(cfg.lens) == 0].any()  # empty sequences
        got = np.stack([got[b, h] for b, h in pairs])
        err = max_abs(got, want)
        log(cfg.name, "splits", S, "max |err|", err)
        assert err <= 2e-4 * max(1.0, float(np.max(np.abs(want))))


@pytest.mark.parametrize("Hq,Hkv", [(1, 1), (4, 1), (12, 2), (12, 1), (32, 2)])
@pytest.mark.parametrize("lens", [[1], [64 * 5 + 1], [700], [63, 0, 64, 65, 0, 200, 130]])
def test_team_split(Hq, Hkv, lens):
    _check(W.custom("team_h%dx%d_%d" % (Hq, Hkv, len(lens)), len(lens), Hq, Hkv, lens,
                    seed_index=300 + Hq + len(lens), k_outliers=(5, 90)), (1, 2, 0, 40))


@pytest.mark.parametrize("B,Hq,Hkv", [(1, 3, 3), (73, 7, 7), (64, 8, 8), (89, 23, 23), (64, 32, 8),
                                      (63, 65, 13), (64, 64, 16), (257, 16, 16),
                                      (33, 31, 31), (64, 16, 8)])
def test_reduce_rows(B, Hq, Hkv):
    """511 / 512, 1023 / 1024, 2047 / 2048, 4095 / 4096 rows and some past them; sampled
    rows."""
    lens = 1 + (np.arange(B) * 37) % 150
    rng = np.random.default_rng(B)
    pairs = sorted({(0, 0), (B - 1, Hq - 1)} |
                   {(int(rng.integers(B)), int(rng.integers(Hq))) for _ in range(60)})
    _check(W.custom("rows_%d" % (B * Hq), B, Hq, Hkv, lens, seed_index=400 + B, k_outliers=(17,)), (0, 5),
           pairs=pairs)


@pytest.mark.parametrize("B,Hq,Hkv", [(16, 32, 8), (33, 31, 31), (16, 64, 8)])
def test_reduce_rows_mixed(B, Hq, Hkv):
    """512, 1023 and 1024 rows over the mixed cache, some of them with nine or more
    pieces beside the bf16 tokens' state."""
    lens = 1 + (np.arange(B, dtype=np.int32) * 37) % 150
    lens[[1, B - 1]] = 2300, 2239
    cfg = W.custom("mixed_rows_%d" % (B * Hq), B, Hq, Hkv, lens, seed_index=450 + B, k_outliers=(17,))
    m = Mixed(cfg, 20, 50)
    pool, seg = m.gpu_prefill(lens - 1)
    got = m.gpu_step(pool, seg, lens, num_splits=12).cpu().numpy()
    want = m.oracle_decode(*m.oracle_build(lens), lens)
    err = max_abs(got, want)
    log(cfg.name, "max |err|", err)
    assert err <= 2e-4 * max(1.0, float(np.max(np.abs(want))))
