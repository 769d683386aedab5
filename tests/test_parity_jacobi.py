"""GPU eigen-decomposition on matrices whose rounds skip many or all rotations (block
diagonal, tridiagonal, nearly diagonal, one coupled pair at each end of the pair
order) and in batches: A U = U diag(lam) and U^T U = 1 within the rounding of the
rotations (about 10 sweeps of 127 rounds, each adding a few 2^-53 to a row in
quadrature: below 1e-13 relative), and a matrix gives the same bits alone and in a
batch."""
import numpy as np
import pytest
import torch

import paper_2605_17757_amd as ok
from helpers import log

pytestmark = pytest.mark.gpu


def _matrix(kind: str) -> np.ndarray:
    rng = np.random.default_rng(len(kind) * 101)
    d = 128
    X = rng.standard_normal((256, d)) * np.geomspace(12.0, 0.1, d)
    C = X.T @ X / 256
    i = np.arange(d)
    if kind == "blocks":
        C = np.where((i[:, None] // 16) == (i[None, :] // 16), C, 0.0)
    elif kind == "tridiagonal":
        C = np.where(np.abs(i[:, None] - i[None, :]) <= 1, C, 0.0)
    elif kind == "nearly_diagonal":
        C = np.diag(np.diag(C)) + 1e-14 * C
    elif kind == "end_pairs":
        C = np.diag(np.diag(C))
        for a, b in ((127, 0), (63, 64), (62, 64), (126, 127), (0, 1)):
            C[a, b] = C[b, a] = 0.25
    return np.ascontiguousarray((C + C.T) / 2)


KINDS = ("dense", "blocks", "tridiagonal", "nearly_diagonal", "end_pairs")


@pytest.mark.parametrize("kind", KINDS)
def test_decomposition(kind):
    batch = torch.from_numpy(np.stack([_matrix(k) for k in KINDS])).cuda()
    n = KINDS.index(kind)
    one, all_ = ok.calib_rotation(batch[n].clone()), ok.calib_rotation(batch)
    torch.cuda.synchronize()
    for key in ("lam", "U", "R64", "R32", "info"):
        assert torch.equal(one[key][0], all_[key][n]), key
    assert int(one["info"][0]) > 0
    A, lam, U = batch[n].cpu().numpy(), one["lam"][0].cpu().numpy(), one["U"][0].cpu().numpy()
    res = float(np.max(np.abs(A @ U - U * lam)) / np.max(np.abs(lam)))
    orth = float(np.max(np.abs(U.T @ U - np.eye(128))))
    log(kind, "sweeps", int(one["info"][0]), "residual", res, "orthogonality", orth)
    assert res <= 1e-13 and orth <= 1e-13 and np.all(np.diff(lam) <= 0)
