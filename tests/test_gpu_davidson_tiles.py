"""Davidson at band counts around the 64-wide tiles of the Hermitian Gram products and of the
products with a triangular inverse factor: one tile, one band into the second, three tiles with a
remainder. Lowest eigenvalues against the dense matrix, orthonormality, and the oracle's residuals.

A residual of 1e-9 bounds an eigenvalue's error by 1e-9 (Krylov-Weinstein).
"""
import numpy as np
import pytest

import oracle
from paper_2501_08697_amd import workload as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nb", [1, 64, 65, 130])
def test_band_counts_around_tiles(nb):
    from paper_2501_08697_amd import binding as b
    p = W.make_problem(W.tiny_config(a=10.0, ecut=20.0, fft=32, natom=4, lmax=1, nb=nb, seed=9))
    print(f"[davidson tiles] nb={nb} npw={list(p.npw)}", flush=True)
    x = torch.from_numpy(p.psi).cuda()
    eig, res, its, st = b.davidson(b.DeviceProblem(p), x, tol=1e-9, max_iter=200)
    assert st == 0 and np.max(res) < 1e-9
    ev = np.linalg.eigvalsh(oracle.dense_h(p, 0))[:nb]
    assert np.max(np.abs(np.sort(eig[0]) - ev)) < 1e-9
    v = x.cpu().numpy().reshape(nb, -1)
    assert np.max(np.abs(v.conj() @ v.T - np.eye(nb))) < 1e-12
    hv = oracle.apply_h(p, v.reshape(-1), nb=nb).reshape(nb, -1)
    assert np.max(np.linalg.norm(hv - eig[0][:, None] * v, axis=1)) < 2e-9
