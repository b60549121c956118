"""Orders at the edges of the many-CU tridiagonal reduction (abacus_pw_eigh_lowest): the switch
from one compute unit (88), one work-group more or less, panel remainders of 8, 256 / 512
threads, the panel in LDS (512) or in memory, rows beyond the pieces fetched ahead. Checked as in test_gpu_dense.py: eigenvalues
against LAPACK to 1e-12 of ||A||, residuals to 1e-11, orthonormality to 1e-9.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1, 2, 87, 88, 89, 95, 176, 177, 255, 256, 257, 258, 321, 512, 513, 515, 1025])
@pytest.mark.parametrize("zero_block", [False, True])
def test_orders_around_the_switches(n, zero_block):
    from paper_2501_08697_amd import binding
    rng = np.random.default_rng(7 * n)
    x = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    a = 0.5 * (x + x.conj().T)
    if zero_block:   # rows that need no reflector (tau = 0) among those that do
        z = slice(n // 3, n // 3 + n // 8)
        d = a.diagonal().copy()
        a[z, :] = 0
        a[:, z] = 0
        a[np.arange(n), np.arange(n)] = d
    nw = max(1, n // 2)
    print(f"[tridiagonal] n={n} zero_block={zero_block}", flush=True)
    w, v = binding.eigh_lowest(torch.from_numpy(a.copy()).cuda(), nw)
    w, v = w.cpu().numpy(), v.cpu().numpy()
    an = np.linalg.norm(a, 2)
    assert np.max(np.abs(w - np.linalg.eigvalsh(a)[:nw])) < 1e-12 * an
    assert np.max(np.linalg.norm(v @ a.T - w[:, None] * v, axis=1)) < 1e-11 * an
    assert np.max(np.abs(v.conj() @ v.T - np.eye(nw))) < 1e-9
