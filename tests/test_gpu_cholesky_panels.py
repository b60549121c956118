"""Cholesky factor and inverse at orders around its panels of 16 columns, the 48 rows a wavefront
takes below a panel, and the 64-column blocks of the large form (from 137 on).

With u = 2^-53 the factor satisfies |G - L L^H| <= c (n + 1) u |L| |L^H| <= c (n + 1) u max_i G_ii
entry by entry (Cauchy-Schwarz), and an inverse by substitution or by block products
|X L - I| <= c (n + 1) u |X| |L|, c = 8 for complex products and sums in blocks.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

U = 2.0 ** -53


def spd(n, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((n, 2 * n)) + 1j * rng.standard_normal((n, 2 * n))
    return x @ x.conj().T / (2 * n)


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 63, 64, 65, 112, 113, 127, 136, 137, 160, 193, 255])
def test_factor_and_inverse(n):
    from paper_2501_08697_amd import binding as b
    g = spd(n, n)
    print(f"[cholesky] n={n}", flush=True)
    t = torch.from_numpy(g.copy()).cuda()
    li = b.cholesky(t).cpu().numpy()
    L = np.tril(t.cpu().numpy())
    tol = 8.0 * (n + 1) * U
    assert np.max(np.abs(g - L @ L.conj().T)) <= tol * np.max(g.diagonal().real)
    assert np.all(np.abs(li @ L - np.eye(n)) <= tol * (np.abs(li) @ np.abs(L)) + 1e-300)
    assert np.max(np.abs(np.triu(li, 1)), initial=0.0) == 0.0
    assert np.all(L.diagonal().imag == 0.0) and np.all(L.diagonal().real > 0.0)


@pytest.mark.parametrize("n,pivot", [(1, 0), (40, 15), (40, 16), (136, 135), (200, 64), (200, 199)])
@pytest.mark.parametrize("value", [-1.0, float("nan")])
def test_pivot_that_is_not_positive(n, pivot, value):
    from paper_2501_08697_amd import binding as b
    g = spd(n, 3)
    g[pivot, pivot] = value
    with pytest.raises(b.AbacusPwError) as e:
        b.cholesky(torch.from_numpy(g).cuda())
    assert e.value.name == "ECHOLESKY"
