"""A matrix of four columns waits for four pivots of its panel, not for sixteen: its factorisation takes
less time than that of a whole panel."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def factor_ms(n):
    from paper_2501_08697_amd import binding as b
    rng = np.random.default_rng(n)
    x = rng.standard_normal((n, 2 * n)) + 1j * rng.standard_normal((n, 2 * n))
    g = torch.from_numpy(x @ x.conj().T).cuda()
    b.cholesky(g.clone())
    try:
        b.profile_enable()
        b.profile_read()
        for _ in range(50):
            b.cholesky(g.clone())
        return b.profile_read()["potrf_inv"][1]
    finally:
        b.profile_enable(False)


def test_four_columns_take_less_than_sixteen():
    t4, t16 = factor_ms(4), factor_ms(16)
    print(f"[cholesky small] 4: {t4:.3f} ms, 16: {t16:.3f} ms for 50", flush=True)
    assert t4 < 0.85 * t16
