"""The column passes of the local term (the automatic FP64 plane mode) against the oracle and
against the slab passes, at grid lengths, sphere radii and band counts where their tiles have
remainders: one column group and many, chunks of one column and of all, spheres inside a
quarter of the grid length (empty codelet slots skipped) and beyond it, unequal x and y
lengths, work-groups whose bands belong to two k-points with different spheres.

Error metric and bar as in test_gpu_apply_h: relative max-norm 1e-12 in FP64.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2501_08697_amd import workload as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

K3 = ((0.0, 0.0, 0.0), (0.5, 0.0, 0.0), (0.25, 0.375, 0.5))


def problem(n1, n2, a1, a2, ecut, kfrac, nb, seed=5):
    """An orthorhombic cell on an n1 x n2 x n2 grid (the generator's cells are cubic in the grid)."""
    lat = np.diag([a1, a2, a2])
    cfg = W.tiny_config(a=a1, ecut=ecut, fft=max(n1, n2), kfrac=kfrac, natom=3, lmax=1, nb=nb, seed=seed)
    p = W.make_problem(cfg, lattice=lat)
    fft = (n1, n2, n2)
    for i in range(3):
        assert 2 * int(np.abs(p.miller[:, i]).max()) + 1 <= fft[i]
    return dataclasses.replace(p, fft=fft, vloc=np.ascontiguousarray(W.gaussian_vloc(lat, fft, p.tau, p.depth)))


CASES = [
    (8, 8, 6.0, 6.0, 5.0, K3[:1], 1),          # the smallest grid, one band
    (8, 8, 6.0, 6.0, 9.0, K3, 3),              # its sphere past a quarter of the length
    (27, 27, 9.0, 9.0, 18.0, K3, 5),           # odd length
    (45, 45, 14.0, 14.0, 22.0, K3, 7),
    (48, 54, 14.3, 16.1, 27.0, K3, 13),        # x and y lengths differ
    (120, 24, 28.0, 6.0, 30.0, K3[:2], 5),     # long in x
    (20, 96, 6.0, 24.0, 16.0, K3[:2], 5),      # long in y
    (24, 32, 9.0, 12.0, 28.0, K3[:2], 4),      # unequal and past a quarter: no column kernel, slab passes
    (72, 72, 17.0, 17.0, 32.0, K3[2:], 9),
    (81, 90, 20.0, 22.0, 26.0, K3[:1], 3),
    (100, 108, 25.0, 27.0, 25.0, K3[:1], 2),
    (128, 128, 30.0, 30.0, 44.0, K3[:1], 2),
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}x{c[1]}_nb{c[6]}" for c in CASES])
def test_columns_match_oracle_and_slab(case):
    from paper_2501_08697_amd import binding as b
    p = problem(*case)
    print(f"[columns] fft={p.fft} npw={list(p.npw)} nb={p.nb}", flush=True)
    dp = b.DeviceProblem(p)
    x = torch.from_numpy(p.psi).cuda()
    ref = oracle.apply_h(p, p.psi)
    scale = np.max(np.abs(ref))
    try:
        # the defaults, then two bands per batch and odd band groups
        for knobs in ({}, dict(band_batch=2, yz_bands=3, x_bands=3), dict(yz_mode=2)):
            b.set_tuning(**knobs)
            y = b.apply_h(dp, x).cpu().numpy()
            assert np.max(np.abs(y - ref)) / scale < 1e-12, knobs
    finally:
        b.set_tuning()


def test_columns_follow_a_changed_potential():
    """V is transposed on every call: another V (and another tensor) behind the same plan is seen at once."""
    from paper_2501_08697_amd import binding as b
    p = problem(32, 32, 9.0, 9.0, 20.0, K3[:2], 6)
    dp = b.DeviceProblem(p)
    x = torch.from_numpy(p.psi).cuda()
    for scale in (1.0, -0.5):
        q = dataclasses.replace(p, vloc=p.vloc * scale)
        dp.vloc.copy_(torch.from_numpy(q.vloc))
        ref = oracle.apply_h(q, q.psi)
        y = b.apply_h(dp, x).cpu().numpy()
        assert np.max(np.abs(y - ref)) / np.max(np.abs(ref)) < 1e-12
    v2 = torch.from_numpy(p.vloc * 2.0).cuda()
    q = dataclasses.replace(p, vloc=p.vloc * 2.0)
    ref = oracle.apply_h(q, q.psi)
    y = b.apply_h(dp, x, vloc=v2).cpu().numpy()
    assert np.max(np.abs(y - ref)) / np.max(np.abs(ref)) < 1e-12
