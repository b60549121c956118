"""The density through the column passes against the oracle and against the slab passes: grid lengths
at the edges of what a thread's sums allow, spheres inside a quarter of the grid length and beyond
it, bands in one batch and in batches of two, work-groups whose bands belong to two k-points.

Bar as in test_gpu_density: relative max-norm 1e-12.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2501_08697_amd import workload as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

K3 = ((0.0, 0.0, 0.0), (0.5, 0.0, 0.0), (0.25, 0.375, 0.5))


@pytest.mark.parametrize("fft,a,ecut,nk,nb", [
    (8, 6.0, 5.0, 1, 1), (8, 6.0, 9.0, 3, 3),      # the smallest grid; past a quarter of the length
    (27, 9.0, 18.0, 3, 5), (45, 14.0, 22.0, 3, 7), (48, 14.0, 27.0, 2, 37), (64, 17.0, 30.0, 1, 9),
    (72, 20.5, 30.0, 2, 5), (72, 20.5, 50.0, 1, 3), (60, 16.0, 30.0, 1, 3), (81, 22.0, 26.0, 1, 4),
    (96, 24.0, 35.0, 2, 3), (96, 24.0, 60.0, 1, 2), (100, 25.0, 25.0, 1, 2), (108, 27.0, 25.0, 1, 3),
    (80, 20.0, 25.0, 1, 2), (120, 28.0, 30.0, 1, 2),   # no kernel: slab passes
])
def test_density_matches_oracle(fft, a, ecut, nk, nb):
    from paper_2501_08697_amd import binding as b
    p = W.make_problem(W.tiny_config(a=a, ecut=ecut, fft=fft, kfrac=K3[:nk], natom=2, lmax=0, nb=nb, seed=3))
    print(f"[density columns] fft={p.fft} npw={list(p.npw)} nb={p.nb}", flush=True)
    occ = np.random.default_rng(7).uniform(0.0, 2.0, (nk, nb))
    ref = oracle.density(p, p.psi, occ)
    dp = b.DeviceProblem(p)
    x = torch.from_numpy(p.psi).cuda()
    try:
        for knobs in ({}, dict(band_batch=2, yz_bands=3), dict(yz_mode=2)):
            b.set_tuning(**knobs)
            rho = b.density(dp, x, occ).cpu().numpy()
            assert np.max(np.abs(rho - ref)) <= 1e-12 * np.max(ref), knobs
    finally:
        b.set_tuning()
