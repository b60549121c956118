"""The column passes of the local term in FP32 against the oracle: smallest
and largest length that takes them, odd lengths, spheres inside a quarter of the length and beyond
it, several k-points, bands in batches of two; unequal lengths, longer grids and the mixed mode keep
the slab passes.

Bar as in test_gpu_apply_h for FP32 transforms: relative max-norm 1e-5.
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
    lat = np.diag([a1, a2, a2])
    cfg = W.tiny_config(a=a1, ecut=ecut, fft=max(n1, n2), kfrac=kfrac, natom=3, lmax=1, nb=nb, seed=seed)
    p = W.make_problem(cfg, lattice=lat)
    fft = (n1, n2, n2)
    return dataclasses.replace(p, fft=fft, vloc=np.ascontiguousarray(W.gaussian_vloc(lat, fft, p.tau, p.depth)))


@pytest.mark.parametrize("case", [
    (8, 8, 6.0, 6.0, 5.0, K3[:1], 1), (8, 8, 6.0, 6.0, 9.0, K3, 3), (27, 27, 9.0, 9.0, 18.0, K3, 5),
    (45, 45, 14.0, 14.0, 22.0, K3, 7), (48, 48, 14.0, 14.0, 27.0, K3, 13), (72, 72, 17.0, 17.0, 32.0, K3[2:], 9),
    (72, 72, 20.0, 20.0, 50.0, K3[:1], 3), (81, 81, 22.0, 22.0, 26.0, K3[:1], 3),
    (90, 90, 22.0, 22.0, 26.0, K3[:1], 2), (96, 96, 24.0, 24.0, 25.0, K3[:1], 2), (48, 54, 14.3, 16.1, 27.0, K3, 5),   # slab passes
], ids=lambda c: f"{c[0]}x{c[1]}_nb{c[6]}")
def test_fp32_columns_match_oracle(case):
    from paper_2501_08697_amd import binding as b
    p = problem(*case)
    print(f"[columns f32] fft={p.fft} npw={list(p.npw)} nb={p.nb}", flush=True)
    dp = b.DeviceProblem(p)
    ref = oracle.apply_h(p, p.psi)
    scale = np.max(np.abs(ref))
    x = torch.from_numpy(p.psi).cuda()
    try:
        for knobs in ({}, dict(band_batch=2, yz_bands=3, x_bands=3), dict(yz_mode=2)):
            b.set_tuning(**knobs)
            for prec in (b.FP32, b.MIXED_FP32):
                y = b.apply_h(dp, x.to(torch.complex64) if prec == b.FP32 else x, prec).cpu().numpy()
                assert np.max(np.abs(y - ref)) / scale < 1e-5, (knobs, prec)
    finally:
        b.set_tuning()


@pytest.mark.parametrize("prec", [1, 3])
def test_fp32_columns_follow_a_changed_potential(prec):
    """V reaches the column passes in FP64 on every call, whatever copies the plan holds."""
    from paper_2501_08697_amd import binding as b
    p = problem(32, 32, 9.0, 9.0, 20.0, K3[:2], 6)
    dp = b.DeviceProblem(p)
    x = torch.from_numpy(p.psi).cuda()
    x = x.to(torch.complex64) if prec == b.FP32 else x
    for scale in (1.0, -0.5):
        q = dataclasses.replace(p, vloc=p.vloc * scale)
        dp.vloc.copy_(torch.from_numpy(q.vloc))
        ref = oracle.apply_h(q, q.psi)
        y = b.apply_h(dp, x, prec).cpu().numpy()
        assert np.max(np.abs(y - ref)) / np.max(np.abs(ref)) < 1e-5
