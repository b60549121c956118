"""Spheres wider than a quarter of the grid, on both sides of the rule that sends them through the column
passes: planes with more slab rows and columns than the kernels keep roles for in registers, or
alone on their CU with 512 threads. The kernels that ran are named. Bars as in test_gpu_apply_h:
relative max-norm 1e-12 in FP64, 1e-5 in FP32, against the oracle.
"""
import math

import numpy as np
import pytest

import oracle
from paper_2501_08697_amd import workload as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,fill,prec,columns", [
    (90, 3.8, 0, True), (90, 2.95, 0, True), (81, 2.95, 0, True), (72, 2.7, 0, True), (96, 2.95, 0, True),
    (108, 2.9, 0, True), (48, 2.2, 0, True), (96, 2.7, 0, False), (80, 2.7, 0, False), (72, 2.3, 0, False),
    (48, 2.2, 1, True), (80, 3.5, 1, True), (80, 3.0, 1, False)])
def test_wide_spheres(n, fill, prec, columns):
    """fill: grid length over the sphere's radius in Miller indices."""
    from paper_2501_08697_amd import binding as b
    a = round(n / fill * 2 * math.pi / math.sqrt(29.7), 2)
    p = W.make_problem(W.tiny_config(a=a, ecut=29.7, fft=n, kfrac=((0.0, 0.0, 0.0), (0.25, 0.375, 0.5)), natom=1, nb=3))
    print(f"[wide] fft={p.fft} npw={list(p.npw)} |m|={np.abs(p.miller).max(0)} prec={prec}", flush=True)
    x = torch.from_numpy(p.psi).cuda()
    try:
        b.profile_enable()
        b.profile_read()
        y = b.apply_h(b.DeviceProblem(p), x.to(torch.complex64) if prec else x, prec).cpu().numpy()
        names = set(b.profile_read())
    finally:
        b.profile_enable(False)
    ref = oracle.apply_h(p, p.psi)
    assert np.max(np.abs(y - ref)) < (1e-5 if prec else 1e-12) * np.max(np.abs(ref))
    assert ("plane" in names) == columns and ("xpass" in names) != columns, names
