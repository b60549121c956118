"""The column passes on spheres wider than a quarter of the grid, where a plane has more slab rows and
columns than the kernels keep roles for in registers, or is alone on its CU with 512 threads. Bars as
in test_gpu_apply_h: relative max-norm 1e-12 in FP64, 1e-5 in FP32, against the oracle.
"""
import math

import numpy as np
import pytest

import oracle
from paper_2501_08697_amd import workload as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,fill,prec", [(90, 3.8, 0), (90, 2.9, 0), (80, 2.7, 0), (81, 2.9, 0), (72, 2.2, 0),
                                         (96, 2.7, 0), (48, 2.2, 1), (80, 2.7, 1)])
def test_wide_spheres(n, fill, prec):
    """fill: grid length over the sphere's radius in Miller indices."""
    from paper_2501_08697_amd import binding as b
    a = round(n / fill * 2 * math.pi / math.sqrt(29.7), 2)
    p = W.make_problem(W.tiny_config(a=a, ecut=29.7, fft=n, kfrac=((0.0, 0.0, 0.0), (0.25, 0.375, 0.5)), natom=1, nb=3))
    print(f"[wide] fft={p.fft} npw={list(p.npw)} |m|={np.abs(p.miller).max(0)} prec={prec}", flush=True)
    x = torch.from_numpy(p.psi).cuda()
    y = b.apply_h(b.DeviceProblem(p), x.to(torch.complex64) if prec else x, prec).cpu().numpy()
    ref = oracle.apply_h(p, p.psi)
    assert np.max(np.abs(y - ref)) < (1e-5 if prec else 1e-12) * np.max(np.abs(ref))
