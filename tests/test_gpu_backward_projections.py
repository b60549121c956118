"""The gradient of D where it reads the projections that H dY made, and where it makes its own (no
gradient of psi wanted): projector counts around the 64 a work-group takes, band counts around its
16 groups, several k-points, atoms of one to nine projectors, against the oracle.
Bars as in test_gpu_backward: relative max-norm 1e-12 in FP64, 1e-5 in FP32.
"""
import numpy as np
import pytest

import oracle
from paper_2501_08697_amd import workload as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("natom,lmax,nb", [(1, 0, 1), (16, 1, 15), (13, 2, 17), (65, 0, 33)])
@pytest.mark.parametrize("prec", [0, 1])
def test_grad_d_with_and_without_grad_psi(natom, lmax, nb, prec):
    from paper_2501_08697_amd import binding as b
    p = W.make_problem(W.tiny_config(fft=16, ecut=16.0, nb=nb, kfrac=((0.1, 0.2, -0.1), (0.5, 0.0, 0.0), (0.0, 0.3, 0.4)),
                                     lmax=lmax, dfull=lmax > 1, natom=natom, with_grad_inputs=True))
    print(f"[backward] nproj={p.nproj} nb={nb} prec={prec}", flush=True)
    dp = b.DeviceProblem(p)
    dt = torch.complex128 if prec == 0 else torch.complex64
    x, g = (torch.from_numpy(a).cuda().to(dt) for a in (p.psi, p.dy))
    ref = oracle.apply_h_backward(p, p.psi, p.dy)[2]
    tol = 1e-12 if prec == 0 else 1e-5
    for want in (("psi", "v", "d"), ("d",), ("psi", "d")):
        gd = b.apply_h_backward(dp, x, g, prec, nb=nb, want=want)[2].cpu().numpy()
        assert np.max(np.abs(gd - ref)) <= tol * np.max(np.abs(ref)), want
