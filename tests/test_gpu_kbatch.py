"""Projector GEMMs of several k-points in one launch, and short K chunks: more k-points than one
launch takes, uneven spheres, tile edges in projectors (64) and bands (64), against the oracle.
Bars as in test_gpu_apply_h: relative max-norm 1e-12 in FP64, 1e-5 in FP32.
"""
import numpy as np
import pytest

import oracle
from paper_2501_08697_amd import workload as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

K10 = tuple((0.05 * i, 0.04 * i - 0.2, 0.5 - 0.07 * i) for i in range(10))


@pytest.mark.parametrize("nk,natom,lmax,nb", [(1, 1, 1, 1), (8, 7, 2, 33), (9, 16, 1, 64), (10, 13, 1, 65)])
@pytest.mark.parametrize("prec", [0, 1])
def test_batched_kpoints_match_oracle(nk, natom, lmax, nb, prec):
    from paper_2501_08697_amd import binding as b
    p = W.make_problem(W.tiny_config(a=7.0, ecut=14.0, fft=18, kfrac=K10[:nk], natom=natom, lmax=lmax, nb=nb,
                                     dfull=lmax > 1, seed=21))
    print(f"[kbatch] nk={nk} npw={list(p.npw)} nproj={p.nproj} nb={nb} prec={prec}", flush=True)
    x = torch.from_numpy(p.psi).cuda()
    if prec == b.FP32:
        x = x.to(torch.complex64)
    y = b.apply_h(b.DeviceProblem(p), x, prec).cpu().numpy()
    ref = oracle.apply_h(p, p.psi)
    assert np.max(np.abs(y - ref)) / np.max(np.abs(ref)) < (1e-12 if prec == 0 else 1e-5)
