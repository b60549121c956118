"""Nonlocal force at the edges of its product's tiles (64 projectors x 64 plane waves, 16 bands a
stage) and over several k-points, against the FP64 oracle. Bar as in test_gpu_force: relative
max-norm 1e-12.
"""
import numpy as np
import pytest

import oracle
from paper_2501_08697_amd import workload as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("natom,lmax,nb,nk", [(1, 0, 1, 1), (16, 1, 16, 2), (13, 1, 17, 3), (15, 2, 33, 1)])
def test_force_tile_edges(natom, lmax, nb, nk):
    from paper_2501_08697_amd import binding as b
    kfrac = ((0.0, 0.0, 0.0), (0.3, -0.2, 0.1), (0.5, 0.5, 0.25))[:nk]
    p = W.make_problem(W.tiny_config(a=7.0, ecut=13.0, fft=18, kfrac=kfrac, natom=natom, lmax=lmax, nb=nb,
                                     dfull=lmax > 1, seed=9))
    occ = W.band_weights(p, 5)
    print(f"[force tiles] npw={list(p.npw)} nproj={p.nproj} nb={nb}", flush=True)
    f = b.force_nl(b.DeviceProblem(p), torch.from_numpy(p.psi).cuda(), occ).cpu().numpy()
    ref = oracle.force_nl(p, p.psi, occ)
    assert np.max(np.abs(f - ref)) / np.max(np.abs(ref)) < 1e-12
