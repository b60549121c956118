"""The band weights of the nonlocal force are formed as the projection's splits are summed: four
launches per k-point. Above the projector count which that kernel takes (4,096) they come from a
kernel of their own. Bar as in test_gpu_force: relative max-norm 1e-12 against the FP64 oracle.
"""
import numpy as np
import pytest

import oracle
from paper_2501_08697_amd import workload as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("natom,lmax,nb,nk,launches", [(3, 1, 5, 3, 4), (455, 2, 2, 1, 4), (456, 2, 2, 1, 5)])
def test_launches_per_kpoint(natom, lmax, nb, nk, launches):
    from paper_2501_08697_amd import binding as b
    kfrac = ((0.0, 0.0, 0.0), (0.3, -0.2, 0.1), (0.5, 0.5, 0.25))[:nk]
    p = W.make_problem(W.tiny_config(a=7.0, ecut=13.0, fft=18, kfrac=kfrac, natom=natom, lmax=lmax, nb=nb,
                                     dfull=lmax > 1, seed=9))
    occ = W.band_weights(p, 5)
    print(f"[force launches] npw={list(p.npw)} nproj={p.nproj} nb={nb}", flush=True)
    dp, x = b.DeviceProblem(p), torch.from_numpy(p.psi).cuda()
    b.force_nl(dp, x, occ)
    try:
        b.profile_enable()
        b.profile_read()
        f = b.force_nl(dp, x, occ).cpu().numpy()
        rec = b.profile_read()
    finally:
        b.profile_enable(False)
    ref = oracle.force_nl(p, p.psi, occ)
    assert np.max(np.abs(f - ref)) / np.max(np.abs(ref)) < 1e-12
    assert sum(n for n, _ in rec.values()) == launches * nk, rec
