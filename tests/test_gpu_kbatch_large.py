"""Eight k-points whose spheres together have more column tiles than one launch's grid holds (589,000
plane waves each at 128^3, which FP32 runs): the accumulation takes fewer of them at a time. Against the
same k-points one by one; only the K chunks of the projection differ, so the FP32 bar of
test_gpu_apply_h holds: relative max-norm 1e-5.
"""
import dataclasses
import itertools

import numpy as np
import pytest

from paper_2501_08697_amd import workload as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_eight_large_spheres():
    from paper_2501_08697_amd import binding as b
    ks = tuple(itertools.product((0.0, 0.5), repeat=3))
    p = W.make_problem(W.tiny_config(a=30.0, ecut=118.6, fft=128, kfrac=ks, natom=1, lmax=0, nb=1))
    tiles = sum(-(-int(n) // 64) for n in p.npw)
    print(f"[large spheres] npw={list(p.npw)} tiles={tiles}", flush=True)
    assert tiles > 65536
    x = torch.from_numpy(p.psi).cuda().to(torch.complex64)
    y = b.apply_h(b.DeviceProblem(p), x, b.FP32).cpu().numpy()
    off = np.concatenate([[0], np.cumsum(p.npw)])
    for k in range(p.nk):
        g = slice(off[k], off[k + 1])
        q = dataclasses.replace(p, kpts=p.kpts[k:k + 1], npw=p.npw[k:k + 1], miller=np.ascontiguousarray(p.miller[g]),
                                beta=np.ascontiguousarray(p.beta[p.nproj * off[k]:p.nproj * off[k + 1]]))
        xk = torch.from_numpy(np.ascontiguousarray(p.psi_k(k)).reshape(-1)).cuda().to(torch.complex64)
        yk = b.apply_h(b.DeviceProblem(q), xk, b.FP32, nb=1).cpu().numpy()
        assert np.max(np.abs(yk - p.psi_k(k, y).reshape(-1))) <= 1e-5 * np.max(np.abs(yk)), k
