"""The sum over K splits of a projection: split counts on both sides of every group size of the
reduction, element counts that leave a work-group part empty, through the gradient of D and the
nonlocal force (bars as in test_gpu_backward and test_gpu_force: relative max-norm 1e-12 against
the FP64 oracle). With the default chunks the sum must take less time than the product whose
splits it adds: in one chain per element it took 38 us after a product of 18 at 32 projectors x 16
bands x 20,000 plane waves.
"""
import numpy as np
import pytest

import oracle
from paper_2501_08697_amd import workload as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def err(a, ref):
    return np.max(np.abs(a.cpu().numpy() - ref)) / np.max(np.abs(ref))


@pytest.mark.parametrize("chunk", [0, 16, 32, 96, 400])
@pytest.mark.parametrize("natom,nb", [(1, 1), (5, 7)])
def test_split_counts(chunk, natom, nb):
    from paper_2501_08697_amd import binding as b
    p = W.make_problem(W.tiny_config(a=10.0, ecut=20.0, fft=32, natom=natom, lmax=1, nb=nb, seed=4,
                                     with_grad_inputs=True))
    occ = W.band_weights(p, 5)
    splits = -(-int(p.npw[0]) // chunk) if chunk else None   # 94, 47, 16 and 4
    print(f"[split sums] npw={int(p.npw[0])} splits={splits} nproj={p.nproj} nb={nb}", flush=True)
    dp, x, g = b.DeviceProblem(p), torch.from_numpy(p.psi).cuda(), torch.from_numpy(p.dy).cuda()
    try:
        b.set_tuning(splitk_chunk=chunk)
        gd = b.apply_h_backward(dp, x, g, want=("d",))[2]
        f = b.force_nl(dp, x, occ)
    finally:
        b.set_tuning()
    assert err(gd, oracle.apply_h_backward(p, p.psi, p.dy)[2]) < 1e-12
    assert err(f, oracle.force_nl(p, p.psi, occ)) < 1e-12


def test_sum_takes_less_time_than_its_product():
    from paper_2501_08697_amd import binding as b
    p = W.make_problem(W.tiny_config(a=20.5, ecut=27.0, fft=72, natom=8, lmax=1, nb=16, seed=4, with_grad_inputs=True))
    dp, x, g = b.DeviceProblem(p), torch.from_numpy(p.psi).cuda(), torch.from_numpy(p.dy).cuda()
    b.apply_h_backward(dp, x, g, want=("d",))
    try:
        b.profile_enable()
        b.profile_read()
        for _ in range(20):
            b.apply_h_backward(dp, x, g, want=("d",))
        rec = b.profile_read()
    finally:
        b.profile_enable(False)
    print(f"[split sums] {rec}", flush=True)
    assert rec["gemm_reduce"][1] < rec["gemm_cn"][1]
